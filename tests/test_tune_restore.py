"""The tuners leave a table or plan as they found it when they are not to apply
what they found: with the shape that was set, or with none, in which the
library picks the shape itself."""

import pytest

from gpu_util import say, to_dev, u64, u8, vals_dev
from paper_1712_09624_amd import ckpp, tune
from paper_1712_09624_amd import workload as W

SHAPES = [{"lanes_per_lookup": 8, "lookups_per_lane": 1, "block": 64, "blocks_per_cu": 0},
          {"lanes_per_lookup": 1, "lookups_per_lane": 4, "block": 256, "blocks_per_cu": 8}]
PLAN_SHAPES = [dict(zip(("lookups_per_lane", "block", "blocks_per_cu", "passes_per_item",
                         "schedule", "lanes_per_lookup"), s))
               for s in ((2, 64, 4, 2, 0, 8), (1, 256, 16, 1, 1, 1))]


class Stub:
    """The launch-shape calls of a table and of a plan, on the host alone."""

    def __init__(self, names, start):
        self.names, self.start = names, start
        self.shape, self.launch_set = dict(start), False

    def set_launch(self, *shape):
        self.shape, self.launch_set = dict(zip(self.names, shape)), True

    def get_launch(self):
        return dict(self.shape)

    def reset_launch(self):
        self.shape, self.launch_set = dict(self.start), False

    set_lookup_launch, get_lookup_launch, reset_lookup_launch = set_launch, get_launch, reset_launch


def stub_and_tuner(kind, monkeypatch):
    if kind == "table":
        import torch
        ms = iter([2.0, 1.0])
        monkeypatch.setattr(tune, "time_lookup", lambda *a, **k: next(ms))
        stub = Stub(list(SHAPES[0]), ckpp.DEFAULT_LAUNCH)
        keys = torch.empty(4, 16, dtype=torch.uint8)
        return stub, lambda apply: tune.tune(stub, [keys], shapes=SHAPES, apply=apply), SHAPES
    ms = iter([2.0, 1.0])
    monkeypatch.setattr(tune, "time_plan", lambda *a, **k: next(ms))
    stub = Stub(list(PLAN_SHAPES[0]), ckpp.DEFAULT_PLAN_LAUNCH)
    return stub, lambda apply: tune.tune_plan(stub, None, None, None, shapes=PLAN_SHAPES,
                                              apply=apply), PLAN_SHAPES


@pytest.mark.parametrize("was_set", [False, True], ids=["unset", "set"])
@pytest.mark.parametrize("kind", ["table", "plan"])
def test_tuner_restores(kind, was_set, monkeypatch):
    stub, tuner, shapes = stub_and_tuner(kind, monkeypatch)
    if was_set:
        stub.set_launch(*shapes[0].values())
    before = (stub.get_launch(), stub.launch_set)
    tuner(False)
    assert (stub.get_launch(), stub.launch_set) == before


@pytest.mark.parametrize("kind", ["table", "plan"])
def test_tuner_applies(kind, monkeypatch):
    stub, tuner, shapes = stub_and_tuner(kind, monkeypatch)
    tuner(True)
    assert (stub.get_launch(), stub.launch_set) == (shapes[1], True)


def test_reset_refuses_null_handles():
    lib = ckpp.load()
    assert lib.ckpp_reset_lookup_launch(None) == ckpp.EINVAL
    assert lib.ckpp_plan_reset_launch(None) == ckpp.EINVAL


@pytest.mark.gpu
def test_reset_on_the_gpu():
    n = W.keys_at_load(10, 0.8)
    keys = W.distinct_five_tuples(n, 90)
    t = ckpp.Table(10, W.HASH_SEED, W.MAX_KICKS, device=0)
    t.insert(to_dev(keys), vals_dev(W.insertion_values(n)))
    plan = ckpp.Plan([t], [0], [n])
    items = plan.info()["nitems"]
    plan.set_launch(2, 64, 4, 2)
    assert plan.info()["nitems"] < items and plan.launch_set
    plan.reset_launch()
    assert plan.get_launch() == ckpp.DEFAULT_PLAN_LAUNCH and not plan.launch_set
    assert plan.info()["nitems"] == items
    t.set_lookup_launch(4, 1, 64, 0)
    t.reset_lookup_launch()
    assert t.get_lookup_launch() == ckpp.DEFAULT_LAUNCH and not t.launch_set
    say("lookups after the shapes were reset")
    for f, v in (plan.lookup(to_dev(keys)), t.lookup(to_dev(keys))):
        assert u8(f).all() and (u64(v) == W.insertion_values(n)).all()
    plan.close()
    t.close()
