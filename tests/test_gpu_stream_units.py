"""The order of the streaming kernel's work units and its row segments against
one step per launch: the whole exported state must be bitwise identical, with
the destination poisoned before each launch, so that a unit left out shows.

Widths around two and three strips (54 columns in FP32 at five steps, 56 at
four, 58 at three), one column into a new strip, and heights of one segment,
two, and more than one and two groups of 16 segments."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(108, 47), (109, 48), (162, 385), (163, 1000), (175, 49), (240, 800)]
STEPS = {"fp32": (5, 4), "fp16": (3,), "bf16": (4,), "mixed": (4,), "fp64": (2,)}


def _layouts(shape, storage):
    return {"rb": W.rayleigh_benard(2, shape, ra=5e4, pr=0.71, storage=storage),
            "rb_periodic": W.rayleigh_benard(2, shape, ra=5e4, pr=0.71, lateral="periodic", storage=storage),
            "side": W.side_heated(2, shape, ra=5e4, pr=0.71, storage=storage),
            "box": W.periodic_box(2, shape, nu=0.02, alpha=0.03, gbeta=1e-4, storage=storage)}


@pytest.mark.parametrize("storage", list(STEPS))
@pytest.mark.parametrize("shape", SHAPES)
def test_units_bitwise(storage, shape):
    for name, cfg in _layouts(shape, storage).items():
        got = {}
        for k in (1,) + STEPS[storage]:
            c = lbm.Cavity(cfg)
            c.steps_per_launch = k
            c.debug_poison = True
            c.init(11, 2e-2)
            c.step(11)
            got[k] = c.export_state()
        for k in STEPS[storage]:
            assert got[k] == got[1], (name, k)


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_batch_units_bitwise(storage, waves):
    cfgs = [c for s in ((163, 500), (109, 48), (20, 30)) for c in _layouts(s, storage).values()]
    b = lbm.Batch(cfgs)
    b.set_config(stream_waves=waves)
    b.steps_per_launch = STEPS[storage][0]
    b.init(list(range(len(cfgs))), [2e-2] * len(cfgs))
    b.step(11)
    for k, cfg in enumerate(cfgs):
        c = lbm.Cavity(cfg)
        c.steps_per_launch = 1
        c.init(k, 2e-2)
        c.step(11)
        assert b.cavity(k).export_state() == c.export_state(), k
    b.close()
