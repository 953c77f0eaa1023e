"""The default launches of small and mid-size 2D grids (K steps per launch
through LDS tiles) against one step per launch: the whole exported state,
populations, wall-flux slots and t, must be bitwise identical.

The shapes sit at the edges of the rule and of the tiles: regions of 16 x 16
(8 x 8 stored), 32 x 16 (24 x 8, from about 33 thousand nodes; FP64 26 x 10)
and 32 x 32 (24 x 24 or 26 x 26, from about 200 thousand nodes), one node more
and less than whole tiles, grids smaller than a halo, grids that wrap inside
one region, and grids too low for tiles.  The step counts leave every
remainder."""
import numpy as np
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2), (1, 33), (40, 1), (5, 7), (8, 8), (9, 15), (65, 64), (129, 129), (193, 191), (240, 130),
          (641, 24), (313, 649), (520, 521), (3000, 23)]


def _state(cfg, spl, steps, poison=False):
    c = lbm.Cavity(cfg)
    if spl:
        c.steps_per_launch = spl
    c.debug_poison = poison
    c.init(17, 2e-2)
    for n in steps:
        c.step(n)
    return c.export_state()


@pytest.mark.parametrize("storage", ["fp32", "fp64", "fp16", "bf16", "mixed"])
@pytest.mark.parametrize("shape", SHAPES)
def test_default_launches_bitwise(storage, shape):
    layouts = {"box": W.periodic_box(2, shape, nu=0.02, alpha=0.03, gbeta=1e-4, storage=storage)}
    if min(shape) >= 2:
        layouts["rb"] = W.rayleigh_benard(2, shape, ra=5e4, pr=0.71, storage=storage)
        layouts["rb_periodic"] = W.rayleigh_benard(2, shape, ra=5e4, pr=0.71, lateral="periodic", storage=storage)
        layouts["side"] = W.side_heated(2, shape, ra=5e4, pr=0.71, storage=storage)
    for name, cfg in layouts.items():
        one = _state(cfg, 1, [24])
        # 1 + 2 + 3 + 4 + 5 + 9 steps: every remainder, both flux parities
        for steps, poison in (([1, 2, 3, 4, 5, 9], False), ([24], True)):
            got = _state(cfg, 0, steps, poison)
            if got != one:
                x, y = np.frombuffer(one, np.uint8), np.frombuffer(got, np.uint8)
                bad = np.flatnonzero(x != y)
                pytest.fail(f"{name} {shape} {storage} {steps}: {bad.size} bytes differ, first at {bad[:8]}")
