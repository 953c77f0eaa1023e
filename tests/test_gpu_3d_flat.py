"""The default launches of flat and thin 3D grids on either side of the rule that
chooses between one and two steps per launch (42 thousand nodes per plane step
of the two-step kernel, or 250 thousand in all), against both counts set: the
whole exported state must be bitwise identical."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(400, 200, 3), (400, 200, 2), (300, 300, 2), (128, 512, 3), (350, 350, 2), (16, 3, 5000)])
def test_default_launches_bitwise(shape):
    cfg = W.rayleigh_benard(3, shape, ra=1e5, pr=0.71, storage="fp32")
    got = []
    for spl in (0, 1, 2):
        c = lbm.Cavity(cfg)
        if spl:
            c.steps_per_launch = spl
        c.init(5, 2e-2)
        for n in (1, 2, 5):
            c.step(n)
        got.append(c.export_state())
    same = got[0] == got[1] == got[2]
    assert same
