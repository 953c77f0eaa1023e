"""The default launches of 3D grids on both sides of the node count that
chooses between one and two steps per launch, against both counts set: the
whole exported state must be bitwise identical."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


# 248,976 and 250,047 nodes (the rule's line is 250,000), and small ones
@pytest.mark.parametrize("shape", [(63, 63, 63), (64, 63, 62), (62, 64, 63), (5, 3, 2), (31, 17, 65)])
@pytest.mark.parametrize("storage", ["fp32", "mixed"])
def test_default_launches_bitwise(shape, storage):
    for cfg in (W.rayleigh_benard(3, shape, ra=1e5, pr=0.71, storage=storage),
                W.periodic_box(3, shape, nu=0.02, alpha=0.03, gbeta=1e-4, storage=storage)):
        got = []
        for spl in (0, 1, 2):
            c = lbm.Cavity(cfg)
            if spl:
                c.steps_per_launch = spl
            c.init(5, 2e-2)
            for n in (1, 2, 5):
                c.step(n)
            got.append(c.export_state())
        assert got[0] == got[1] == got[2]
