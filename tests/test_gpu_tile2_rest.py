"""Step counts that leave a remainder on grids whose remainder is streamed, and
on the largest whose is not, against one step per launch: the whole exported
state must be bitwise identical, with the destination poisoned."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

# either side of the node counts of the rule: FP32 2 M (four steps) and 2.8 M,
# FP16-f+FP32-g 3.5 M, FP16 and BF16 3.3 M (three) and 4.8 M (two)
SHAPES = {"fp32": [(1400, 1429), (1673, 1674)], "mixed": [(1870, 1872)], "fp16": [(1816, 1818), (2190, 2192)],
          "bf16": [(1816, 1818), (2190, 2192)], "fp64": [(1673, 1674)]}


@pytest.mark.parametrize("storage,shape", [(st, s) for st in SHAPES for s in SHAPES[st]])
@pytest.mark.parametrize("less", [0, 1])
def test_remainders_bitwise(storage, shape, less):
    cfg = W.rayleigh_benard(2, (shape[0], shape[1] - less), ra=1e6, pr=0.71, storage=storage)
    got = []
    for spl in (0, 1):
        c = lbm.Cavity(cfg)
        if spl:
            c.steps_per_launch = spl
        c.debug_poison = True
        c.init(3, 2e-2)
        for n in (2, 3, 4, 6, 7, 9):
            c.step(n)
        got.append(c.export_state())
    same = got[0] == got[1]
    assert same
