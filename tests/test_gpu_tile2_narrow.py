"""A grid of a few columns and so many rows that the default tiles of FP64 storage
would need 2^32 threads in one launch: it takes the launches of a set count."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


def test_more_tiles_than_a_launch_holds():
    import torch
    cfg = W.rayleigh_benard(2, (3, 84_000_000), ra=1e4, pr=0.71, storage="fp64")
    if torch.cuda.mem_get_info()[0] < 80e9:
        pytest.skip("needs 60 GB of device memory")
    seen = []
    for spl in (0, 1):
        c = lbm.Cavity(cfg)
        if spl:
            c.steps_per_launch = spl
        c.init(1, 1e-3)
        c.step(5)
        seen.append((c.diagnostics(), c.nusselt()))
        c.close()
        del c
        torch.cuda.empty_cache()
    assert seen[0] == seen[1]
    assert seen[0][0]["nonfinite"] == 0
