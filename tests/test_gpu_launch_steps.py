"""What a launch advances, the bytes per update that follow from it, and the way
back from a count that was set."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

# small, mid-size and large grids of each rule: 2D tiles of 5 or 4 steps and the
# streaming counts above them, 3D one step and two
CASES = [(2, (65, 65), "fp32", 5), (2, (65, 65), "fp16", 5), (2, (129, 129), "fp64", 5), (2, (300, 300), "fp64", 4),
         (2, (1025, 700), "fp16", 4), (2, (1025, 700), "fp32", 5), (2, (3000, 3001), "fp16", 3),
         (2, (3000, 23), "bf16", 4), (3, (33, 33, 33), "fp32", 1), (3, (65, 65, 65), "fp32", 2),
         (3, (400, 200, 3), "fp32", 2), (3, (65, 65, 65), "mixed", 1)]


@pytest.mark.parametrize("dim,shape,storage,steps", CASES)
def test_launch_steps_and_bytes_per_update(dim, shape, storage, steps):
    cfg = W.rayleigh_benard(dim, shape, ra=1e4, pr=0.71, storage=storage)
    c = lbm.Cavity(cfg)
    count = c.steps_per_launch
    assert c.launch_steps == steps
    assert c.bytes_per_update() == lbm.bytes_per_update(cfg) / steps
    c.steps_per_launch = 1
    assert c.launch_steps == c.steps_per_launch == 1 and c.bytes_per_update() == lbm.bytes_per_update(cfg)
    c.steps_per_launch = count  # taken exactly, where the grid can
    assert c.launch_steps == count
    c.reset_steps_per_launch()
    assert c.launch_steps == steps and c.steps_per_launch == count


def test_batch_members_step_with_their_batch():
    b = lbm.Batch([W.rayleigh_benard(2, (33, 17), ra=1e4, pr=0.71, storage="fp32")])
    v = b.cavity(0)
    assert v.launch_steps == 1
    with pytest.raises(lbm.LBMError) as e:
        v.reset_steps_per_launch()
    assert e.value.status == -4
