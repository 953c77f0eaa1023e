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


def _batch_cfgs(storage, kind):
    """Batches that take each region shape (16 x 16, 32 x 16, 32 x 32; FP64
    the first two), ragged and with every boundary kind."""
    rb = lambda n, **k: W.rayleigh_benard(2, n, ra=5e4, pr=0.71, storage=storage, **k)  # noqa: E731
    if kind == "small":
        return [rb((33, 17)), W.side_heated(2, (41, 41), ra=1e6, storage=storage), rb((66, 33), lateral="periodic"),
                rb((3, 2)), rb((130, 57))]
    if kind == "mid":
        return [rb((129, 129)), rb((193, 97)), W.side_heated(2, (65, 66), ra=1e5, storage=storage),
                rb((200, 200), lateral="periodic")]
    return [rb((257, 257)), rb((513, 257)), W.side_heated(2, (300, 127), ra=1e5, storage=storage)]


@pytest.mark.parametrize("storage", ["fp32", "fp64", "fp16", "bf16", "mixed"])
@pytest.mark.parametrize("kind", ["small", "mid", "big"])
def test_batch_tile_launches_equal_single_steps(storage, kind):
    """The default launches of a batch (and their graph replay, checked after
    each) against the same batch in single steps: fields, wall fluxes and
    Nusselt numbers bit for bit."""
    cfgs = _batch_cfgs(storage, kind)
    seeds = [3 + k for k in range(len(cfgs))]
    one, default, graph = (lbm.Batch(cfgs) for _ in range(3))
    one.steps_per_launch = 1
    graph.set_config(graph_steps=14)
    for b in (one, default, graph):
        b.init(seeds, [2e-2] * len(cfgs))
    for n in (5, 14, 3, 28):
        for b in (one, default, graph):
            b.step(n)
        assert not default.unstable().any()
        for k in range(len(cfgs)):
            ref = one.cavity(k).fields()
            for b in (default, graph):
                got = b.cavity(k)
                assert all(np.array_equal(x, y) for x, y in zip(ref, got.fields())), (n, k)
                assert np.array_equal(one.cavity(k).wall_flux(), got.wall_flux()), (n, k)
        assert np.array_equal(np.nan_to_num(one.nusselt()), np.nan_to_num(default.nusselt()))


def test_batch_tiles_flag_a_diverging_member_only():
    cfgs = [W.rayleigh_benard(2, (65, 65), ra=1e5, pr=0.71, storage="fp32") for _ in range(3)]
    b = lbm.Batch(cfgs)
    b.init([1, 2, 3], [1e-3] * 3)
    n = 65 * 65
    u = np.zeros((2, n))
    u[0, n // 2] = 0.9  # faster than the lattice sound speed
    b.init_fields(1, None, u, np.full(n, 0.5))
    b.step(5)
    assert b.unstable().tolist() == [False, True, False]


def test_autotuner_leaves_wall_flux_and_state_to_its_steps():
    """The tile launches the autotuner times do not advance the batch: after
    tuning, state and Nusselt numbers are those of t single steps."""
    cfgs = _batch_cfgs("fp32", "mid")
    a, b = lbm.Batch(cfgs), lbm.Batch(cfgs)
    b.steps_per_launch = 1
    for x in (a, b):
        x.init([1] * len(cfgs), [1e-2] * len(cfgs))
    a.tune(steps=1)
    b.step(a.t)
    for extra in (0, 7):
        a.step(extra)
        b.step(extra)
        assert np.array_equal(a.nusselt(), b.nusselt())
        for k in range(len(cfgs)):
            assert all(np.array_equal(x, y) for x, y in zip(a.cavity(k).fields(), b.cavity(k).fields()))
