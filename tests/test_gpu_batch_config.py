"""Batches whose configuration changes between steps: captured graphs, the
autotuner's choice and explicit counts must leave the state where single steps
put it, bit for bit."""
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(33, 17), (66, 33), (41, 41), (130, 57)]
LARGE = [(513, 513)] * 16  # streaming beats one step per launch, tiles beat streaming


def _batch(storage, shapes=SHAPES):
    b = lbm.Batch([W.rayleigh_benard(2, s, ra=5e4, pr=0.71, storage=storage) for s in shapes])
    return b


def _init(b):
    b.init([3 + k for k in range(b.count)], [2e-2] * b.count)


def _same_as_single_steps(b, storage, shapes=SHAPES):
    one = _batch(storage, shapes)
    one.steps_per_launch = 1
    _init(one)
    one.step(b.t)
    for k in range(b.count):
        same = b.cavity(k).export_state() == one.cavity(k).export_state()
        assert same, f"cavity {k} at t = {b.t}"


@pytest.mark.parametrize("storage,shapes,graph_steps", [
    ("fp32", SHAPES, 10), ("fp64", SHAPES, 10), ("fp16", LARGE, 4), ("bf16", LARGE, 12), ("fp32", LARGE, 20)])
def test_reapplied_configuration_after_tuning(storage, shapes, graph_steps):
    """Graphs captured after tuning, then the batch's own configuration set
    again, whole and with the streaming shape only: a graph of launches of
    another kind must not be replayed, whatever the parity of its launches."""
    b = _batch(storage, shapes)
    _init(b)
    b.set_config(graph_steps=graph_steps)
    b.tune(steps=3)
    b.step(2 * graph_steps)
    cfg = b.config()
    b.set_config(**cfg)
    b.step(graph_steps)
    _same_as_single_steps(b, storage, shapes)
    cfg.pop("tiles", None)
    b.set_config(**cfg)
    b.step(2 * graph_steps)
    _same_as_single_steps(b, storage, shapes)
    # a count that is set, with graphs of the former launches at hand
    b.steps_per_launch = 2
    b.step(2 * graph_steps + 3)
    _same_as_single_steps(b, storage, shapes)


@pytest.mark.parametrize("storage,shapes", [("fp16", LARGE), ("fp64", SHAPES)])
def test_tuned_choice_is_part_of_the_configuration(storage, shapes):
    """Giving the tuner's configuration back, changed in its graphs only,
    keeps the launches it chose, on this batch and on a new one."""
    b = _batch(storage, shapes)
    _init(b)
    assert b.config() == dict(block=256, grid_per_cu=0, graph_steps=0, stream_rows=0, stream_waves=0)
    tiles = b.launch_steps
    assert tiles in (4, 5) and tiles != b.steps_per_launch
    best, _ = b.tune(steps=3)
    chosen = b.launch_steps
    assert chosen == (tiles if "tiles" in best else b.steps_per_launch)
    b.set_config(**{**best, "graph_steps": 8})
    assert b.launch_steps == chosen
    b.step(27)
    _same_as_single_steps(b, storage, shapes)
    c = _batch(storage, shapes)
    if "tiles" not in best:
        c.steps_per_launch = b.steps_per_launch
    c.set_config(**best)
    assert c.launch_steps == chosen


def test_launch_kind_follows_the_configuration():
    b = _batch("fp16")
    tiles, count = b.launch_steps, b.steps_per_launch
    b.set_config(graph_steps=4, block=128)
    assert b.launch_steps == tiles
    b.set_config(stream_rows=24)
    assert b.launch_steps == count
    b.set_config(**b.config())
    assert b.launch_steps == count
    b.set_config(stream_rows=24, tiles=1)
    assert b.launch_steps == tiles
    with pytest.raises(lbm.LBMError):
        b.set_config(stream_rows=5, stream_waves=4)  # refused: nothing changes
    assert b.launch_steps == tiles
    b.steps_per_launch = count  # a count that is set is taken exactly
    assert b.launch_steps == count
    b.set_config(tiles=1)
    assert b.launch_steps == count


@pytest.mark.parametrize("storage,shapes", [("fp16", [(700, 700)] * 4 + [(300, 203)]), ("fp16", [(700, 700)] * 4),
                                            ("bf16", LARGE), ("fp64", [(700, 700)] * 5)])
def test_steps_left_over_by_tiles(storage, shapes):
    """Every remainder of the tile launches, on either side of the two million
    nodes from which FP16 streams three steps, launched and from graphs."""
    b = _batch(storage, shapes)
    _init(b)
    for n in (1, 2, 3, 5, 6, 7):
        b.step(n)
    _same_as_single_steps(b, storage, shapes)
    b.set_config(graph_steps=14)
    b.step(31)
    _same_as_single_steps(b, storage, shapes)
