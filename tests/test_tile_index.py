"""Tile index 0 leaves the choice to the library and is no shape of its own; every shape, 8x28 included,
has an explicit index, and the autotuner times each shape once and stores explicit indices only."""
import pytest

from paper_2402_10914_amd import api, autotune

SHAPES = {(8, 28), (16, 28), (8, 60), (16, 12), (4, 60)}


def test_every_shape_has_one_explicit_index():
    shapes = api.tile_shapes()
    assert shapes[0] == (0, 0)  # not the shape that a call with index 0 happens to take
    assert len(shapes) == len(SHAPES) + 1 and set(shapes[1:]) == SHAPES


class _Clock:
    """Stands for the timing of one candidate: records the tile and prefers the last one asked for."""

    def __init__(self):
        self.tiles = []

    def __call__(self, grids, Ws, alphas, params, dtype, order, steps, reps):
        self.tiles.append(params.tile)
        return 1.0 / len(self.tiles)


def test_tuner_times_every_shape_and_keys_by_the_list(tmp_path, monkeypatch):
    monkeypatch.setenv("DFW_TUNE_CACHE", str(tmp_path / "tuning.json"))
    clock = _Clock()
    monkeypatch.setattr(autotune, "_time_batch", clock)
    shapes = api.tile_shapes()
    grids = [(8, 9, 0.1, 0.1, 0, 0)]
    tile, order, timings = autotune.tune_batch(grids, None, None, api.Params(), steps=1)
    assert sorted(set(clock.tiles)) == list(range(1, len(shapes)))
    assert len(clock.tiles) == 3 * (len(shapes) - 1)
    assert shapes[tile] in SHAPES
    # an entry stored under a list in which index 0 was a shape does not answer for this one
    with monkeypatch.context() as m:
        m.setattr(api, "tile_shapes", lambda: [(8, 28), (16, 28), (8, 60), (16, 12), (4, 60)])
        before = autotune._key("batch", [(8, 9, 0, 0)], api.torch.float64, api.Params())
    assert before != autotune._key("batch", [(8, 9, 0, 0)], api.torch.float64, api.Params())


@pytest.mark.parametrize("tile", [-1, 6])
def test_index_outside_the_list_is_refused(tile):
    import ctypes

    from paper_2402_10914_amd import _lib
    tf = ctypes.c_int32()
    assert _lib.load().dfw_tile_shape(tile, ctypes.byref(tf), ctypes.byref(tf)) == _lib.DFW_EINVAL
