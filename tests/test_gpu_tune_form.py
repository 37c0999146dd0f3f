"""The autotuner's PCG grid of a mesh whose product does not use one (at most 384 tiles) stays with such meshes: a
larger mesh of the same size bucket finds its own."""
import json

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg
import pytest

from gpu_util import ctx, note

pytestmark = pytest.mark.gpu


def test_small_mesh_grid_does_not_reach_a_larger_one(tmp_path):
    cache = tmp_path / "tune.json"
    small = mg.kuhn_cube(1, patches="channel", nxyz=(36, 36, 36))   # 279,936 cells, 274 tiles
    large = mg.kuhn_cube(1, patches="channel", nxyz=(38, 38, 47))   # 407,208 cells, 398 tiles
    assert -(-small.n_cells // 1024) <= 384 < -(-large.n_cells // 1024)
    assert small.n_cells.bit_length() == large.n_cells.bit_length()
    Ms, Ml = B.Mesh(ctx(), small), B.Mesh(ctx(), large)
    B.difvm_mesh_set_launch(Ms.h, B.TUNE_PCG_GRID, 512)
    assert B.difvm_tune(Ms.h, cache) == len(B.TUNE_KNOBS)
    assert B.difvm_mesh_get_launch(Ms.h, B.TUNE_PCG_GRID) == 0
    n = B.difvm_tune(Ml.h, cache)
    grid = B.difvm_mesh_get_launch(Ml.h, B.TUNE_PCG_GRID)
    entries = {k: v for k, v in json.loads(cache.read_text()).items() if "|pcg_grid|" in k}
    note("tuned grids", entries)
    assert n == 1 and len(entries) == 2 and sorted(entries.values()) == sorted((0, grid))
    for M, g in ((Ms, 0), (Ml, grid)):  # both found again
        assert B.difvm_tune(M.h, cache) == 0 and B.difvm_mesh_get_launch(M.h, B.TUNE_PCG_GRID) == g
