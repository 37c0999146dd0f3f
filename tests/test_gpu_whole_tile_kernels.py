"""The Krylov kernels of meshes above 384 tiles (a tile per block): the grid of the PCG product, whose blocks walk
several tiles and segments, and BiCGStab's totals in a kernel of their own."""
import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import ctx, dev, empty, host, note

pytestmark = pytest.mark.gpu


def tiles(starts):
    return sum(-(-int(c) // 1024) for c in np.diff(starts))


def small_members(n, big):
    """n members of one tile (48 tets each) with one of six tiles among them, which keeps every solve out of the
    one-block form"""
    one = mg.kuhn_cube(2, jitter=0.1, patches="walls", seed=5)
    ms = [one] * (n // 2) + [mg.kuhn_cube(10, jitter=0.1, patches="walls", seed=6)] * big + [one] * (n - n // 2)
    return ms, mg.pack(ms)


@pytest.mark.parametrize("packed", [False, True])
def test_pcg_grid_does_not_show(packed):
    if packed:
        _, (m, starts) = small_members(390, 1)
    else:
        m, starts = mg.kuhn_cube(1, jitter=0.1, patches="walls", seed=9, nxyz=(38, 38, 47)), None
    nt = tiles(starts) if packed else -(-m.n_cells // 1024)
    assert nt > 384
    M = B.Mesh(ctx(), m, seg_cell_start=starts)
    A = B.ldu(empty(m.n_cells), empty(m.n_internal_faces))
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(m.n_boundary_faces)), A, empty(m.n_cells))
    b = M.to_internal(dev(np.random.default_rng(2).standard_normal(m.n_cells)), B.KIND_CELL)
    ref = None
    for grid in (0, 8, 24, 104, 200, 256, 392, 4096):
        B.difvm_mesh_set_launch(M.h, B.TUNE_PCG_GRID, grid)
        x = b.clone().zero_()
        note("pcg grid", nt, grid)
        out = B.difvm_solve_pcg(M.h, A, b, x, 1e-10, 60), host(x)
        ref = ref or out
        assert out[0] == ref[0] and ref[0][1] > 5
        np.testing.assert_array_equal(out[1], ref[1], err_msg=f"grid {grid}")


def momentum(mesh, seg, flux, U, Ub, ncomp):
    M = B.Mesh(ctx(), mesh, seg_cell_start=seg)
    A = B.ldu(empty(mesh.n_cells), empty(mesh.n_internal_faces), empty(mesh.n_internal_faces))
    b = empty((mesh.n_cells, 3))
    B.difvm_ldu_assemble_momentum(M.h, 0.01, 1e-2, M.to_internal(dev(flux), B.KIND_FACE_FLUX),
                                  M.to_internal(dev(U), B.KIND_CELL), M.to_internal(dev(Ub), B.KIND_BFACE), A, b)
    if ncomp == 1:
        b = b[:, 1].contiguous()
    x = b.clone().zero_()
    st, it, _ = B.difvm_solve_bicgstab(M.h, A, ncomp, b, x, 1e-12, 200)
    assert st == 0
    return host(M.to_user(x, B.KIND_CELL)), it


@pytest.mark.parametrize("members", [378, 379])
@pytest.mark.parametrize("ncomp", [1, 3])
def test_bicgstab_on_either_side_of_the_limit(members, ncomp):
    """384 and 385 tiles: every member has the bits of its standalone solve (one block, or quarter-tile blocks)"""
    ms, (m, starts) = small_members(members, 1)
    assert tiles(starts) == members + 6
    rng = np.random.default_rng(8)
    flux = [0.1 * rng.standard_normal(k.n_faces) for k in ms]
    U, Ub = rng.standard_normal((m.n_cells, 3)), rng.standard_normal((m.n_boundary_faces, 3))
    packed = np.concatenate([f[:k.n_internal_faces] for f, k in zip(flux, ms)] +
                            [f[k.n_internal_faces:] for f, k in zip(flux, ms)])
    note("bicgstab tiles", members + 6, ncomp)
    x, it = momentum(m, starts, packed, U, Ub, ncomp)
    fb, most = np.cumsum([0] + [k.n_boundary_faces for k in ms]), []
    for k in (0, 1, members // 2 - 1, members // 2, members // 2 + 1, members):
        c = slice(starts[k], starts[k + 1])
        xk, itk = momentum(ms[k], None, flux[k], U[c], Ub[fb[k]:fb[k + 1]], ncomp)
        most.append(list(itk)[:ncomp])
        np.testing.assert_array_equal(x[c], xk)
    assert (np.max(most, axis=0) <= list(it)[:ncomp]).all() and np.min(most) >= 2
