"""The solvers' dispatch by size must not show in the results: a member of a packed mesh keeps the bits of
its standalone solve on either side of each limit.

BiCGStab sums the tiles' partials in every block up to 384 tiles and in a kernel of its own above; many
tiny members reach the limit with few cells (a tile each)."""
import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg
from gpu_util import ctx, dev, empty, host, note

pytestmark = pytest.mark.gpu


def momentum_solve(mesh, seg, flux, U, Ub, ncomp):
    M = B.Mesh(ctx(), mesh, seg_cell_start=seg)
    nc, nfi = mesh.n_cells, mesh.n_internal_faces
    A = B.ldu(empty(nc), empty(nfi), empty(nfi))
    b = empty((nc, 3))
    B.difvm_ldu_assemble_momentum(M.h, 0.01, 1e-2, M.to_internal(dev(flux), B.KIND_FACE_FLUX),
                                  M.to_internal(dev(U), B.KIND_CELL), M.to_internal(dev(Ub), B.KIND_BFACE), A, b)
    if ncomp == 1:
        b = b[:, 1].contiguous()
    x = b.clone().zero_()
    st, it, _ = B.difvm_solve_bicgstab(M.h, A, ncomp, b, x, 1e-12, 200)
    assert st == 0
    return host(M.to_user(x, B.KIND_CELL)), it


@pytest.mark.parametrize("members", [384, 385])
@pytest.mark.parametrize("ncomp", [1, 3])
def test_bicgstab_totals_limit(members, ncomp):
    m = mg.kuhn_cube(2, jitter=0.1, patches="walls", seed=5)
    packed, starts = mg.pack([m] * members)
    rng = np.random.default_rng(8)
    fi, fb = m.n_internal_faces, m.n_boundary_faces
    flux = [0.1 * rng.standard_normal(fi + fb) for _ in range(members)]
    U = rng.standard_normal((packed.n_cells, 3))
    Ub = rng.standard_normal((packed.n_boundary_faces, 3))
    flux_p = np.concatenate([f[:fi] for f in flux] + [f[fi:] for f in flux])
    note("bicgstab packed", members, ncomp)
    x, it = momentum_solve(packed, starts, flux_p, U, Ub, ncomp)
    assert min(it) >= 2
    for k in (0, members // 2, members - 1):
        c = slice(starts[k], starts[k + 1])
        xk, _ = momentum_solve(m, None, flux[k], U[c], Ub[k * fb:(k + 1) * fb], ncomp)
        np.testing.assert_array_equal(x[c], xk)
