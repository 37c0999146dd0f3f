"""The solvers' dispatch by size must not show in the results: a member of a packed mesh keeps the bits of
its standalone solve on either side of each limit.

The Krylov kernels take a quarter of a 1,024-cell tile per block up to 384 tiles and a tile above (where
BiCGStab also sums its partials in a kernel of its own); many tiny members reach the limit with few cells
(a tile each).  Jacobi-CG of segments of at most four tiles runs in one block per segment; while the
kernels are being timed (difvm_ctx_profile) the same solve takes the two kernels per iteration, whose
results must be the same bits.  The momentum assembly has two slots of a row in flight below 131,072 cells and
four from there on."""
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


@pytest.mark.parametrize("member,members", [("tets", 42), ("tets", 43), ("hexes", 61)])
def test_momentum_rows_keep_their_bits(member, members):
    """rows of four and of six slots, on either side of the limit"""
    m = mg.kuhn_cube(8, jitter=0.1, patches="walls", seed=5) if member == "tets" else mg.hex_box(14, 13, 12)
    packed, starts = mg.pack([m] * members)
    assert (packed.n_cells >= 131072) == (members >= 43)
    rng = np.random.default_rng(8)
    fi, fb = m.n_internal_faces, m.n_boundary_faces
    flux, U, Ub = 0.1 * rng.standard_normal(fi + fb), rng.standard_normal((m.n_cells, 3)), rng.standard_normal((fb, 3))
    out = []
    for mesh, seg, f, u, ub in ((m, None, flux, U, Ub), (packed, starts, np.concatenate(
            [np.tile(flux[:fi], members), np.tile(flux[fi:], members)]), np.tile(U, (members, 1)), np.tile(Ub, (members, 1)))):
        M = B.Mesh(ctx(), mesh, seg_cell_start=seg)
        D, b = empty(mesh.n_cells), empty((mesh.n_cells, 3))
        A = B.ldu(D, empty(mesh.n_internal_faces), empty(mesh.n_internal_faces))
        note("momentum", member, mesh.n_cells)
        B.difvm_ldu_assemble_momentum(M.h, 0.01, 1e-2, M.to_internal(dev(f), B.KIND_FACE_FLUX),
                                      M.to_internal(dev(u), B.KIND_CELL), M.to_internal(dev(ub), B.KIND_BFACE), A, b)
        out.append((host(M.to_user(D, B.KIND_CELL)), host(M.to_user(b, B.KIND_CELL))))
    for one, all_ in zip(*out):
        for k in (0, members - 1):
            np.testing.assert_array_equal(all_[starts[k]:starts[k + 1]], one)


@pytest.mark.parametrize("shape", ["tets", "prisms"])
@pytest.mark.parametrize("ncomp", [1, 3])
@pytest.mark.parametrize("small", [True, False])
def test_bicgstab_segment_members_keep_their_bits(shape, ncomp, small):
    """members of one to four tiles, all in the one-block form or (beside a larger one) in the general form,
    against their standalone solves (one block): the same bits and counts"""
    one = (lambda n: mg.kuhn_cube(n, jitter=0.1, patches="walls", seed=n)) if shape == "tets" else mg.cavity
    ms = [one(n) for n in ((2, 5, 7, 8) if shape == "tets" else (8, 22, 32, 45))] + ([] if small else [one(
        10 if shape == "tets" else 50)])
    packed, starts = mg.pack(ms)
    rng = np.random.default_rng(8)
    flux = [0.1 * rng.standard_normal(m.n_internal_faces + m.n_boundary_faces) for m in ms]
    U = rng.standard_normal((packed.n_cells, 3))
    Ub = rng.standard_normal((packed.n_boundary_faces, 3))
    flux_p = np.concatenate([f[:m.n_internal_faces] for f, m in zip(flux, ms)] +
                            [f[m.n_internal_faces:] for f, m in zip(flux, ms)])
    note("bicgstab segments", shape, ncomp, small)
    x, it = momentum_solve(packed, starts, flux_p, U, Ub, ncomp)
    its, fb = [], 0
    for k, m in enumerate(ms):
        c = slice(starts[k], starts[k + 1])
        xk, itk = momentum_solve(m, None, flux[k], U[c], Ub[fb:fb + m.n_boundary_faces], ncomp)
        fb += m.n_boundary_faces
        its.append(itk)
        np.testing.assert_array_equal(x[c], xk)
    assert list(it)[:ncomp] == list(np.max(its, axis=0))[:ncomp]


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


def laplace_system(mesh, seg=None, seed=2):
    M = B.Mesh(ctx(), mesh, seg_cell_start=seg)
    A = B.ldu(empty(mesh.n_cells), empty(max(1, mesh.n_internal_faces)))
    rhs = empty(mesh.n_cells)
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(mesh.n_boundary_faces)), A, rhs)
    return M, A


def pcg_both_forms(M, A, b, tol, maxit):
    out = []
    for stride in (0, 1 << 20):
        B.difvm_ctx_profile(ctx().h, stride)
        x = b.clone().zero_()
        try:
            out.append((B.difvm_solve_pcg(M.h, A, b, x, tol, maxit), host(x)))
        finally:
            B.difvm_ctx_profile(ctx().h, 0)
            B.difvm_ctx_profile_read(ctx().h)
    return out


# cells at the edges of the block shapes: one and two tiles in 256 threads, three and four in 512, five in
# the general form; prisms (three slots), tets (four), hexes (six, rows from memory)
SHAPES = {"prism_2": lambda: mg.cavity(1), "prism_1922": lambda: mg.cavity(31), "prism_2048": lambda: mg.cavity(32),
          "prism_2178": lambda: mg.cavity(33), "prism_4050": lambda: mg.cavity(45), "prism_4232": lambda: mg.cavity(46),
          "tet_6": lambda: mg.kuhn_cube(1), "tet_1032": lambda: mg.kuhn_cube(1, nxyz=(2, 2, 43)),
          "tet_2058": lambda: mg.kuhn_cube(7), "tet_3072": lambda: mg.kuhn_cube(8),
          "tet_4104": lambda: mg.kuhn_cube(1, nxyz=(6, 6, 19)), "hex_1": lambda: mg.hex_box(1, 1, 1),
          "hex_1728": lambda: mg.hex_box(12, 12, 12), "hex_4096": lambda: mg.hex_box(16, 16, 16)}


@pytest.mark.parametrize("name", SHAPES)
def test_pcg_segment_form_same_bits(name):
    m = SHAPES[name]()
    M, A = laplace_system(m)
    b = dev(np.random.default_rng(3).standard_normal(m.n_cells))
    note("pcg forms", name, m.n_cells)
    for tol, maxit in ((1e-10, 4000), (1e-10, 3), (1e-10, 0)):
        (s1, x1), (s2, x2) = pcg_both_forms(M, A, b, tol, maxit)
        assert s1 == s2
        np.testing.assert_array_equal(x1, x2)


@pytest.mark.parametrize("maxit", [2048, 2049, 4100])
def test_pcg_segment_form_over_several_launches(maxit):
    """A zero tolerance: the solve goes on through several launches of at most 2,048 iterations, to its cap or
    until the recursive residual underflows to zero (3,310 iterations here)."""
    m = mg.cavity(45)
    M, A = laplace_system(m)
    b = dev(np.random.default_rng(4).standard_normal(m.n_cells))
    note("pcg cap", maxit)
    (s1, x1), (s2, x2) = pcg_both_forms(M, A, b, 0.0, maxit)
    assert s1 == s2 and s1[1] >= 2048
    assert s1[0] == (B.WARN_NOT_CONVERGED if s1[1] == maxit else 0)
    np.testing.assert_array_equal(x1, x2)


@pytest.mark.parametrize("sizes", [(1, 7, 2), (8, 3), (12, 2)])
def test_pcg_members_keep_their_bits(sizes):
    """Packed tet cubes of 6 to 10,368 cells: all in the segment form, or beside a member that is not."""
    ms = [mg.kuhn_cube(n, seed=n) for n in sizes]
    packed, starts = mg.pack(ms)
    M, A = laplace_system(packed, starts)
    b = np.random.default_rng(5).standard_normal(packed.n_cells)
    x = empty(packed.n_cells).zero_()
    note("pcg packed", sizes)
    st = B.difvm_solve_pcg(M.h, A, M.to_internal(dev(b), B.KIND_CELL), x, 1e-11, 4000)
    got, its = host(M.to_user(x, B.KIND_CELL)), []
    for k, m in enumerate(ms):
        Mk, Ak = laplace_system(m)
        xk = empty(m.n_cells).zero_()
        c = slice(starts[k], starts[k + 1])
        its.append(B.difvm_solve_pcg(Mk.h, Ak, Mk.to_internal(dev(b[c]), B.KIND_CELL), xk, 1e-11, 4000)[1])
        np.testing.assert_array_equal(got[c], host(Mk.to_user(xk, B.KIND_CELL)))
    assert st[0] == 0 and st[1] == max(its)
