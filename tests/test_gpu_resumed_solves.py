"""Solves in one block that go on through several launches: a launch makes at most 2,048 iterations (AMG-CG 256) and
leaves what the next one needs."""
import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import ctx, dev, empty, host, note

pytestmark = pytest.mark.gpu


# two, four, six and eight cells per thread; rows of three and of four slots
MESHES = {"prisms 968": lambda: mg.cavity(22), "prisms 2048": lambda: mg.cavity(32), "prisms 2178": lambda: mg.cavity(33),
          "prisms 4050": lambda: mg.cavity(45),
          "tets 3888": lambda: mg.kuhn_cube(1, jitter=0.1, patches="walls", nxyz=(8, 9, 9), seed=5)}


@pytest.mark.parametrize("name", MESHES)
def test_amg_block_directions_stay_conjugate_over_launches(name):
    """A hierarchy made from 1e-10 times the matrix gives a preconditioner of condition 1e10: some 300 iterations.
    CG's neighbouring directions are conjugate and its residual orthogonal to its last step; the steps are the
    differences of the iterates at caps 254 to 259, the residuals the true ones.  From rounding (2e-16 x 1e10
    through the preconditioner; 1e-16 of the iterate against steps of 1e-8) both cosines are below 1e-4; with a
    direction, a step length or a residual lost between two launches they are some tenths."""
    m = MESHES[name]()
    M = B.Mesh(ctx(), m)
    D, U = empty(m.n_cells), empty(m.n_internal_faces)
    A = B.ldu(D, U)
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(m.n_boundary_faces)), A, empty(m.n_cells))
    D0, U0 = 1e-10 * D, 1e-10 * U
    amg = B.difvm_amg_create(M.h, B.ldu(D0, U0))
    b = dev(np.random.default_rng(3).standard_normal(m.n_cells))

    def product(v):
        y = empty(m.n_cells)
        B.difvm_ldu_spmv(M.h, 1, 0, A, v, y)
        return y

    x = {}
    for cap in range(254, 260):
        x[cap] = empty(m.n_cells).zero_()
        st, it, res = B.difvm_solve_pcg_amg(amg, A, b, x[cap], 0.0, cap)
        assert (st, it) == (B.WARN_NOT_CONVERGED, cap)
    note("conjugate", name, "residual", res)
    steps = {cap: x[cap] - x[cap - 1] for cap in range(255, 260)}
    for cap in range(256, 260):
        old, new = steps[cap - 1], steps[cap]
        k_old, k_new = product(old), product(new)
        conj = float(new @ k_old) / (float(new @ k_new) * float(old @ k_old)) ** 0.5
        r = b - product(x[cap])
        orth = float(r @ new) / (float(r.norm()) * float(new.norm()))
        note("cosines at", cap, conj, orth)
        assert abs(conj) <= 1e-4 and abs(orth) <= 1e-4
    B.difvm_amg_destroy(amg)


@pytest.mark.parametrize("layers", [170, 340, 510, 680])
@pytest.mark.parametrize("ncomp", [1, 3])
def test_bicgstab_block_over_launches(layers, ncomp):
    """Flat tets (one to four tiles), a zero tolerance: no component stops before its cap.  The solve in one block per
    component against the kernels of an iteration, which the mesh takes beside a member of six tiles (long stopped, at
    a residual of 1e-161): the same bits of iterate and residual at the seam and after it."""
    m = mg.kuhn_cube(1, jitter=0.1, patches="walls", nxyz=(1, 1, layers), seed=5)
    both, starts = mg.pack([m, mg.kuhn_cube(10, patches="walls")])
    rng = np.random.default_rng(8)
    rhs = rng.standard_normal((both.n_cells, 3))[:, :ncomp]
    runs = {}
    for key, mesh, seg, b in (("block", m, None, rhs[:m.n_cells]), ("kernels", both, starts, rhs)):
        M = B.Mesh(ctx(), mesh, seg_cell_start=seg)
        A = B.ldu(empty(mesh.n_cells), empty(mesh.n_internal_faces), empty(mesh.n_internal_faces))
        zero = dev(np.zeros((mesh.n_cells, 3)))
        B.difvm_ldu_assemble_momentum(M.h, 1.0, 1e3, dev(np.zeros(mesh.n_faces)), zero,
                                      dev(np.zeros((mesh.n_boundary_faces, 3))), A, empty((mesh.n_cells, 3)))
        b = M.to_internal(dev(b if ncomp == 3 else b[:, 0]), B.KIND_CELL)
        for cap in (2047, 2048, 2049, 2060):
            x = b.clone().zero_()
            note("bicgstab", key, layers, ncomp, cap)
            st, it, res = B.difvm_solve_bicgstab(M.h, A, ncomp, b, x, 0.0, cap)
            runs[key, cap] = host(M.to_user(x, B.KIND_CELL))[:m.n_cells], np.array(res[:ncomp])
            assert list(it[:ncomp]) == [cap] * ncomp
            if key == "block":
                assert st == B.WARN_NOT_CONVERGED
    for cap in (2047, 2048, 2049, 2060):
        for one, other in zip(runs["block", cap], runs["kernels", cap]):
            assert np.isfinite(one).all()
            np.testing.assert_array_equal(one, other)
    assert (runs["block", 2049][1] != runs["block", 2048][1]).all()
