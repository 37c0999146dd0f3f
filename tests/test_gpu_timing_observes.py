"""Kernel timing (difvm_ctx_profile) observes: it changes neither what a step captured meanwhile replays nor,
with any preconditioner, the bits of a solve."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import dev, empty, host, note

pytestmark = pytest.mark.gpu


def cavity_run(n, timed, graph=False):
    """five AMG steps of the lid-driven cavity; timed: kernel timing is on during the first (in graph mode the
    one that captures), or with "all" throughout"""
    m = mg.cavity(n)
    c = B.Context(0)
    M = B.Mesh(c, m)
    P = B.Piso(M, B.piso_params(0.01, 1e-3, precond="amg"))
    Ub = np.zeros((m.n_boundary_faces, 3))
    lid = m.patch("lid")
    Ub[lid.start - m.n_internal_faces:lid.start - m.n_internal_faces + lid.size, 0] = 1.0
    P.set_boundary(dev(Ub), dev(np.zeros(m.n_boundary_faces)))
    U0 = np.zeros((m.n_cells, 3))
    start = dev(U0), dev(np.zeros(m.n_cells)), dev(O.initial_flux(m, U0, Ub))
    P.set_state(*start)
    if graph:
        P.set_graph(True, 8)
    out = []
    for k in range(5):
        B.difvm_ctx_profile(c.h, 3 if timed == "all" or (timed and k == 0) else 0)
        if graph:  # the same step again and again: what the timed one left does not reach the replays
            P.set_state(*start)
        st, it, res = P.step(1)
        assert st == 0
        out.append((it, res) + tuple(host(a) for a in P.get_state()[:3]))
    B.difvm_ctx_profile(c.h, 0)
    B.difvm_ctx_profile_read(c.h)
    info = P.graph_info()
    P.close()
    M.close()
    return out, info


# one tile, three tiles (the AMG solve of either in one block) and five (its update joined with the cycle)
@pytest.mark.parametrize("n", [16, 33, 50])
def test_step_captured_while_timed_replays_the_untimed_bits(n):
    """captured during a timed step, replayed after timing is off, against a graph that was never timed: from the
    first replay on the same bits"""
    note("captured while timed", n)
    a, ia = cavity_run(n, True, graph=True)
    b, ib = cavity_run(n, False, graph=True)
    assert ia == ib and ia[0] >= 1
    for k, (x, y) in enumerate(zip(a[1:], b[1:])):
        for u, v in zip(x, y):
            np.testing.assert_array_equal(u, v, err_msg=f"step {k + 1}")


def test_eager_steps_keep_their_bits_while_timed():
    for n in (16, 50):
        note("timed steps", n)
        for x, y in zip(cavity_run(n, "all")[0], cavity_run(n, False)[0]):
            for u, v in zip(x, y):
                np.testing.assert_array_equal(u, v)


LAP = lambda n: mg.kuhn_cube(n, jitter=0.1, patches="walls", seed=5)
# the whole solve in one block: one tile of tets, four of prisms; the update joined with the cycle: five tiles of tets,
# members that stop at different iterations, six slots a row, three levels; above the limit of 384 tiles
SOLVES = {"tets 750": lambda: LAP(5), "prisms 4050": lambda: mg.cavity(45), "tets 4374": lambda: LAP(9),
          "members": lambda: mg.pack([LAP(8), LAP(5), LAP(9)]), "hexes 2184": lambda: mg.hex_box(14, 13, 12),
          "tets 52272": lambda: mg.kuhn_cube(1, jitter=0.1, patches="walls", seed=5, nxyz=(22, 22, 18)),
          "tets 407208": lambda: mg.kuhn_cube(1, jitter=0.1, patches="walls", seed=5, nxyz=(38, 38, 47))}


def amg_solve(cx, m, starts, bh, x0, maxit, stride=0):
    M = B.Mesh(cx, m, seg_cell_start=starts)
    A = B.ldu(empty(m.n_cells), empty(m.n_internal_faces))
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(m.n_boundary_faces)), A, empty(m.n_cells))
    amg = B.difvm_amg_create(M.h, A)
    x = M.to_internal(dev(x0), B.KIND_CELL)
    B.difvm_ctx_profile(cx.h, stride)
    out = B.difvm_solve_pcg_amg(amg, A, M.to_internal(dev(bh), B.KIND_CELL), x, 1e-10, maxit)
    times = {k: v for k, v in B.difvm_ctx_profile_read(cx.h).items() if v[0]}
    B.difvm_ctx_profile(cx.h, 0)
    x = host(M.to_user(x, B.KIND_CELL))
    B.difvm_amg_destroy(amg)
    M.close()
    return out, x, times


@pytest.mark.parametrize("name", SOLVES)
@pytest.mark.parametrize("maxit", [3, 200])
def test_amg_solve_keeps_its_bits_while_timed(name, maxit):
    m = SOLVES[name]()
    m, starts = m if name == "members" else (m, None)
    rng = np.random.default_rng(3)
    bh, x0 = rng.standard_normal(m.n_cells), 0.1 * rng.standard_normal(m.n_cells)
    cx = B.Context(0)
    note("timed solve", name, maxit)
    s0, xa, _ = amg_solve(cx, m, starts, bh, x0, maxit)
    for stride in (1, 7):
        s1, xb, times = amg_solve(cx, m, starts, bh, x0, maxit, stride)
        assert s1 == s0
        np.testing.assert_array_equal(xa, xb)
        if name in ("tets 750", "prisms 4050"):
            assert list(times) == ["pcg_amg_block"] and times["pcg_amg_block"][0] == 1
        else:
            assert {"pcg_spmv_dot", "pcg_update_dot", "pcg_amg_vcycle"} <= set(times)


def cg_of_cycles(M, A, amg, b, x, tol, maxit):
    """CG made of the library's product and of single V-cycles (difvm_amg_apply: the cycle as kernels)"""
    q, z, p, rho_old = b.clone(), b.clone(), None, None
    B.difvm_ldu_spmv(M.h, 1, 0, A, x, q)
    r, bn = b - q, float(b.norm())
    for k in range(1, maxit + 1):
        B.difvm_amg_apply(amg, r, z)
        rho = float(r @ z)
        p = z.clone() if p is None else z + (rho / rho_old) * p
        B.difvm_ldu_spmv(M.h, 1, 0, A, p, q)
        alpha = rho / float(p @ q)
        x, r, rho_old = x + alpha * p, r - alpha * q, rho
        if float(r.norm()) <= tol * bn:
            return 0, k, float(r.norm()) / bn, x
    return B.WARN_NOT_CONVERGED, maxit, float(r.norm()) / bn, x


@pytest.mark.parametrize("name", ["tets 750", "tets 3888", "prisms 968", "prisms 2048", "prisms 2178", "prisms 4050"])
@pytest.mark.parametrize("maxit", [1, 4, 200])
def test_amg_block_against_kernels(name, maxit):
    """The solve in one block against CG with the cycle as kernels: equal counts and status, iterates equal up to
    the rounding of sums of at most 4,050 terms in another order, carried through some 20 iterations."""
    m = {"tets 750": lambda: LAP(5), "prisms 968": lambda: mg.cavity(22), "prisms 2048": lambda: mg.cavity(32),
         "prisms 2178": lambda: mg.cavity(33), "prisms 4050": lambda: mg.cavity(45),
         "tets 3888": lambda: mg.kuhn_cube(1, jitter=0.1, patches="walls", nxyz=(8, 9, 9), seed=5)}[name]()
    rng = np.random.default_rng(3)
    cx = B.Context(0)
    M = B.Mesh(cx, m)
    A = B.ldu(empty(m.n_cells), empty(m.n_internal_faces))
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(m.n_boundary_faces)), A, empty(m.n_cells))
    amg = B.difvm_amg_create(M.h, A)
    b, x = dev(rng.standard_normal(m.n_cells)), dev(0.1 * rng.standard_normal(m.n_cells))
    note("block against kernels", name, maxit)
    sb, ib, rb, xb = cg_of_cycles(M, A, amg, b, x.clone(), 1e-10, maxit)
    B.difvm_ctx_profile(cx.h, 1)
    sa, ia, ra = B.difvm_solve_pcg_amg(amg, A, b, x, 1e-10, maxit)
    times = B.difvm_ctx_profile_read(cx.h)
    B.difvm_ctx_profile(cx.h, 0)
    assert times["pcg_amg_block"][0] == 1
    assert (sa, ia) == (sb, ib)
    assert abs(ra - rb) <= 1e-6 * rb
    assert float((x - xb).abs().max()) <= 1e-11 * float(xb.abs().max())
    B.difvm_amg_destroy(amg)
