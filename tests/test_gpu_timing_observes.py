"""Kernel timing (difvm_ctx_profile) observes: it changes neither what a step captured meanwhile replays nor,
with any preconditioner, the bits of a solve."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import dev, host, note

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
