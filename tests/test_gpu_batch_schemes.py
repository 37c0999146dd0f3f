"""Members of a batch of more than 131,072 cells, where the momentum assembly has four slots of a row in flight
instead of two: with every convection and time scheme the bits of the member stepped alone."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import ctx, dev, host, note

pytestmark = pytest.mark.gpu


def steps(m, starts, U0, Ub, conv, time, n=2):
    M = B.Mesh(ctx(), m, seg_cell_start=starts)
    P = B.Piso(M, B.piso_params(0.02, 2e-3, conv=conv, time=time))
    P.set_boundary(dev(Ub), dev(np.zeros(m.n_boundary_faces)))
    P.set_state(dev(U0), dev(np.zeros(m.n_cells)), None)
    for _ in range(n):
        st, _, _ = P.step(1)
        assert st == 0
    out = [host(a) for a in P.get_state()[:2]]
    P.close()
    M.close()
    return out


@pytest.mark.parametrize("member,members", [("tets", 43), ("prisms", 69), ("hexes", 61)])
@pytest.mark.parametrize("conv", ["upwind", "linear", "sou", "quick"])
@pytest.mark.parametrize("time", ["backward_euler", "crank_nicolson"])
def test_members_keep_their_bits(member, members, conv, time):
    m = {"tets": lambda: mg.kuhn_cube(8, jitter=0.1, patches="walls", seed=5), "prisms": lambda: mg.cavity(31),
         "hexes": lambda: mg.hex_box(14, 13, 12)}[member]()
    packed, starts = mg.pack([m] * members)
    assert packed.n_cells >= 131072 > m.n_cells
    rng = np.random.default_rng(3)
    U0, Ub = 0.1 * rng.standard_normal((m.n_cells, 3)), np.zeros((m.n_boundary_faces, 3))
    if member == "prisms":
        U0[:, 2] = 0.0
    note("batch schemes", member, conv, time)
    one = steps(m, None, U0, Ub, conv, time)
    all_ = steps(packed, starts, np.tile(U0, (members, 1)), np.tile(Ub, (members, 1)), conv, time)
    for a, b in zip(one, all_):
        for k in (0, members - 1):
            np.testing.assert_array_equal(b[starts[k]:starts[k + 1]], a)
