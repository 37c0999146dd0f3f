"""The deferred correction's arithmetic, slot by slot: every operation rounded once, sums and products fused where
the library fuses them (worked out here in rational numbers), whichever slots of a row are in flight together."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import ctx, dev, empty, host, note

pytestmark = pytest.mark.gpu

MESHES = {"tets": lambda: mg.kuhn_cube(3, jitter=0.1, patches="sides", seed=4), "hexes": lambda: mg.hex_box(
    4, 3, 5, A=[[1.0, 0.3, 0.0], [0.0, 1.1, 0.2], [0.1, 0.0, 0.9]]), "prisms": lambda: mg.cavity(6)}


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def dot(g, x, y, z):
    return fma(g[2], z, fma(g[0], x, g[1] * y))


@pytest.mark.parametrize("name", MESHES)
@pytest.mark.parametrize("conv", ["linear", "sou", "quick"])
@pytest.mark.parametrize("ncomp", [1, 3])
def test_each_slot_is_fused_the_same(name, conv, ncomp):
    m = MESHES[name]()
    M = B.Mesh(ctx(), m)
    r = B.difvm_mesh_renumber_host(m, geometry=True)
    nc, nfi = m.n_cells, m.n_internal_faces
    rng = np.random.default_rng(3)
    phi, g, F = (rng.standard_normal(s) for s in ((nc, ncomp), (nc, ncomp, 3), m.n_faces))  # internal order
    C, Cf = m.C[r["cell_perm"]], m.Cf[:nfi][r["face_perm"]]
    out = empty((nc, ncomp) if ncomp > 1 else nc)
    note("deferred correction", name, conv, ncomp)
    B.difvm_op_deferred_correction(M.h, conv, ncomp, dev(F), dev(phi if ncomp > 1 else phi[:, 0]),
                                   dev(g.reshape(nc, 3 * ncomp)), out)
    got, want = host(out).reshape(nc, ncomp), np.zeros((nc, ncomp))
    own, nbr, w = r["owner"], r["neighbour"], r["w"]
    for i in range(nc):
        own_faces = range(r["own_start"][i], r["own_start"][i + 1])
        nbr_faces = r["losort"][r["losort_start"][i]:r["losort_start"][i + 1]]
        for f, nb in [(f, False) for f in own_faces] + [(f, True) for f in nbr_faces]:
            j = own[f] if nb else nbr[f]
            up = i if (F[f] >= 0) != nb else j
            down = j if up == i else i
            ws = 1.0 - w[f] if nb else w[f]
            rC, rD = Cf[f] - C[up], Cf[f] - C[down]
            for c in range(ncomp):
                gc = [float(v) for v in g[up, c]]
                if conv == "linear":
                    d = fma(ws, phi[i, c], (1.0 - ws) * phi[j, c]) - phi[up, c]
                elif conv == "sou":
                    d = dot(gc, *rC)
                else:
                    d = fma(0.25, dot(gc, *(rC - rD)), 0.25 * (phi[down, c] - phi[up, c]))
                want[i, c] = fma(F[f] if nb else -F[f], d, want[i, c])
    np.testing.assert_array_equal(got, want)
