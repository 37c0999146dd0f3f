"""Reordering of fields between user and internal order (difvm_permute): every row width, type, array
kind and direction, against the host renumbering's permutations in numpy.  Values move unchanged (a flux
of a re-oriented face changes sign), so the comparison is exact, signed zeros, infinities and NaN included.
The meshes leave a partly filled last block of rows (and one has fewer rows than a block)."""
import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg
from gpu_util import ctx, dev, empty, host, note, torch

pytestmark = pytest.mark.gpu

MESHES = {"cavity4": lambda: mg.cavity(4), "kuhn7": lambda: mg.kuhn_cube(7, jitter=0.1, patches="sides", seed=11)}
KINDS = {"cell": B.KIND_CELL, "face": B.KIND_FACE, "flux": B.KIND_FACE_FLUX, "bface": B.KIND_BFACE}


@pytest.mark.parametrize("name", MESHES)
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_permute_exact(name, kind, dtype):
    m = MESHES[name]()
    M = B.Mesh(ctx(), m)
    r = B.difvm_mesh_renumber_host(m)
    nfi = m.n_internal_faces
    bp = r["bface_perm"]
    perm = {"cell": r["cell_perm"], "bface": bp}.get(kind, np.concatenate([r["face_perm"], nfi + bp]))
    sign = np.ones(perm.size, dtype)
    if kind == "flux":
        sign[:nfi][r["face_flip"] != 0] = -1
    rng = np.random.default_rng(7)
    for nc in range(1, 10):
        note("permute", name, kind, dtype, nc)
        a = rng.standard_normal((perm.size, nc)).astype(dtype)
        a.flat[:4] = [-0.0, np.inf, -np.inf, np.nan]
        dt = getattr(torch(), dtype)
        src, out = dev(a, dt), empty(a.shape, dt)
        B.difvm_permute(M.h, nc, KINDS[kind], B.TO_INTERNAL, src, out)
        want = sign[:, None] * a[perm]
        got = host(out)
        assert np.array_equal(got, want, equal_nan=True) and np.array_equal(np.signbit(got), np.signbit(want))
        back = empty(a.shape, dt)
        B.difvm_permute(M.h, nc, KINDS[kind], B.FROM_INTERNAL, out, back)
        assert np.array_equal(host(back), a, equal_nan=True)
