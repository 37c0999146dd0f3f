"""The AMG setup when device memory ends in the middle of it: DIFVM_ERR_OOM, and the next setup on the same mesh is
what the first was."""
import numpy as np
import pytest

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

from gpu_util import dev, empty, host, note

pytestmark = pytest.mark.gpu

# two levels with the layout for a solve in one block; three levels with the middle one in two passes; in three
# passes (a dense product above the limit)
MESHES = {"block": lambda: mg.cavity(33), "two passes": lambda: mg.kuhn_cube(1, nxyz=(14, 14, 14)),
          "three passes": lambda: mg.kuhn_cube(1, nxyz=(38, 38, 47))}


def failing_setups(name, after_failure):
    m = MESHES[name]()
    c = B.Context(0, torch_allocator=False)
    T = B.TorchAllocator(0)
    budget = {"n": 1 << 30}
    inner = T.alloc_fn

    def alloc(nbytes, stream, user):
        if budget["n"] <= 0:
            return None
        budget["n"] -= 1
        return inner(nbytes, stream, user)

    fn = B.ALLOC_FN(alloc)
    B.difvm_ctx_set_allocator(c.h, fn, T.free_fn)
    M = B.Mesh(c, m)
    A = B.ldu(empty(m.n_cells), empty(m.n_internal_faces))
    B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, dev(np.zeros(m.n_boundary_faces)), A, empty(m.n_cells))
    r, z = dev(np.random.default_rng(1).standard_normal(m.n_cells)), empty(m.n_cells)

    def cycle():
        amg = B.difvm_amg_create(M.h, A)
        B.difvm_amg_apply(amg, r, z)
        out = host(z)
        B.difvm_amg_destroy(amg)
        return out

    want = cycle()
    before = T.n_alloc
    np.testing.assert_array_equal(cycle(), want)
    total, held = T.n_alloc - before, len(T.live)
    note("setup", name, m.n_cells, "allocations", total)
    for n in sorted(set(range(0, total, 1 if m.n_cells < 20000 else 5)) | {total - 1, total - 2, total - 3}):
        budget["n"] = n
        with pytest.raises(B.DifvmError) as e:
            B.difvm_amg_create(M.h, A)
        assert e.value.status == B.ERR_OOM
        after_failure(n, len(T.live) - held)
    budget["n"] = 1 << 30
    np.testing.assert_array_equal(cycle(), want)
    M.close()


@pytest.mark.parametrize("name", MESHES)
def test_setup_fails_and_works_again(name):
    failing_setups(name, lambda n, left: None)


@pytest.mark.parametrize("name", MESHES)
def test_failed_setup_gives_everything_back(name):
    left = {}
    failing_setups(name, left.__setitem__)
    assert not any(left.values()), left
