"""The workspace of the neighbour search: down to what the cells alone take the search goes through them.  Asked of the library without a
GPU: the filling pass refuses cells that were never built (EGNN_EINVAL, before any launch); a sweep would not ask for them."""
import ctypes as C
import os

import pytest

# (the pointers are made up: a library that sweeps would launch kernels on them where there is a GPU)
pytestmark = pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="asked where nothing can be launched")


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.load_library()
    return binding


def cells_alone(n):
    """Bounding box and grid, cell of every atom, starts and cursors of 64^3 cells, atoms in the order of the cells."""
    up = lambda b: (b + 255) // 256 * 256
    return 256 + 2 * up(4 * n) + up(4 * (64 ** 3 + 1)) + up(4 * 64 ** 3)


def refuses_missing_cells(m, n, nbytes):
    box, pbc, at = (C.c_float * 3)(100, 100, 100), (C.c_uint8 * 3)(1, 1, 1), C.c_void_p(4096)     # (no pointer is followed)
    rc = m.lib.egnn_nlist_fill(m.ctx, at, n, n, box, pbc, at, C.c_int64(5), at, at, None, at, C.c_size_t(nbytes), None)
    return rc == -1


@pytest.mark.parametrize("n", [1, 64, 3000, 32769, 100001, 262144])
def test_workspace_of_the_cells_alone(B, n):
    m = B.Egnn(1, 8, 8, 4.0, 1.0)
    assert m.egnn_nlist_workspace_bytes(n) > cells_alone(n)
    for nbytes in (cells_alone(n), cells_alone(n) + 256, m.egnn_nlist_workspace_bytes(n) - 1, m.egnn_nlist_workspace_bytes(n)):
        assert refuses_missing_cells(m, n, nbytes)
