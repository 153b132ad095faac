"""GPU tests of the neighbour search (nlist.hip) where its parts change: cells along an axis from one to several, periodic or not; atoms
far outside the box; pairs at the cutoff to the last bit; rows longer than what the counting pass keeps; more candidates than are put
in order at a time; more atoms or cells than one workgroup builds; and the row scan at its block sizes."""
import ctypes as C

import numpy as np
import pytest

from oracle import egnn_oracle as O
from tests.test_nlist_workspace import cells_alone

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def _check(B, pos, n_owned, box, pbc, r_cut):
    pos, box, pbc = np.asarray(pos, np.float32), np.asarray(box, np.float32), np.asarray(pbc, np.uint8)
    g = B.Egnn(1, 8, 8, r_cut, 1.0).egnn_nlist(B.to_device(pos), n_owned, box, pbc)
    src, dst, shift, row_ptr = O.neighbour_list(pos, n_owned, box, pbc, r_cut)
    print("  edges", len(src), "longest row", np.diff(row_ptr).max(), flush=True)
    assert g.n_edges == len(src)
    assert np.array_equal(g.row_ptr.cpu().numpy(), row_ptr)
    assert np.array_equal(g.src.cpu().numpy(), src) and np.array_equal(g.dst.cpu().numpy(), dst)
    assert np.array_equal(g.shift.cpu().numpy().reshape(-1, 3), shift)
    return row_ptr


@pytest.mark.parametrize("pbc", [(1, 1, 1), (1, 1, 0), (0, 1, 1), (0, 0, 0)])
@pytest.mark.parametrize("cells", [(2, 2, 2), (3, 2, 4), (4, 3, 2), (2, 5, 3), (6, 4, 5)])
def test_cells_along_an_axis(B, cells, pbc):
    """Two cells an axis are the fewest of a periodic one; atoms are moved out of the box by up to 40 of its lengths."""
    rng = np.random.default_rng([*cells, *pbc])
    box = np.array([2.03 * c for c in cells], np.float32)
    n = 700
    pos = rng.random((n, 3)) * box
    pos += rng.integers(-40, 41, (n, 3)) * box.astype(np.float64) * np.array(pbc)
    print("case", cells, pbc, flush=True)
    _check(B, pos, 611, box, pbc, 2.0)


@pytest.mark.parametrize("scale", [1.0, 1e-3, 3e4])
def test_pairs_at_the_cutoff(B, scale):
    """A lattice whose third shell lies at the cutoff up to the rounding of the coordinates: half of it in, half of it out."""
    rng = np.random.default_rng(4)
    g = np.stack(np.meshgrid(*[np.arange(8)] * 3, indexing="ij"), -1).reshape(-1, 3) * 1.1
    pos = (g + 5.0 + 3e-7 * rng.normal(size=g.shape)) * scale
    _check(B, pos, len(pos), [8 * 1.1 * scale] * 3, [1, 1, 1], np.float32(1.1 * np.sqrt(3.0) * scale))
    _check(B, pos, len(pos), [8 * 1.1 * scale] * 3, [0, 0, 0], np.float32(1.1 * np.sqrt(3.0) * scale))


@pytest.mark.parametrize("n,n_owned", [(257, 257), (258, 258), (400, 300), (1024, 64), (1026, 300), (2100, 50), (2100, 1000)])
def test_rows_and_candidate_lists(B, n, n_owned):
    """All atoms in reach of each other: rows of n - 1 (256 sources an atom are kept), n candidates (1,024 are put in order at a time)."""
    rng = np.random.default_rng(n)
    row_ptr = _check(B, rng.random((n, 3)), n_owned, [1, 1, 1], [0, 0, 0], 3.0)
    assert np.array_equal(np.diff(row_ptr), np.full(n_owned, n - 1))


@pytest.mark.parametrize("pbc", [(1, 1, 1), (1, 0, 1), (0, 0, 0)])
@pytest.mark.parametrize("n,n_owned", [(32768, 50), (32769, 50), (70000, 40), (250000, 25), (262144, 20), (262145, 9)])
def test_large_structures(B, n, n_owned, pbc):
    """Above 32,768 atoms the cells come from kernels of their own and an atom's wavefront has a workgroup to itself, above 245,760 with more
    than 64 KB of LDS; above 262,144 all atoms are swept."""
    rng = np.random.default_rng([n, *pbc])
    side = (n / 0.05) ** (1 / 3)
    print("case", n, pbc, flush=True)
    _check(B, rng.random((n, 3)) * side, n_owned, [side] * 3, pbc, 8.0)


@pytest.mark.parametrize("pbc", [(1, 1, 1), (0, 0, 0)])
@pytest.mark.parametrize("cells", [(32, 16, 16), (33, 16, 16), (64, 2, 64), (64, 64, 64), (17, 23, 41)])
def test_more_cells_than_are_counted_at_once(B, cells, pbc):
    """Few atoms in a large box: 8,192 cells are built by one workgroup, more are made coarser."""
    rng = np.random.default_rng([*cells, *pbc])
    box = np.array([2.001 * c for c in cells])
    n = 2500
    centres = rng.random((60, 3)) * box
    pos = (centres[rng.integers(0, 60, n)] + rng.normal(size=(n, 3))) % box
    pos[0], pos[1] = 0.0, np.nextafter(box.astype(np.float32), np.float32(0))       # (an open box is as large as its atoms)
    print("case", cells, pbc, flush=True)
    _check(B, pos, n, box, pbc, 2.0)


def test_rows_kept_of_many_atoms(B):
    """16,777,216 sources are kept in all, here 167 of an atom's 130 to 270; every 1,999th row against the oracle, all rows in order."""
    rng = np.random.default_rng(8)
    n, side = 100000, 126.0
    pos, box, pbc = (rng.random((n, 3)) * side).astype(np.float32), np.array([side] * 3, np.float32), np.array([1, 1, 1], np.uint8)
    m = B.Egnn(1, 8, 8, 10.0, 1.0)
    g = m.egnn_nlist(B.to_device(pos), n, box, pbc)
    src, dst, shift, row_ptr = (t.cpu().numpy() for t in (g.src, g.dst, g.shift, g.row_ptr))
    lengths = np.diff(row_ptr)
    print("edges", len(src), "rows of", lengths.min(), "to", lengths.max(), flush=True)
    assert lengths.min() <= 167 < lengths.max() and row_ptr[0] == 0 and row_ptr[-1] == len(src)
    assert np.array_equal(dst, np.repeat(np.arange(n), lengths))
    assert (np.diff(src.astype(np.int64) + dst.astype(np.int64) * n) > 0).all()
    for j in range(0, n, 1999):
        order = np.concatenate([[j], np.delete(np.arange(n), j)])            # (the oracle's owned atom comes first)
        s, _, sh, _ = O.neighbour_list(pos[order], 1, box, pbc, 10.0)
        at = np.argsort(order[s])
        rows = slice(row_ptr[j], row_ptr[j + 1])
        assert np.array_equal(src[rows], order[s][at]) and np.array_equal(shift[rows], sh[at]), j


@pytest.mark.parametrize("n,n_owned", [(700, 611), (33000, 70)])
def test_shorter_workspaces(B, n, n_owned):
    """Cells alone; positions in their order, but nothing kept; one source kept per atom; a workspace that is shorter in the filling pass."""
    import torch
    rng = np.random.default_rng(n)
    pos = (rng.random((n, 3)) * 20.0).astype(np.float32)
    box, pbc = np.array([20.0] * 3, np.float32), np.array([1, 0, 1], np.uint8)
    r_cut = 3.0 * (700 / n) ** (1 / 3)
    src, dst, _, row_ptr = O.neighbour_list(pos, n_owned, box, pbc, r_cut)
    m = B.Egnn(1, 8, 8, r_cut, 1.0)
    least, most = cells_alone(n), m.egnn_nlist_workspace_bytes(n)
    positions = least + (16 * n + 255) // 256 * 256 - (4 * n + 255) // 256 * 256
    p, bx, pb = B.to_device(pos), (C.c_float * 3)(*box), (C.c_uint8 * 3)(*[int(v) for v in pbc])
    ws = torch.full((most,), -1, dtype=torch.int8, device="cuda").view(torch.uint8)
    for first, second in ((least, least), (least - 1, least - 1), (positions, positions), (positions - 1, positions - 1),
                          (positions + 4 * n_owned, positions + 4 * n_owned), (most, most), (most, most - 256), (most, positions),
                          (most, least), (least, most)):
        print("case", n, first, second, flush=True)
        rp, ne = torch.empty(n_owned + 1, dtype=torch.int32, device="cuda"), C.c_int64()
        m._check(m.lib.egnn_nlist_count(m.ctx, B._ptr(p), n_owned, n, bx, pb, B._ptr(rp), C.byref(ne), B._ptr(ws), C.c_size_t(first), None))
        assert ne.value == len(src) and np.array_equal(rp.cpu().numpy(), row_ptr)
        got = [torch.full((len(src),), -1, dtype=torch.int32, device="cuda") for _ in range(2)]
        m._check(m.lib.egnn_nlist_fill(m.ctx, B._ptr(p), n_owned, n, bx, pb, B._ptr(rp), ne, B._ptr(got[0]), B._ptr(got[1]), None,
                                       B._ptr(ws), C.c_size_t(second), None))
        assert np.array_equal(got[0].cpu().numpy(), src) and np.array_equal(got[1].cpu().numpy(), dst)


@pytest.mark.parametrize("n_total", [1, 7, 8191, 8193, 32767, 32768, 32769, 40960, 65537, 100000])
def test_row_scan(B, n_total):
    """The scan takes 32,768 rows at a time (through the index of the edges by source)."""
    import torch
    rng = np.random.default_rng(n_total)
    n_edges = 30000
    src = rng.integers(0, n_total, n_edges).astype(np.int32)
    dst = np.sort(rng.integers(0, 40, n_edges)).astype(np.int32) % max(1, min(40, n_total))
    dst = np.sort(dst).astype(np.int32)
    n_owned = int(dst.max()) + 1
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n_owned))]).astype(np.int32)
    m = B.Egnn(1, 8, 4, 8.0, 1.0)
    g = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), None, n_owned, n_total)
    ws = torch.empty(m.egnn_backward_workspace_bytes(n_edges, n_owned, n_total), dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(g, ws)
    assert np.array_equal(col_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n_total))]))
    assert np.array_equal(perm.cpu().numpy(), np.argsort(src, kind="stable"))
