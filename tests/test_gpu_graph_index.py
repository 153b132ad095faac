"""Per-graph indices (edges by length, edges by source) at the sizes where their kernels change behaviour, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


# edges: fewer than one chunk of 2,048, around two chunks, ragged last chunk, more than 1,024 chunks' worth; nodes: one, more
# than one round of the scan (8,192); outgoing edges of a node: none, below and above the 1,024 that are sorted in LDS
@pytest.mark.parametrize("n_edges,n_owned,n_total", [(1, 1, 2), (63, 1, 64), (2047, 30, 40), (2048, 30, 40), (4095, 3, 3), (4097, 50, 50),
                                                     (70001, 9000, 20000), (2100000, 8193, 16385), (9001, 5, 9),
                                                     # the parts that a chunk's four waves take: one edge, one short of four parts, ragged
                                                     (65, 3, 4), (255, 9, 9), (257, 9, 9), (2113, 20, 30), (8450, 300, 300)])
def test_length_bins_and_transpose(B, n_edges, n_owned, n_total):
    import torch
    rng = np.random.default_rng(n_edges)
    src = rng.integers(0, n_total, n_edges).astype(np.int32)
    src[n_total // 2 == src] = 0                                    # one node without outgoing edges, one with more
    if n_edges == 4097:
        src[:1500] = 7                                              # above the limit of the sort in LDS
    dst = np.sort(rng.integers(0, n_owned, n_edges)).astype(np.int32)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n_owned))]).astype(np.int32)
    pos = (rng.random((n_total, 3)) * 4.0).astype(np.float32)
    m = B.Egnn(1, 8, 4, 8.0, 1.0)
    g = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), None, n_owned, n_total)
    p, box = B.to_device(pos), np.ones(3, np.float32)
    print("case", n_edges, n_owned, n_total, flush=True)
    m.egnn_length_bins(g, p, box)
    d = m.egnn_edge_geometry(g, p, box)[0].cpu().numpy()[:, 3]
    key = np.clip(np.floor(d * (np.float32(B.LENGTH_BINS) / np.float32(8.0))), 0, B.LENGTH_BINS - 1).astype(np.int64)
    assert np.array_equal(np.diff(g.len_ptr.cpu().numpy()), np.bincount(key, minlength=B.LENGTH_BINS))
    assert np.array_equal(g.len_perm.cpu().numpy(), np.argsort(key, kind="stable"))
    ws = torch.empty(m.egnn_backward_workspace_bytes(n_edges, n_owned, n_total), dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(g, ws)
    assert np.array_equal(np.diff(col_ptr.cpu().numpy()), np.bincount(src, minlength=n_total))
    assert np.array_equal(perm.cpu().numpy(), np.argsort(src, kind="stable"))
