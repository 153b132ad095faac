"""SO(2) message sums whose channels are mixed per node: sizes at which the gathering kernel changes behaviour."""
import numpy as np
import pytest

from oracle import so2_oracle as S
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# Operands are cut to 22 bits twice (harmonics x features, coupled sums x weights), relative error 2^-22 per operand and
# product at most, four operands: 4 * 2.4e-7; as much again for the 32-bit sums over up to 300 edges and 3,300 products.
TOL = 2e-6
# The attention weights: __expf of a score difference of up to ~10, whose 32-bit rounding (a sum of up to 3,000 products)
# enters as an absolute error, 10 * 6e-8 times a few.
TOL_ATT = 5e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def case(lmax, E, n, n_owned, n_rbf):
    """Every atom within the cutoff of every other: degree n - 1."""
    w = synth.small_cluster(n, n_owned, lmax, E, n_rbf, 30.0, 300 + n)
    g = U.oracle_graph(w)
    assert len(g[0]) == n_owned * (n - 1)
    rng = np.random.default_rng([n, lmax, E])
    x = synth.node_features(rng, w.n_total, lmax, E)
    W_e, W0, Wr, Wi = synth.so2_weights(rng, lmax, E, n_rbf)
    return w, g, x, W_e, W0, Wr, Wi


@pytest.mark.parametrize("lmax,E,n,n_owned,n_rbf", [
    # around a step of 16 edges and the smallest degree of this route; one node, ragged numbers of nodes
    (4, 32, 25, 1, 2), (4, 32, 32, 9, 16), (4, 32, 33, 31, 16), (4, 32, 34, 5, 31),
    # around a batch of 256 staged edges
    (4, 32, 256, 3, 16), (4, 32, 257, 2, 32), (4, 32, 258, 3, 16), (2, 32, 300, 4, 8),
    # every degree and slice width (a partial tile of columns at 0/8, 0/16, 2/8, 2/16, 4/8, 4/16), several slices
    (0, 8, 40, 33, 5), (0, 16, 40, 8, 6), (0, 32, 30, 7, 6), (1, 8, 40, 9, 6), (1, 16, 33, 11, 6), (1, 64, 40, 9, 6),
    (2, 8, 30, 17, 6), (2, 16, 41, 16, 6), (3, 8, 29, 10, 6), (3, 16, 65, 10, 6), (3, 32, 49, 10, 6), (4, 8, 40, 13, 6),
    (4, 16, 47, 12, 6), (4, 64, 48, 11, 16), (3, 128, 31, 9, 8), (4, 128, 30, 5, 16),
    # lmax 0 takes this route only with many edges
    (0, 8, 130, 110, 5), (0, 16, 100, 80, 6), (0, 32, 60, 30, 6), (0, 128, 40, 21, 8)])
def test_message_sum_per_node(B, lmax, E, n, n_owned, n_rbf):
    import torch
    print("case", lmax, E, n, n_owned, n_rbf, flush=True)
    w, g, x, W_e, W0, Wr, Wi = case(lmax, E, n, n_owned, n_rbf)
    agg = 7.0
    ref = S.so2_message_sum(g, w.pos, w.box, x, W_e, W0, Wr, Wi, lmax, E, n_rbf, w.r_cut, agg)
    m = B.Egnn(lmax, E, n_rbf, w.r_cut, agg)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    args = (graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(W_e), B.to_device(S.so2_pack(W0, Wr, Wi)))
    # the workspace holds garbage at first: nothing of it may reach the result
    ws = torch.full((m.egnn_so2_workspace_bytes(graph.n_edges),), 0xFF, dtype=torch.uint8, device="cuda")
    a = m.egnn_so2_message_sum(*args, ws).cpu().numpy()
    e = U.rel_err(a, ref)
    print(f"  {graph.n_edges} edges, rel err {e:.2e}", flush=True)
    assert e < TOL
    assert np.array_equal(a, m.egnn_so2_message_sum(*args, ws).cpu().numpy())


@pytest.mark.parametrize("lmax,E,n,n_owned", [
    # around the smallest degree of this route (31 is below it), ragged tiles of 32 edges, a batch of 256
    (4, 32, 32, 9), (4, 32, 33, 1), (4, 32, 33, 31), (4, 32, 34, 5), (4, 32, 257, 2), (4, 32, 258, 3), (2, 32, 300, 4),
    (0, 8, 40, 33), (0, 16, 40, 8), (0, 32, 36, 7), (1, 8, 40, 9), (1, 64, 40, 9), (2, 8, 37, 17), (2, 16, 41, 16), (3, 8, 39, 10),
    (3, 16, 65, 10), (3, 32, 49, 10), (3, 64, 34, 10), (4, 8, 40, 13), (4, 16, 47, 12), (4, 64, 48, 11),
    # where fewer channels or degrees need more edges a node or more edges in all for this route
    (4, 8, 62, 5), (4, 16, 58, 7), (1, 8, 90, 80), (0, 8, 180, 150), (0, 16, 130, 110), (0, 64, 60, 58),
    (3, 128, 35, 9)])                                                  # (more channels than this route takes)
def test_node_block_per_node(B, lmax, E, n, n_owned):
    import torch
    print("case", lmax, E, n, n_owned, flush=True)
    w, g, x, W_e, W0, Wr, Wi = case(lmax, E, n, n_owned, 8)
    rng = np.random.default_rng(n)
    T = rng.standard_normal((len(g[0]), (lmax + 1) ** 2, E)).astype(np.float32)
    w_att = synth.normal(rng, (E,)).astype(np.float32)
    ref = S.so2_node_block(g, w.pos, w.box, x, T, W0, Wr, Wi, w_att, lmax, E, w.r_cut)
    m = B.Egnn(lmax, E, 8, w.r_cut, 7.0)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    args = (graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(T), B.to_device(S.so2_pack(W0, Wr, Wi)), B.to_device(w_att))
    ws = torch.full((m.egnn_so2_blocks_workspace_bytes(graph.n_edges),), 0xFF, dtype=torch.uint8, device="cuda")
    a = m.egnn_so2_node_block(*args, ws).cpu().numpy()
    e = U.rel_err(a, ref)
    print(f"  {graph.n_edges} edges, rel err {e:.2e}", flush=True)
    assert e < TOL_ATT
    assert np.array_equal(a, m.egnn_so2_node_block(*args, ws).cpu().numpy())


@pytest.mark.parametrize("lmax,E,n,n_owned", [
    # tiles of 64 edges: one edge, 63, 64, 65, several; units of one and of two slots; one and two blocks of output channels
    (4, 32, 2, 1), (4, 32, 64, 1), (4, 32, 65, 1), (4, 32, 66, 1), (4, 16, 30, 9), (4, 64, 41, 3), (3, 16, 23, 5), (3, 32, 40, 7),
    (3, 64, 33, 2), (2, 16, 66, 1), (2, 64, 20, 7), (1, 32, 25, 8), (0, 16, 30, 7), (0, 64, 30, 5),
    (3, 128, 20, 4), (4, 8, 20, 4)])                                   # (outside this route)
def test_edge_block_tiles(B, lmax, E, n, n_owned):
    import torch
    print("case", lmax, E, n, n_owned, flush=True)
    w, g, x, W_e, W0, Wr, Wi = case(lmax, E, n, n_owned, 8)
    rng = np.random.default_rng(n)
    # rows of very different size: every edge has a scale of its own; one row is zero
    size = 10.0 ** rng.uniform(-6, 6, size=(len(g[0]), 1, 1))
    T = (size * rng.standard_normal((len(g[0]), (lmax + 1) ** 2, E))).astype(np.float32)
    T[len(g[0]) // 2] = 0
    ref = S.so2_edge_block(g, w.pos, w.box, x, T, W0, Wr, Wi, lmax, E, w.r_cut)
    m = B.Egnn(lmax, E, 8, w.r_cut, 7.0)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    Td = B.to_device(T)
    args = (graph, B.to_device(w.pos), w.box, B.to_device(x))
    Wd = B.to_device(S.so2_pack(W0, Wr, Wi))
    ws = torch.full((m.egnn_so2_blocks_workspace_bytes(graph.n_edges),), 0xFF, dtype=torch.uint8, device="cuda")
    out = m.egnn_so2_edge_block(*args, Td, Wd, ws)
    got = out.cpu().numpy().astype(np.float64)
    # update of each edge against the largest of that edge (the per-edge kernels scale all edges alike, so only by 1e-2 of all)
    upd, want = got - T, ref - T
    tiles = 16 <= E <= 64
    rows = np.abs(want).max(axis=(1, 2)) if tiles else np.full(len(T), np.abs(want).max())
    rounding = 2.0 ** -23 * np.abs(ref).max(axis=(1, 2))                # of T + update
    err = np.abs(upd - want).max(axis=(1, 2))
    print(f"  {len(T)} edges, worst {np.max(err / (rows + rounding)):.2e}", flush=True)
    assert np.all(err <= TOL * rows + rounding)
    # in place
    T2 = Td.clone()
    m.egnn_so2_edge_block(*args, T2, Wd, ws, out=T2)
    if E != 64:
        assert torch.equal(T2, out)
    else:
        assert np.all(np.abs(T2.cpu().numpy() - ref).max(axis=(1, 2)) <= 2 * TOL * np.abs(want).max() + rounding)


@pytest.mark.parametrize("lmax,E,n,n_owned", [(4, 64, 41, 3), (0, 64, 30, 5), (2, 64, 20, 7), (3, 32, 40, 7), (3, 128, 20, 4), (4, 8, 20, 4)])
def test_edge_block_in_place(B, lmax, E, n, n_owned):
    """The result does not depend on whether the output is the input, on any route."""
    import torch
    print("case", lmax, E, n, n_owned, flush=True)
    w, g, x, W_e, W0, Wr, Wi = case(lmax, E, n, n_owned, 8)
    rng = np.random.default_rng(n)
    T = (10.0 ** rng.uniform(-6, 6, size=(len(g[0]), 1, 1)) * rng.standard_normal((len(g[0]), (lmax + 1) ** 2, E))).astype(np.float32)
    m = B.Egnn(lmax, E, 8, w.r_cut, 7.0)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    args = (graph, B.to_device(w.pos), w.box, B.to_device(x))
    Td, Wd = B.to_device(T), B.to_device(S.so2_pack(W0, Wr, Wi))
    ws = torch.full((m.egnn_so2_blocks_workspace_bytes(graph.n_edges),), 0xFF, dtype=torch.uint8, device="cuda")
    out = m.egnn_so2_edge_block(*args, Td, Wd, ws)
    ws.fill_(0xFF)
    T2 = Td.clone()
    assert m.egnn_so2_edge_block(*args, T2, Wd, ws, out=T2) is T2
    assert torch.equal(T2, out)


# Weight gradients are differences of sums over all edges: the fp32 rounding of the terms enters with the ratio of their
# size to the result's, a few times at these shapes.
TOL_BWD = 5e-6


@pytest.mark.parametrize("lmax,E,n,n_owned,n_rbf", [
    (4, 32, 34, 31, 16), (4, 32, 40, 28, 31), (4, 32, 270, 30, 16), (0, 8, 40, 33, 5), (0, 32, 30, 29, 6), (1, 8, 40, 30, 6),
    (1, 64, 41, 36, 6), (2, 16, 51, 49, 2), (2, 32, 47, 47, 32), (3, 8, 33, 30, 6), (3, 32, 49, 40, 6), (4, 8, 40, 33, 6),
    (4, 16, 35, 33, 6), (4, 64, 36, 31, 16), (3, 128, 31, 29, 8), (4, 128, 30, 27, 16)])
def test_message_sum_backward_per_node(B, lmax, E, n, n_owned, n_rbf):
    import torch
    from tests.test_gpu_so2_backward import check, unpack
    print("case", lmax, E, n, n_owned, n_rbf, flush=True)
    assert n_owned * (n - 1) >= 24 * n     # (otherwise the per-edge route)
    w, g, x, W_e, W0, Wr, Wi = case(lmax, E, n, n_owned, n_rbf)
    agg = 7.0
    da = np.random.default_rng(n).standard_normal((n_owned, (lmax + 1) ** 2, E)).astype(np.float32)
    ref = S.so2_message_sum_backward(g, w.pos, w.box, x, W_e, W0, Wr, Wi, lmax, E, n_rbf, w.r_cut, agg, da)
    m = B.Egnn(lmax, E, n_rbf, w.r_cut, agg)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    ws = torch.full((max(m.egnn_so2_backward_workspace_bytes(graph.n_edges, n_owned),
                         m.egnn_backward_workspace_bytes(graph.n_edges, n_owned, n)),), 0xFF, dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    args = (graph, col_ptr, perm, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(W_e),
            B.to_device(S.so2_pack(W0, Wr, Wi)), B.to_device(da))
    ws.fill_(0xFF)
    dx, dW_e, dW = m.egnn_so2_message_sum_backward(*args, ws)
    g0, gr, gi = unpack(dW.cpu().numpy(), lmax, E)
    got, want = dict(dx=dx.cpu().numpy(), dW_e=dW_e.cpu().numpy(), dW0=g0), dict(dx=ref[0], dW_e=ref[1], dW0=ref[2])
    for i in range(lmax):
        got[f"dWr{i + 1}"], got[f"dWi{i + 1}"], want[f"dWr{i + 1}"], want[f"dWi{i + 1}"] = gr[i], gi[i], ref[3][i], ref[4][i]
    print(f"  {graph.n_edges} edges, worst rel err {check(got, want, TOL_BWD):.2e}", flush=True)
    again = m.egnn_so2_message_sum_backward(*args, ws)
    assert all(torch.equal(a, b) for a, b in zip((dx, dW_e, dW), again))


# Open clusters with few edges a node: chains of steps that are mostly empty, nodes with no edge at all, halo nodes.
@pytest.mark.parametrize("lmax,E,n,n_owned,r_cut", [
    (2, 8, 40, 40, 2.7), (2, 32, 97, 80, 3.0), (2, 128, 33, 33, 3.4), (3, 16, 70, 60, 4.0), (3, 64, 65, 65, 3.6),
    (4, 8, 64, 64, 4.2), (4, 32, 129, 110, 4.6), (4, 64, 50, 50, 4.6)])
def test_message_sum_backward_few_edges(B, lmax, E, n, n_owned, r_cut):
    from tests.test_gpu_so2_backward import check, unpack
    print("case", lmax, E, n, n_owned, r_cut, flush=True)
    w = synth.small_cluster(n, n_owned, lmax, E, 8, r_cut, 500 + n)
    g = U.oracle_graph(w)
    rng = np.random.default_rng([n, lmax, E, 1])
    x, da = synth.node_features(rng, n, lmax, E), rng.standard_normal((n_owned, (lmax + 1) ** 2, E)).astype(np.float32)
    W_e, W0, Wr, Wi = synth.so2_weights(rng, lmax, E, 8)
    ref = S.so2_message_sum_backward(g, w.pos, w.box, x, W_e, W0, Wr, Wi, lmax, E, 8, w.r_cut, 3.0, da)
    m = B.Egnn(lmax, E, 8, w.r_cut, 3.0)
    graph = m.egnn_nlist(B.to_device(w.pos), n_owned, w.box, w.pbc)
    import torch
    ws = torch.full((max(m.egnn_so2_backward_workspace_bytes(graph.n_edges, n_owned),
                         m.egnn_backward_workspace_bytes(graph.n_edges, n_owned, n)),), 0xFF, dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    ws.fill_(0xFF)
    dx, dW_e, dW = m.egnn_so2_message_sum_backward(graph, col_ptr, perm, B.to_device(w.pos), w.box, B.to_device(x),
                                                   B.to_device(W_e), B.to_device(S.so2_pack(W0, Wr, Wi)), B.to_device(da), ws)
    g0, gr, gi = unpack(dW.cpu().numpy(), lmax, E)
    got, want = dict(dx=dx.cpu().numpy(), dW_e=dW_e.cpu().numpy(), dW0=g0), dict(dx=ref[0], dW_e=ref[1], dW0=ref[2])
    for i in range(lmax):
        got[f"dWr{i + 1}"], got[f"dWi{i + 1}"], want[f"dWr{i + 1}"], want[f"dWi{i + 1}"] = gr[i], gi[i], ref[3][i], ref[4][i]
    print(f"  {graph.n_edges / n:.1f} edges a node, worst rel err {check(got, want, TOL_BWD):.2e}", flush=True)


# The rows of the edges are added per source 16 bytes a lane, or 4 where the result does not begin at a multiple of 16: the same
# sums in the same order.  Segments of 0, 1, 7, 8, 9 ... rows; 32 to 1152 words a row.
@pytest.mark.parametrize("lmax,E,n,r_cut", [(1, 8, 60, 4.4), (0, 32, 40, 4.0), (1, 64, 33, 4.0), (2, 128, 21, 2.3), (1, 16, 11, 9.0)])
def test_sums_over_outgoing_edges_alignment(B, lmax, E, n, r_cut):
    import ctypes as C
    import torch
    print("case", lmax, E, n, r_cut, flush=True)
    w = synth.small_cluster(n, n, lmax, E, 6, r_cut, 700 + n)
    rng = np.random.default_rng([n, lmax, E, 2])
    D = (lmax + 1) ** 2
    x, da = (B.to_device(rng.standard_normal((n, D, E)).astype(np.float32)) for _ in range(2))
    W_e, W0, Wr, Wi = synth.so2_weights(rng, lmax, E, 6)
    W_e, W = B.to_device(W_e), B.to_device(S.so2_pack(W0, Wr, Wi))
    m = B.Egnn(lmax, E, 6, w.r_cut, 3.0)
    pos = B.to_device(w.pos)
    graph = m.egnn_nlist(pos, n, w.box, w.pbc)
    ws = torch.empty((max(m.egnn_so2_backward_workspace_bytes(graph.n_edges, n),
                          m.egnn_backward_workspace_bytes(graph.n_edges, n, n)),), dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    dx = m.egnn_so2_message_sum_backward(graph, col_ptr, perm, pos, w.box, x, W_e, W, da, ws)[0]
    room = torch.full((n * D * E + 2,), float("nan"), dtype=torch.float32, device="cuda")
    dW_e, dW, g = torch.empty_like(W_e), torch.empty_like(W), graph.desc()
    m._check(m.lib.egnn_so2_message_sum_backward(
        m.ctx, C.byref(g), B._ptr(col_ptr), B._ptr(perm), B._ptr(pos), B._f3(w.box), B._ptr(x), B._ptr(W_e), B._ptr(W),
        B._ptr(da), B._ptr(room[1:]), B._ptr(dW_e), B._ptr(dW), B._ptr(ws), C.c_size_t(ws.numel()), B._stream()))
    assert torch.equal(room[1:-1].view_as(dx), dx)
    assert torch.isnan(room[0]) and torch.isnan(room[-1])
