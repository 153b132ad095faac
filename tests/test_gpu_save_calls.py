"""GPU tests of the calls that keep forward quantities (egnn_*_save) and of those that recompute them (egnn_*_backward, and
egnn_*_backward_saved without some of them): what they prepare, and the bits that they promise."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# Products of 64 terms of 22-bit operands and about 30 fp32 operations in a row before them, 2^-24 each, added without sign.
TOL_W = 2e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def _case(B, lmax, E, n, n_owned, n_rbf, r_cut, shared, orb=(0, 0, 1, 1, 2)):
    import torch
    w = synth.small_cluster(n, n_owned, lmax, E, n_rbf, r_cut, 900 + n + lmax)
    m = B.Egnn(lmax, E, n_rbf, r_cut, 20.0, orb_l=orb)
    pos = B.to_device(w.pos)
    g = m.egnn_nlist(pos, n_owned, w.box, w.pbc)
    if shared:
        m.egnn_edge_pairs(g)
    rng = np.random.default_rng([lmax, E, n])
    W = synth.layer_weights(rng, lmax, E, n_rbf, 64, m.n_paths)
    R = synth.readout_weights(rng, lmax, E, n_rbf, 64, m.n_paths_readout, sum(m.n_out))
    ws = torch.empty(max(m.egnn_backward_workspace_bytes(g.n_edges, n_owned, n), m.egnn_workspace_bytes(g.n_edges, n_owned, n)),
                     dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(g, ws)
    x = B.to_device(synth.node_features(rng, n, lmax, E))
    dy = B.to_device(synth.node_features(rng, n_owned, lmax, E))
    dH = B.to_device(rng.standard_normal((g.n_edges, m.n_orb, m.n_orb)).astype(np.float32))
    return w, m, g, pos, W, R, B.to_device(W), B.to_device(R), ws, col_ptr, perm, x, dy, dH


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("lmax,E", [(2, 32), (4, 16)])
def test_saving_and_recomputing_calls_prepare_once(B, lmax, E, shared):
    """Launches: edge vectors, scalings, pieces and hidden layer once for the weights that are kept and for the sums; one pre mix."""
    import torch
    w, m, g, pos, _, _, W, R, ws, col_ptr, perm, x, dy, _ = _case(B, lmax, E, 150, 150, 11, 7.0, shared)
    assert U.fused_route(B, m, "layer", g.n_edges, 150, 150) and U.fused_route(B, m, "readout", g.n_edges, 150, 150)
    count = lambda f: U.recorded_nodes(m.lib, f)
    plain = count(lambda: m.egnn_layer_forward(g, pos, w.box, x, W, ws))
    save = count(lambda: m.egnn_layer_forward_save(g, pos, w.box, x, W, ws))
    ro = count(lambda: m.egnn_readout_hij(g, pos, w.box, x, R, ws))
    ro_save = count(lambda: m.egnn_readout_hij_save(g, pos, w.box, x, R, ws))
    _, kept = m.egnn_layer_forward_save(g, pos, w.box, x, W, ws)
    back = count(lambda: m.egnn_layer_backward(g, col_ptr, perm, pos, w.box, x, W, dy, ws))
    back_saved = count(lambda: m.egnn_layer_backward_saved(g, col_ptr, perm, pos, w.box, x, W, kept, dy, ws))
    torch.cuda.synchronize()
    print(f"nodes: layer {plain} {save}, readout {ro} {ro_save}, adjoint {back} {back_saved}", flush=True)
    assert save == plain + 1 and ro_save == ro + 1          # S3 beside the rest
    assert back == back_saved + 3                           # pieces, S3 and sums beside the edge vectors and the pre mix


# Both routes (lmax 0 and 1, and sparse graphs, take the weight tensor), all channel counts, halo nodes, more than 16 Gaussians;
# few and many rows of weights, column blocks of S3 shared out over workgroups and not.
@pytest.mark.parametrize("lmax,E,n,n_owned,n_rbf,r_cut", [
    (0, 32, 60, 60, 8, 6.0), (1, 32, 90, 70, 11, 6.0), (1, 64, 400, 400, 8, 5.0), (2, 8, 150, 150, 20, 7.0), (2, 64, 333, 250, 16, 6.5),
    (2, 16, 30, 30, 8, 2.5), (3, 32, 200, 200, 32, 6.0), (3, 128, 80, 60, 8, 6.0), (4, 16, 220, 180, 16, 8.0), (4, 64, 70, 70, 5, 7.0)])
@pytest.mark.parametrize("shared", [False, True])
def test_bits_of_saved_and_recomputed_quantities(B, lmax, E, n, n_owned, n_rbf, r_cut, shared):
    import torch
    w, m, g, pos, Wh, Rh, W, R, ws, col_ptr, perm, x, dy, dH = _case(B, lmax, E, n, n_owned, n_rbf, r_cut, shared)
    routes = [U.fused_route(B, m, k, g.n_edges, n_owned, n) for k in ("layer", "readout")]
    print("case", lmax, E, n, "edges", g.n_edges, "shared", shared, "routes", routes, flush=True)
    same = lambda a, b: all(torch.equal(a[k], b[k]) for k in a)
    y = m.egnn_layer_forward(g, pos, w.box, x, W, ws)
    ws.fill_(0xFF)
    y2, (w_k, a_k) = m.egnn_layer_forward_save(g, pos, w.box, x, W, ws)
    assert torch.equal(y, y2)
    H = m.egnn_readout_hij(g, pos, w.box, x, R, ws)
    ws.fill_(0xFF)
    H2, wr_k = m.egnn_readout_hij_save(g, pos, w.box, x, R, ws)
    assert torch.equal(H, H2)
    # the kept weights against the oracle, row by row
    edges = g.src.cpu().numpy(), g.dst.cpu().numpy(), g.shift.cpu().numpy().reshape(-1, 3)
    d = np.linalg.norm(O.edge_vectors(w.pos, w.box, *edges), axis=1)
    row = np.arange(g.n_edges)
    if shared:
        row = g.w_row.cpu().numpy()
        row = np.where(row < 0, ~row, row)
    for kept, mats, l_out in ((w_k, Wh, lmax), (wr_k, Rh, O.L_READOUT)):
        paths = O.tp_paths(lmax, lmax, l_out)
        ref = O.radial_weights(d, mats["W_r1"], mats["W_r2"], paths, E, n_rbf, r_cut)
        e = U.rel_err(kept.cpu().numpy()[row], ref)
        print(f"  kept weights: {e:.2e}", flush=True)
        assert e < TOL_W
    # gradients: nothing, either or both kept
    dx, grads = m.egnn_layer_backward(g, col_ptr, perm, pos, w.box, x, W, dy, ws)
    for kept in ((None, None), (w_k, None), (None, a_k), (w_k, a_k)):
        ws.fill_(0xFF)
        dx2, grads2 = m.egnn_layer_backward_saved(g, col_ptr, perm, pos, w.box, x, W, kept, dy, ws)
        assert torch.equal(dx, dx2) and same(grads, grads2)
    dx, grads = m.egnn_readout_backward(g, col_ptr, perm, pos, w.box, x, R, dH, ws)
    for kept in (None, wr_k):
        ws.fill_(0xFF)
        dx2, grads2 = m.egnn_readout_backward_saved(g, col_ptr, perm, pos, w.box, x, R, kept, dH, ws)
        assert torch.equal(dx, dx2) and same(grads, grads2)


@pytest.mark.parametrize("lmax,E,shared", [(2, 32, True), (3, 128, False), (4, 16, True)])
def test_saving_and_recomputing_calls_replay_from_a_graph(B, lmax, E, shared):
    """Recorded once (kernels only), replayed with new features and positions in the recorded buffers: the bits of eager calls."""
    import torch
    w, m, g, pos, _, _, W, R, ws, col_ptr, perm, x, dy, _ = _case(B, lmax, E, 120, 100, 11, 7.0, shared)
    readout = U.fused_route(B, m, "readout", g.n_edges, 100, 120)         # (the other route copies tables: not meant to be recorded)

    def calls():
        y, kept = m.egnn_layer_forward_save(g, pos, w.box, x, W, ws)
        out = [y, *kept]
        if readout:
            out += m.egnn_readout_hij_save(g, pos, w.box, x, R, ws)
        dx, grads = m.egnn_layer_backward(g, col_ptr, perm, pos, w.box, x, W, dy, ws)
        return out + [dx] + [grads[k] for k in sorted(grads)]

    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        recorded = calls()
    rng = np.random.default_rng(5)
    for rep in range(4):
        print("replay", rep, "readout", readout, flush=True)
        if rep >= 2:
            x.copy_(B.to_device(rng.standard_normal(tuple(x.shape)).astype(np.float32)))
            pos.add_(B.to_device((1e-3 * rng.standard_normal(tuple(pos.shape))).astype(np.float32)))
        want = [t.clone() for t in calls()]
        torch.cuda.synchronize()
        ws.fill_(0xFF)
        for t in recorded:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(recorded, want))
