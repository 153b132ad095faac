"""GPU tests of the adjoint of the edge block where the weight gradients of all orders share a launch: edges at the ends of its
chunks (64 edges at least), results of fewer than four 128 x 64 quarters, and a workspace that only holds one order's sums."""
import numpy as np
import pytest

from oracle import so2_oracle as S
from paper_2507_03840_amd import synth
from tests import gpu_util as U
from tests.test_gpu_so2_backward import check
from tests.test_gpu_so2_blocks_backward import oracle_weight_grads, weight_grads

pytestmark = pytest.mark.gpu

# Rotations, a contraction of up to 480 products of 22-bit operands and a sum over 2,901 edges: 100 roundings of 2^-24 in a row at most.
TOL = 6e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("lmax,E,n_edges", [(0, 8, 65), (0, 32, 1), (1, 8, 63), (1, 64, 129), (2, 16, 64), (2, 32, 257), (3, 8, 700), (3, 32, 191),
                                            (4, 16, 66), (4, 32, 640), (4, 64, 130), (2, 128, 67), (1, 128, 2901)])
def test_edge_block_backward_orders(B, lmax, E, n_edges):
    import torch
    n = 30 if n_edges <= 870 else 60
    w = synth.small_cluster(n, n, lmax, E, 6, 20.0, 500 + lmax + E)
    src, dst, shift, _ = U.oracle_graph(w)
    src, dst, shift = src[:n_edges], dst[:n_edges], shift[:n_edges]
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n))]).astype(np.int32)
    g = (src, dst, shift, row_ptr)
    rng = np.random.default_rng(lmax * 100 + E)
    x = synth.node_features(rng, n, lmax, E)
    T, dT = (rng.standard_normal(size=(n_edges, (lmax + 1) ** 2, E), dtype=np.float32) for _ in range(2))
    W = synth.so2_weights(rng, lmax, E, 6)
    flat = np.concatenate([W[1].ravel()] + [m.ravel() for ri in zip(W[2], W[3]) for m in ri])
    m = B.Egnn(lmax, E, 6, 20.0, 1.0)
    graph = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), B.to_device(shift), n, n)
    most = m.egnn_so2_blocks_backward_workspace_bytes(n_edges, n)
    ws = torch.empty(max(most, m.egnn_backward_workspace_bytes(n_edges, n, n)), dtype=torch.uint8, device="cuda")
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    args = (graph, col_ptr, perm, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(T), B.to_device(flat), B.to_device(dT))
    ref = S.so2_edge_block_backward(g, w.pos, w.box, x, T, W[1], W[2], W[3], lmax, E, 20.0, dT)
    want = dict(dx=ref[0], dT=ref[1], **oracle_weight_grads(ref[2], ref[3], ref[4]))

    def run(nbytes):
        dx, dT_in, dW = m.egnn_so2_edge_block_backward(*args, ws[:nbytes])
        got = dict(dx=dx.cpu().numpy(), dT=dT_in.cpu().numpy(), **weight_grads(dW.cpu().numpy(), lmax, E))
        return check(got, want, TOL), got

    worst, got = run(most)
    lo, hi = 0, most                       # (refused, accepted)
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            run(mid)
            hi = mid
        except B.EgnnError as err:
            assert err.code == -3
            lo = mid
    small, again = run(hi)
    print(f"lmax {lmax} E {E} edges {n_edges}: {worst:.2e}, workspace {hi} of {most}: {small:.2e}", flush=True)
    assert hi + 512 < most or n_edges < 2901   # (less than the orders' sums take: a launch per order)
    assert np.array_equal(got["dx"], again["dx"]) and np.array_equal(got["dT"], again["dT"])
