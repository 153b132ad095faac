"""GPU tests of the edge block over tiles of 32 edges (so2_edge.hip) at the ends of its tiles, for every number of units of work that
its four wavefronts share, and on the calls of few degrees that take the tiles, against the oracle; not finite rows stay with their edges."""
import numpy as np
import pytest

from oracle import so2_oracle as S
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# Two rotations, contractions of up to 480 products of 22-bit operands and the sum with T: 100 roundings of 2^-24 in a row at most.
TOL = 6e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("lmax,E,n_edges", [(0, 16, 321), (0, 32, 351), (1, 32, 320), (1, 64, 353), (2, 16, 319), (2, 64, 322), (3, 32, 321), (3, 16, 352),
                                            (4, 32, 319), (4, 32, 353), (4, 64, 321), (4, 16, 350)])
def test_ends_of_tiles(B, lmax, E, n_edges):
    import torch
    n = 30
    w = synth.small_cluster(n, n, lmax, E, 6, 20.0, 300 + lmax + E)
    src, dst, shift, _ = U.oracle_graph(w)
    src, dst, shift = src[:n_edges], dst[:n_edges], shift[:n_edges]
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n))]).astype(np.int32)
    g = (src, dst, shift, row_ptr)
    rng = np.random.default_rng(lmax * 100 + E)
    x = synth.node_features(rng, n, lmax, E)
    T = rng.standard_normal(size=(n_edges, (lmax + 1) ** 2, E), dtype=np.float32)
    W = synth.so2_weights(rng, lmax, E, 6)
    flat = np.concatenate([W[1].ravel()] + [m.ravel() for ri in zip(W[2], W[3]) for m in ri])
    m = B.Egnn(lmax, E, 6, 20.0, 1.0)
    graph = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), B.to_device(shift), n, n)
    ws = torch.empty(m.egnn_so2_blocks_workspace_bytes(n_edges), dtype=torch.uint8, device="cuda")
    run = lambda x, T: m.egnn_so2_edge_block(graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(T), B.to_device(flat), ws).cpu().numpy()
    got = run(x, T)
    ref = S.so2_edge_block(g, w.pos, w.box, x, T, W[1], W[2], W[3], lmax, E, 20.0)
    e = np.abs((got - T) - (ref - T)).max() / np.abs(ref - T).max()
    print(f"lmax {lmax} E {E} edges {n_edges}: update {e:.2e}", flush=True)
    assert e < TOL
    T2 = T.copy()
    T2[n_edges - 1] = np.nan
    again = run(x, T2)
    assert np.array_equal(again[:-1], got[:-1]) and not np.isfinite(again[-1]).any()


@pytest.mark.parametrize("lmax,E,n", [(0, 16, 560), (0, 32, 460), (0, 64, 310), (1, 64, 290), (2, 64, 220)])
def test_calls_of_few_degrees(B, lmax, E, n):
    """Up to 100,000 edges at 64 channels, 1,000,000 and more below, they take the same kernels as small calls."""
    import torch
    w = synth.small_cluster(n, n, lmax, E, 6, 40.0, 700 + lmax + E)
    g = src, dst, shift, row_ptr = U.oracle_graph(w)
    n_edges = len(src)
    assert n_edges == n * (n - 1)
    rng = np.random.default_rng(lmax * 100 + E)
    x = synth.node_features(rng, n, lmax, E)
    T = rng.standard_normal(size=(n_edges, (lmax + 1) ** 2, E), dtype=np.float32)
    W = synth.so2_weights(rng, lmax, E, 6)
    flat = np.concatenate([W[1].ravel()] + [m.ravel() for ri in zip(W[2], W[3]) for m in ri])
    m = B.Egnn(lmax, E, 6, 40.0, 1.0)
    ws = torch.empty(m.egnn_so2_blocks_workspace_bytes(n_edges), dtype=torch.uint8, device="cuda")
    pos, x_d, T_d, W_d = (B.to_device(v) for v in (w.pos, x, T, flat))
    out = torch.empty_like(T_d)

    def call(k):
        graph = B.Graph(B.to_device(src[:k]), B.to_device(dst[:k]), B.to_device(np.minimum(row_ptr, k).astype(np.int32)),
                        B.to_device(shift[:k]), n, n)
        return lambda: m.egnn_so2_edge_block(graph, pos, w.box, x_d, T_d[:k], W_d, ws, out=out[:k])

    small, large = U.recorded_nodes(m.lib, call(1000)), U.recorded_nodes(m.lib, call(n_edges))
    print(f"lmax {lmax} E {E} edges {n_edges}: {small}, {large} launches", flush=True)
    assert small == large
    call(n_edges)()
    for k in ((0, 300), (n_edges - 300, n_edges)):
        got = out[k[0]:k[1]].cpu().numpy()
        ref = S.so2_edge_block(g, w.pos, w.box, x, T, W[1], W[2], W[3], lmax, E, 40.0, k_range=k)
        ref = ref[k[0]:k[1]] if len(ref) == n_edges else ref
        assert np.abs((got - T[k[0]:k[1]]) - (ref - T[k[0]:k[1]])).max() / np.abs(ref - T[k[0]:k[1]]).max() < TOL
    if E == 64:                       # (through the workspace)
        again = T_d.clone()
        graph = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), B.to_device(shift), n, n)
        m.egnn_so2_edge_block(graph, pos, w.box, x_d, again, W_d, ws, out=again)
        assert torch.equal(again, out)
