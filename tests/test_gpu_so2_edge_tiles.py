"""GPU tests of the edge block over tiles of 32 edges (so2_edge.hip) at the ends of its tiles, for every number of units of work that
its four wavefronts share, against the oracle; not finite rows stay with their edges."""
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
