"""GPU tests of the layer kernel that keeps the radial weights in registers (edge_fused.hip), at the edges of its tiles: nodes
of 0, 1, 15, 16, 17, 31, 32 and 33 edges, every channel count that it takes, with and without shared rows of weights, wavefronts that
take one node and wavefronts that take several, against the oracle on the same edge list; and the graphs that go through a weight
tensor instead."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

DEGREES = (0, 1, 15, 16, 17, 31, 32, 33)
# About 100 fp32 operations in a row between an input and a sum (two rotations, 64-term products of 22-bit operands, up to 33
# edges), 2^-24 each, added without sign: 6e-6 of the largest result.
TOL = 6e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def _pruned(lmax, E, n, n_owned, seed, want=None, r_cut=14.0):
    """A cluster whose owned atoms keep as many edges as `want` or else DEGREES says in turn (the cutoff gives each at least 33)."""
    w = synth.small_cluster(n, n_owned, lmax, E, 11, r_cut, seed)
    src, dst, shift, row_ptr = U.oracle_graph(w)
    rank = np.arange(len(src)) - row_ptr[:-1][dst]
    want = np.array([DEGREES[j % len(DEGREES)] for j in range(n_owned)] if want is None else want)
    keep = rank < want[dst]
    count = np.bincount(dst[keep], minlength=n_owned)
    assert np.array_equal(count, want)
    row_ptr2 = np.concatenate([[0], np.cumsum(count)]).astype(np.int32)
    return w, (src[keep], dst[keep], shift[keep], row_ptr2)


def _run(B, w, g, W, x, shared, half=False):
    m = B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, 7.0)
    if half:
        m.egnn_set_option(B.OPT_W_FP16, 1)
    graph = B.Graph(B.to_device(g[0]), B.to_device(g[1]), B.to_device(g[3]), B.to_device(g[2]), w.n_owned, w.n_total)
    if shared:
        m.egnn_edge_pairs(graph)
    y = m.egnn_layer_forward(graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(W), m.workspace(graph))
    return y.cpu().numpy()


@pytest.mark.parametrize("lmax,E,n,n_owned,half", [(1, 32, 90, 90, False), (1, 64, 90, 60, False), (2, 16, 90, 61, False),
                                                   (2, 64, 75, 75, True), (3, 8, 90, 70, False), (3, 128, 70, 50, False),
                                                   (4, 16, 80, 80, True), (4, 32, 90, 67, False)])
def test_tile_edges(B, lmax, E, n, n_owned, half):
    w, g = _pruned(lmax, E, n, n_owned, 60 + lmax + E)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.layer_weights(rng, lmax, E, w.n_rbf, 64, len(O.tp_paths(lmax, lmax, lmax)))
    x = synth.node_features(rng, n, lmax, E)
    ref = O.layer_forward(g, w.pos, w.box, x, W, lmax, lmax, E, w.n_rbf, w.r_cut, 7.0,
                          w_dtype=np.float16 if half else None)
    a = _run(B, w, g, W, x, False, half)
    b = _run(B, w, g, W, x, True, half)
    assert np.array_equal(a, b)                  # the rows of an edge and its reverse are the same numbers
    e = U.rel_err(a, ref)
    print(f"lmax {lmax} E {E} half {half}: rel err {e:.2e}", flush=True)
    assert e < (1e-4 if half else TOL)           # (half: a weight next to a rounding boundary may fall to either side)


def test_what_is_not_finite_stays_with_its_edges(B):
    """Lanes past a node's last edge work on edges of other nodes: a source that is not finite shows in its own destinations only."""
    lmax, E, n = 3, 32, 90
    w, g = _pruned(lmax, E, n, n, 5)
    rng = np.random.default_rng(8)
    W = synth.layer_weights(rng, lmax, E, w.n_rbf, 64, len(O.tp_paths(lmax, lmax, lmax)))
    x = synth.node_features(rng, n, lmax, E)
    clean = _run(B, w, g, W, x, True)
    for bad in (np.nan, np.inf):
        x2 = x.copy()
        x2[17] = bad
        got = _run(B, w, g, W, x2, True)
        hit = np.zeros(n, bool)
        hit[g[1][g[0] == 17]] = True
        hit[17] = True                           # (its own row, by the self term)
        assert hit.sum() < n // 2
        assert np.array_equal(got[~hit], clean[~hit])
        assert not np.isfinite(got[hit]).all(axis=(1, 2)).any()


def _stride(E):
    """Nodes between two that one wavefront takes, where there are enough of them: the workgroups that the chip holds, four wavefronts
    each, shared out over the groups of four channels."""
    return 4 * 2 * 256 // (E // 4)


# Degrees of the nodes that a wavefront takes one after the other: runs of empty ones, one tile after several, the last of a tile.
CHAINS = ((33, 0, 0, 16, 1), (0, 0, 0, 17, 0), (16, 16, 31, 0, 32), (1, 0, 33, 0, 15), (0, 32, 1, 0, 0), (17, 33, 0, 15, 16))


def _chains(E, n_owned):
    s = _stride(E)
    return [CHAINS[j % s % len(CHAINS)][j // s % 5] for j in range(n_owned)]


@pytest.mark.parametrize("lmax,E,n,n_owned,half", [(4, 128, 330, 300, False), (3, 64, 400, 390, False), (1, 64, 400, 400, False),
                                                   (4, 32, 700, 650, True), (2, 16, 1200, 1100, False), (2, 8, 2200, 2200, False)])
def test_several_nodes_a_wavefront(B, lmax, E, n, n_owned, half):
    assert n_owned > 2 * _stride(E) or E < 64
    w, g = _pruned(lmax, E, n, n_owned, 160 + lmax + E, _chains(E, n_owned), 14.0 if n < 1000 else 12.0)
    m = B.Egnn(lmax, E, 11, w.r_cut, 7.0)
    assert U.fused_route(B, m, "layer", len(g[0]), n_owned, n)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.layer_weights(rng, lmax, E, w.n_rbf, 64, len(O.tp_paths(lmax, lmax, lmax)))
    x = synth.node_features(rng, n, lmax, E)
    print("case", lmax, E, n_owned, len(g[0]), flush=True)
    ref = O.layer_forward(g, w.pos, w.box, x, W, lmax, lmax, E, w.n_rbf, w.r_cut, 7.0, w_dtype=np.float16 if half else None)
    a = _run(B, w, g, W, x, False, half)
    assert np.array_equal(a, _run(B, w, g, W, x, True, half))
    e = U.rel_err(a, ref)
    print(f"  rel err {e:.2e}", flush=True)
    assert e < (1e-4 if half else TOL)
    # a source that is not finite: neither the other lanes of its tiles nor the later nodes of their wavefronts see it
    clean = _run(B, w, g, W, x, False, half)
    for bad in (np.nan, np.inf):
        x2 = x.copy()
        sources = np.unique(g[0])[::23]
        x2[sources] = bad
        got = _run(B, w, g, W, x2, False, half)
        hit = np.zeros(n_owned, bool)
        hit[g[1][np.isin(g[0], sources)]] = True
        hit[sources[sources < n_owned]] = True
        assert 0 < hit.sum() < n_owned and not np.isfinite(got[hit]).all(axis=(1, 2)).any()
        assert np.array_equal(got[~hit], clean[~hit])


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("lmax,E,n,n_owned,r_cut", [(2, 16, 30, 30, 2.5), (2, 64, 60, 40, 1.9), (3, 8, 50, 50, 2.0), (3, 128, 40, 40, 2.2),
                                                    (4, 32, 60, 50, 2.0), (0, 32, 60, 60, 5.0), (1, 64, 450, 450, 4.0)])
def test_graphs_that_go_through_a_weight_tensor(B, lmax, E, n, n_owned, r_cut, shared):
    """Sparse and tiny graphs, whose weight tensor is less than the scratch of the other route; lmax 0; many nodes at lmax 1."""
    w = synth.small_cluster(n, n_owned, lmax, E, 9, r_cut, 260 + lmax + E)
    g = U.oracle_graph(w)
    m = B.Egnn(lmax, E, 9, w.r_cut, 7.0)
    assert len(g[0]) > 5 and not U.fused_route(B, m, "layer", len(g[0]), n_owned, n)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.layer_weights(rng, lmax, E, 9, 64, len(O.tp_paths(lmax, lmax, lmax)))
    x = synth.node_features(rng, n, lmax, E)
    ref = O.layer_forward(g, w.pos, w.box, x, W, lmax, lmax, E, 9, w.r_cut, 7.0)
    e = U.rel_err(_run(B, w, g, W, x, shared), ref)
    print(f"lmax {lmax} E {E}: {len(g[0])} edges, rel err {e:.2e}", flush=True)
    assert e < TOL
