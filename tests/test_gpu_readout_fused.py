"""GPU tests of the readout kernel that keeps the radial weights in registers (readout_fused.hip): its batches of 128 edges and tiles
of 16 with odd remainders, one and several batches a workgroup, several orbital sets, every channel count that it takes, with and
without shared rows of weights, with the weights kept and rounded to half precision, against the oracle.  The cases that are
meant for this kernel ask the library whether it takes them; others go through a weight tensor (few edges, rows of V that it has
no room for)."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# About 150 fp32 operations in a row between an input and an entry of a block (mixing, rotations, 64-term products of 22-bit
# operands, the sum over channels, the coupling), 2^-24 each, added without sign: 9e-6 of the largest entry.
TOL = 9e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("lmax,E,orb,n_edges", [(1, 32, (0, 0, 1, 1, 2), 1), (2, 16, (0, 1), 15), (2, 8, (0, 0, 1, 1, 2), 129),
                                                (3, 32, (0, 0, 1, 1, 2), 1041), (4, 32, (0, 0, 1, 1, 2), 128),
                                                (4, 16, (1, 0, 2), 16), (3, 16, (2, 2, 1), 300), (4, 8, (0, 1, 0), 255)])
def test_odd_edge_counts_and_orbital_sets(B, lmax, E, orb, n_edges):
    """Either route: all but two of these are too few edges for the kernel, or too many rows of V."""
    w = synth.small_cluster(60, 40, lmax, E, 11, 9.0, 80 + lmax + E)
    src, dst, shift, _ = U.oracle_graph(w)
    keep = np.sort(np.random.default_rng(n_edges).permutation(len(src))[:n_edges])
    assert len(keep) == n_edges
    src, dst, shift = src[keep], dst[keep], shift[keep]
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=w.n_owned))]).astype(np.int32)
    g = (src, dst, shift, row_ptr)
    m = B.Egnn(lmax, E, 11, w.r_cut, 7.0, orb_l=orb)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.readout_weights(rng, lmax, E, 11, 64, len(O.tp_paths(lmax, lmax, O.L_READOUT)), sum(m.n_out))
    x = synth.node_features(rng, 60, lmax, E)
    ref = O.readout_hij(g, w.pos, w.box, x, W, lmax, lmax, E, 11, w.r_cut, orb)
    got = []
    for shared in (False, True):
        graph = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), B.to_device(shift), w.n_owned, w.n_total)
        if shared:
            m.egnn_edge_pairs(graph)
        got.append(m.egnn_readout_hij(graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(W),
                                      m.workspace(graph)).cpu().numpy())
    assert np.array_equal(got[0], got[1])
    e = U.rel_err(got[0], ref)
    print(f"lmax {lmax} E {E} orbitals {orb} edges {n_edges}: rel err {e:.2e}", flush=True)
    assert e < TOL


def _inputs(B, lmax, E, orb, n, n_edges, seed, r_cut=14.0):
    w = synth.small_cluster(n, n, lmax, E, 11, r_cut, seed)
    src, dst, shift, _ = U.oracle_graph(w)
    keep = np.sort(np.random.default_rng(n_edges).permutation(len(src))[:n_edges])
    assert len(keep) == n_edges
    src, dst, shift = src[keep], dst[keep], shift[keep]
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n))]).astype(np.int32)
    m = B.Egnn(lmax, E, 11, w.r_cut, 7.0, orb_l=orb)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.readout_weights(rng, lmax, E, 11, 64, len(O.tp_paths(lmax, lmax, O.L_READOUT)), sum(m.n_out))
    x = synth.node_features(rng, n, lmax, E)
    return w, (src, dst, shift, row_ptr), m, W, x


def _call(B, w, g, m, W, x, shared=False, save=False):
    graph = B.Graph(B.to_device(g[0]), B.to_device(g[1]), B.to_device(g[3]), B.to_device(g[2]), w.n_owned, w.n_total)
    if shared:
        m.egnn_edge_pairs(graph)
    ws = m.workspace(graph)
    ws.fill_(0xFF)
    args = (graph, B.to_device(w.pos), w.box, B.to_device(x), B.to_device(W), ws)
    return (m.egnn_readout_hij_save(*args)[0] if save else m.egnn_readout_hij(*args)).cpu().numpy()


SSPPD = (0, 0, 1, 1, 2)


@pytest.mark.parametrize("lmax,E,orb,n_edges", [
    (1, 32, SSPPD, 385), (1, 32, SSPPD, 511), (1, 16, (1, 2), 1501), (2, 16, (0, 1), 255), (2, 8, SSPPD, 399), (2, 32, SSPPD, 272), (2, 16, (1, 1), 641),
    (3, 32, SSPPD, 127), (3, 32, SSPPD, 129), (3, 16, (2, 1), 301), (4, 32, SSPPD, 128), (4, 32, SSPPD, 143), (4, 16, (1, 0, 2), 145),
    (4, 8, (0, 1, 0), 256), (4, 8, (2,), 1041), (4, 16, (0, 0, 0), 1551)])
def test_remainders_of_tiles_and_batches(B, lmax, E, orb, n_edges):
    w, g, m, W, x = _inputs(B, lmax, E, orb, 40, n_edges, 300 + lmax + E)
    assert U.fused_route(B, m, "readout", n_edges, 40, 40)
    ref = O.readout_hij(g, w.pos, w.box, x, W, lmax, lmax, E, 11, w.r_cut, orb)
    print("case", lmax, E, orb, n_edges, flush=True)
    H = _call(B, w, g, m, W, x)
    assert np.array_equal(H, _call(B, w, g, m, W, x, shared=True)) and np.array_equal(H, _call(B, w, g, m, W, x, save=True))
    e = U.rel_err(H, ref)
    m.egnn_set_option(B.OPT_W_FP16, 1)
    H16 = _call(B, w, g, m, W, x)
    assert np.array_equal(H, _call(B, w, g, m, W, x, save=True))       # (kept weights are fp32 whatever the option says)
    e16 = U.rel_err(H16, O.readout_hij(g, w.pos, w.box, x, W, lmax, lmax, E, 11, w.r_cut, orb, w_dtype=np.float16))
    print(f"  rel err {e:.2e}, half {e16:.2e}", flush=True)
    # (half: a weight next to a rounding boundary may fall to either side, 2^-10 of it; an entry is a sum over dozens of them, none of
    # which makes up a fifth of the largest entry)
    assert e < TOL and e16 < 2e-4
    assert not np.array_equal(H, H16)


# More than one batch for every workgroup (32,768 edges are one each), odd remainders: the first, some middle and the last edges
# against the oracle.  64 channels: on both sides of the line from which this kernel is taken there.
@pytest.mark.parametrize("lmax,E,orb,n,n_edges", [(3, 8, (0, 1), 200, 32769 + 6), (4, 16, SSPPD, 270, 65536 + 129), (2, 32, SSPPD, 260, 49153 + 16),
                                                  (4, 64, SSPPD, 400, 149999), (4, 64, SSPPD, 400, 150001), (2, 64, (0, 1, 1, 2), 400, 155555),
                                                  (1, 64, (0, 1, 2), 400, 150017)])
def test_several_batches_a_workgroup(B, lmax, E, orb, n, n_edges):
    w, g, m, W, x = _inputs(B, lmax, E, orb, n, n_edges, 400 + lmax + E, 40.0)
    assert U.fused_route(B, m, "readout", n_edges, n, n) == (n_edges != 149999)
    print("case", lmax, E, orb, n_edges, flush=True)
    H = _call(B, w, g, m, W, x, shared=True)
    scale = np.abs(H).max()
    for k0 in (0, 32768 - 150, n_edges // 2, n_edges - 300):
        k1 = min(k0 + 300, n_edges)
        ref = O.readout_hij(g, w.pos, w.box, x, W, lmax, lmax, E, 11, w.r_cut, orb, k_range=(k0, k1))
        e = np.abs(H[k0:k1] - ref).max() / scale
        print(f"  edges {k0} .. {k1}: rel err {e:.2e}", flush=True)
        assert e < TOL
