"""GPU tests of the readout kernel that keeps the radial weights in registers (readout_fused.hip): its batches of 128 edges and tiles
of 16 with odd remainders, both orbital sets, every channel count that it takes, with and without shared rows of weights, against
the oracle."""
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
