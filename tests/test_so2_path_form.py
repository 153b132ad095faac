"""The node-wise form of the SO(2) message sum, in 64 bits: sums of harmonics times features first, then coupling tensors and
path weights from the library's table generator, against the per-edge oracle."""
import importlib.util
import os

import numpy as np
import pytest

from oracle import egnn_oracle as O
from oracle import so2_oracle as S
from paper_2507_03840_amd import synth
from tests import gpu_util as U


@pytest.fixture(scope="module")
def G():
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_03840_amd", "csrc", "gen_tables.py")
    spec = importlib.util.spec_from_file_location("gen_tables", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("lmax,E,n,n_owned", [(0, 8, 12, 12), (1, 8, 14, 9), (2, 8, 16, 12), (3, 8, 12, 7), (4, 8, 14, 10)])
def test_node_wise_sum_is_the_per_edge_sum(G, lmax, E, n, n_owned):
    w = synth.small_cluster(n, n_owned, lmax, E, 6, 5.0, 40 + lmax)
    g = U.oracle_graph(w)
    src, dst, shift, _ = g
    rng = np.random.default_rng(lmax)
    x = synth.node_features(rng, n, lmax, E).astype(np.float64)
    W_e, W0, Wr, Wi = synth.so2_weights(rng, lmax, E, 6)
    ref = S.so2_message_sum(g, w.pos, w.box, x, W_e, W0, Wr, Wi, lmax, E, 6, w.r_cut, 3.0)
    r = O.edge_vectors(w.pos, w.box, src, dst, shift)
    d = np.sqrt((r * r).sum(1))
    Y = G.eval_harmonics(r / d[:, None]) * O.envelope(d, w.r_cut)[:, None]
    e0 = O.radial_basis(d, 6, w.r_cut) @ W_e.astype(np.float64).T
    a = np.zeros((n_owned, (lmax + 1) ** 2, E))
    for j in range(n_owned):
        k = np.nonzero(dst == j)[0]
        Sj = np.einsum("kL,kqc->Lqc", Y[k], x[src[k]])
        gj = Y[k].sum(0)
        for lo in range(lmax + 1):
            rows = slice((lo) * E, (lo + 1) * E)
            a[j, O.sl(lo)] += np.einsum("kM,kc,dc->Md", Y[k][:, O.sl(lo)], e0[k], W0[rows, 2 * E:3 * E]) / np.sqrt(2 * lo + 1)
            for li in range(lmax + 1):
                for L in range(abs(lo - li), lo + li + 1):
                    C, beta = G.coupling_real(lo, li, L), G.so2_beta(lo, li, L)
                    T = [np.einsum("oiM,Mic->oc", C, Sj[O.sl(L)][:, O.sl(li)]), np.einsum("oiM,M,ic->oc", C, gj[O.sl(L)], x[j, O.sl(li)])]
                    for m in range(min(lo, li) + 1):
                        Wm = (W0 if m == 0 else Wr[m - 1]) if (lo + li + L) % 2 == 0 else (None if m == 0 else Wi[m - 1])
                        if Wm is None:
                            assert beta[m] == 0.0
                            continue
                        for grp in range(2):
                            c0 = (li - m) * 3 * E + grp * E
                            a[j, O.sl(lo)] += beta[m] * T[grp] @ Wm[(lo - m) * E:(lo - m + 1) * E, c0:c0 + E].T
    assert np.abs(a / np.sqrt(3.0) - ref).max() < 1e-10 * np.abs(ref).max()
