"""GPU tests of the readout's reverse pass on the matrix cores with the radial weights' gradient summed per length interval
(readout_adjoint.hip): channel counts, orbital sets that fill and that leave empty the room of a degree, ragged edge counts, intervals of
no, few and hundreds of edges, halo atoms, against the oracle and the route with dw in memory."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from paper_2507_03840_amd import synth
from tests import gpu_util as U
from tests.test_gpu_tp_bins import _cluster

pytestmark = pytest.mark.gpu

# As in test_gpu_tp_bins: about 100 fp32 operations in a row, 2^-24 each, added without sign.
TOL = 6e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


SSPPD, SPPD, PPPP, SSDD, SP, PD = (0, 0, 1, 1, 2), (0, 1, 1, 2), (1, 1, 1, 1), (0, 0, 2, 2), (0, 1), (1, 2)


@pytest.mark.parametrize("lmax,E,n,n_owned,lattice,orb", [
    (1, 64, 118, 103, False, SSPPD), (2, 32, 119, 119, True, PPPP), (2, 128, 118, 118, False, SPPD), (3, 16, 120, 107, False, SSPPD),
    (3, 64, 118, 118, True, SSDD), (4, 32, 118, 117, False, SSPPD), (4, 16, 118, 118, True, SSDD), (4, 64, 118, 110, False, SP),
    (4, 128, 111, 111, False, PD), (4, 32, 205, 204, True, SP)])
def test_readout_adjoint(B, lmax, E, n, n_owned, lattice, orb):
    w = _cluster(lmax, E, n, n_owned, lattice, 70 + lmax + E)
    g = U.oracle_graph(w)
    n_edges, n_orb = len(g[0]), sum(2 * l + 1 for l in orb)
    print("case", lmax, E, n, n_owned, n_edges, orb, flush=True)
    m = B.Egnn(lmax, E, w.n_rbf, w.r_cut, float(n), orb_l=orb)
    assert n_edges == n_owned * (n - 1) and U.readout_adjoint_route(m, n_edges)
    pos = B.to_device(w.pos)
    graph = m.egnn_nlist(pos, n_owned, w.box, w.pbc)
    if n_owned % 2:
        m.egnn_edge_pairs(graph)
    ws = m.backward_workspace(graph)
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.readout_weights(rng, lmax, E, w.n_rbf, 64, m.n_paths_readout, sum(m.n_out))
    x = synth.node_features(rng, n, lmax, E)
    dH = synth.normal(rng, (n_edges, n_orb, n_orb))
    dx_ref, g_ref = O.readout_backward(g, w.pos, w.box, x, W, lmax, lmax, E, w.n_rbf, w.r_cut, orb, dH.astype(np.float64))

    def run(route, dH):
        m.egnn_set_option(B.OPT_RADIAL_BWD, route)
        dx, grads = m.egnn_readout_backward(graph, col_ptr, perm, pos, w.box, B.to_device(x), B.to_device(W), B.to_device(dH), ws)
        return dict(dx=dx.cpu().numpy(), **{k: v.cpu().numpy() for k, v in grads.items()})

    ref = dict(dx=dx_ref, **g_ref)
    grid, again, exact = run(2, dH), run(2, dH), run(1, dH)
    for k in ref:
        e, e1 = U.rel_err(grid[k], ref[k]), U.rel_err(exact[k], ref[k])
        print(f"  {k}: {e:.2e} (exact route {e1:.2e})", flush=True)
        assert np.abs(ref[k]).max() > 0 and e < TOL and e1 < U.TOL, k      # (the exact route: bf16 pieces, its own bar)
        assert np.array_equal(grid[k], again[k]), k
    # a block that is not finite stays with the atoms of its edge
    k_bad = n_edges // 3
    hit = np.zeros(n, bool)
    hit[[g[0][k_bad], g[1][k_bad]]] = True
    for bad in (np.nan, np.inf):
        dH2 = dH.copy()
        dH2[k_bad] = bad
        got = run(2, dH2)["dx"]
        assert np.array_equal(got[~hit], grid["dx"][~hit]) and not np.isfinite(got[hit]).all()
