"""GPU tests of the radial weights' gradient summed per length interval as it is made (tp_bins.hip): intervals of no, few and
hundreds of edges, every channel count, odd numbers of paths, halo atoms, against the oracle and the exact route."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# About 100 fp32 operations in a row between an input and a sum (two rotations, products, sums of an interval and of the intervals),
# 2^-24 each, added without sign: 6e-6 of the largest result; the interpolation is below 5e-9 of it for such weights.
TOL = 6e-6


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def _cluster(lmax, E, n, n_owned, lattice, seed):
    """All atoms within reach of each other.  lattice: a cubic one with 1e-4 Angstrom of jitter, whose shells put hundreds of edges into
    one interval of lengths and none into most."""
    w = synth.small_cluster(n, n_owned, lmax, E, 7, 32.0, seed)
    if lattice:
        side = int(np.ceil(n ** (1 / 3) - 1e-9))
        g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
        rng = np.random.default_rng(seed)
        w.pos[:] = (2.7 * g + 1.0 + 1e-4 * rng.normal(size=(n, 3))).astype(np.float32)
    return w


@pytest.mark.parametrize("lmax,E,n,n_owned,lattice", [(1, 8, 118, 118, False), (1, 64, 118, 118, True), (2, 16, 121, 110, True),
                                                      (2, 128, 118, 118, False), (3, 32, 118, 118, False), (3, 16, 180, 170, True),
                                                      (4, 32, 125, 118, True), (4, 64, 118, 118, False), (4, 16, 175, 175, False),
                                                      (4, 8, 246, 246, True)])
def test_layer_adjoint(B, lmax, E, n, n_owned, lattice):
    w = _cluster(lmax, E, n, n_owned, lattice, 40 + lmax + E)
    g = U.oracle_graph(w)
    n_edges = len(g[0])
    assert n_edges == n_owned * (n - 1)
    print("case", lmax, E, n, n_owned, n_edges, flush=True)
    m = B.Egnn(lmax, E, w.n_rbf, w.r_cut, float(n))
    assert U.tp_bins_route(m, n_edges)
    pos = B.to_device(w.pos)
    graph = m.egnn_nlist(pos, n_owned, w.box, w.pbc)
    assert graph.n_edges == n_edges
    ws = m.backward_workspace(graph)
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    rng = np.random.default_rng(lmax * 100 + E)
    W = synth.layer_weights(rng, lmax, E, w.n_rbf, 64, m.n_paths)
    x, dy = synth.node_features(rng, n, lmax, E), synth.node_features(rng, n_owned, lmax, E)
    dx_ref, g_ref = O.layer_backward(g, w.pos, w.box, x, W, lmax, lmax, E, w.n_rbf, w.r_cut, float(n), dy.astype(np.float64))

    def run(route):
        m.egnn_set_option(B.OPT_RADIAL_BWD, route)
        dx, grads = m.egnn_layer_backward(graph, col_ptr, perm, pos, w.box, B.to_device(x), B.to_device(W), B.to_device(dy), ws)
        return dict(dx=dx.cpu().numpy(), **{k: v.cpu().numpy() for k, v in grads.items()})

    ref = dict(dx=dx_ref, **g_ref)
    grid, again, exact = run(2), run(2), run(1)
    for k in ref:
        e, e1 = U.rel_err(grid[k], ref[k]), U.rel_err(exact[k], ref[k])
        print(f"  {k}: {e:.2e} (exact route {e1:.2e})", flush=True)
        assert np.abs(ref[k]).max() > 0 and e < TOL and e1 < TOL, k
        assert np.array_equal(grid[k], again[k]), k
    for k in ref:      # what does not go through the radial MLP is the same either way
        if k not in ("W_r1", "W_r2"):
            assert U.rel_err(grid[k], exact[k]) < 1e-6, k
