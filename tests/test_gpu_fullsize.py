"""GPU parity at the full sizes of configs 3 and 4, in the launch configuration bench.py times.

The oracle needs minutes for these chains, so its outputs at sampled rows are stored under tests/golden/
(written by tests/golden/make_golden.py, which calls only the oracle).  The inputs are regenerated here from
the same seeds; the edge set must equal the brute-force oracle's (run live) array for array, and every sampled row
must lie within 1e-4 of the scale of its own block: per degree l for node tensors and gradients, per shell block
(alpha, beta) for H.  The stored rows include the first and last node, the nodes of least and greatest degree, the
owned atoms next to the halo and the last 64 edges.
"""
import os
import numpy as np
import pytest

from paper_2507_03840_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


_graphs = {}


def full_oracle_graph(index):
    """The brute-force oracle's edge list of a full-size configuration (seconds; computed once per test session)."""
    if index not in _graphs:
        _graphs[index] = U.oracle_graph(synth.workload(index))
    return _graphs[index]


def assert_same_graph(graph, g):
    """Edge set array for array: sources, destinations, periodic images and the row index."""
    assert graph.n_edges == len(g[0])
    assert np.array_equal(graph.row_ptr.cpu().numpy(), g[3])
    assert np.array_equal(graph.src.cpu().numpy(), g[0])
    assert np.array_equal(graph.dst.cpu().numpy(), g[1])
    assert np.array_equal(graph.shift.cpu().numpy(), g[2])


def rel_err_per_degree(got, ref, scales, lmax):
    """Largest error of every degree l over the sampled rows, relative to that degree's largest magnitude over the
    whole tensor: a degree whose values are far below the tensor's maximum is still held to the bar."""
    return [float(np.abs(got[:, l * l:(l + 1) ** 2, :] - ref[:, l * l:(l + 1) ** 2, :]).max() / scales[l])
            for l in range(lmax + 1)]


def rel_err_per_shell_block(got, ref, scales, orb_l):
    off = np.concatenate([[0], np.cumsum([2 * l + 1 for l in orb_l])])
    return np.array([[np.abs(got[:, off[a]:off[a + 1], off[b]:off[b + 1]] - ref[:, off[a]:off[a + 1], off[b]:off[b + 1]]).max()
                      / scales[a, b] for b in range(len(orb_l))] for a in range(len(orb_l))])


@pytest.mark.parametrize("index,cell_list", [(3, True), (3, False), (4, True), (5, True)])
def test_fullsize_edge_set_bit_exact(index, cell_list):
    """src, dst, shift and row_ptr of the full-size graphs against the brute-force oracle run live: both search
    strategies at 3,000 atoms, the cell list on the slab with its halo (13 x 5 x 5 cells, periodic in x and y)."""
    import torch
    from paper_2507_03840_amd import binding as B
    assert torch.cuda.is_available()
    print(f"config {index}, cell_list={cell_list}: oracle graph", flush=True)
    w = synth.workload(index)
    g = full_oracle_graph(index)
    m = B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, 1.0, n_layers=w.n_layers, orb_l=w.orb_l)
    graph = m.egnn_nlist(B.to_device(w.pos), w.n_owned, w.box, w.pbc, cell_list=cell_list)
    assert_same_graph(graph, g)
    assert graph.n_edges > 600000


@pytest.mark.parametrize("index,fused", [(3, False), (4, False), (3, "shared"), (4, "shared"), (3, True), (4, True),
                                         (3, 2), (4, 2)])
def test_fullsize_sampled_rows(index, fused):
    """fused: False = the default route (S3 and S4 in one kernel, S3 and S6 in one kernel), one row of weights per edge; "shared" = the
    same with one row per unordered pair of owned atoms (what bench.py times); True / 2 = the two older fused designs."""
    import torch
    assert torch.cuda.is_available()
    path = os.path.join(GOLDEN, f"config{index}_samples.npz")
    assert os.path.exists(path), "run tests/golden/make_golden.py"
    gold = np.load(path)
    print(f"config {index}: building inputs", flush=True)
    w = synth.workload(index)
    wt = U.model_weights(w)
    shared = fused == "shared"
    m, graph, xs, H = U.gpu_forward(w, wt, float(gold["agg"]), with_readout=w.readout, fused=False if shared else fused,
                                    shared_rows=shared)
    assert_same_graph(graph, full_oracle_graph(index))
    if shared:
        n_halo_src = int((graph.src >= w.n_owned).sum())
        assert graph.n_w_rows == n_halo_src + (graph.n_edges - n_halo_src) // 2
    assert graph.n_edges == int(gold["n_edges"])
    nodes = gold["nodes"]
    deg = np.diff(graph.row_ptr.cpu().numpy())
    for j in (0, w.n_owned - 1, int(np.argmin(deg)), int(np.argmax(deg))):
        assert j in nodes                      # the stored rows include the aimed ones
    for t in range(w.n_layers):
        got = xs[t][torch.from_numpy(nodes).cuda()].cpu().numpy().astype(np.float64)
        errs = rel_err_per_degree(got, gold[f"x{t + 1}_rows"], gold[f"x{t + 1}_maxabs_l"], w.lmax)
        print(f"config {index} layer {t}: sampled rel err per degree " + " ".join(f"{e:.1e}" for e in errs), flush=True)
        assert max(errs) < U.TOL
        assert abs(float(xs[t].abs().max()) / float(gold[f"x{t + 1}_maxabs"]) - 1) < 1e-3
    if w.readout:
        edges = gold["edges"]
        assert graph.n_edges - 1 in edges and 0 in edges
        got = H[torch.from_numpy(edges).cuda()].cpu().numpy().astype(np.float64)
        errs = rel_err_per_shell_block(got, gold["H_rows"], gold["H_maxabs_blocks"], w.orb_l)
        print(f"config {index} H_ij: sampled rel err, worst shell block {errs.max():.2e}", flush=True)
        assert errs.max() < U.TOL
        # and every sampled edge on its own scale: an edge near the cutoff has a small block (the envelope tends to
        # zero there), which the tensor's scale would hide.  The fp32 length of an edge is off by up to half an ulp
        # (5e-7 A at 10 A), which alone changes the envelope by 1e-6 / (r_cut - d) of its value, so blocks below 1e-3
        # of the largest are judged on that floor instead of their own size.
        own = np.abs(gold["H_rows"]).reshape(len(edges), -1).max(axis=1)
        per_edge = np.abs(got - gold["H_rows"]).reshape(len(edges), -1).max(axis=1) / \
            np.maximum(own, 1e-3 * float(gold["H_maxabs"]))
        print(f"config {index} H_ij: worst edge on its own scale {per_edge.max():.2e} "
              f"(smallest block {own.min() / float(gold['H_maxabs']):.1e} of the largest)", flush=True)
        assert per_edge.max() < U.TOL


def test_stage_timing_records_every_stage():
    import torch
    from paper_2507_03840_amd import binding as B
    w = synth.workload(1)
    wt = U.model_weights(w)
    m = B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, 20.0, orb_l=w.orb_l)
    pos = B.to_device(w.pos)
    graph = m.egnn_nlist(pos, w.n_owned, w.box, w.pbc)
    ws = m.workspace(graph)
    x = B.to_device(wt["x0"])
    m.egnn_timing_enable(3)
    for _ in range(2):
        y = m.egnn_layer_forward(graph, pos, w.box, x, B.to_device(wt["layers"][0]), ws)
    m.egnn_readout_hij(graph, pos, w.box, y, B.to_device(wt["readout"]), ws)
    m.egnn_layer_forward(graph, pos, w.box, x, B.to_device(wt["layers"][0]), ws)   # beyond max_calls: not recorded
    ms, n = m.egnn_timing_read()
    assert n == [2, 1, 0, 0] and all(v > 0 for v in ms[:10]) and sum(ms[10:]) == 0
    ms2, n2 = m.egnn_timing_read()
    assert n2 == [0, 0, 0, 0] and sum(ms2) == 0
    m.egnn_timing_enable(0)


@pytest.mark.parametrize("keep,shared", [(False, False), (True, False), (False, True), (True, True)])
def test_fullsize_training_step_config5(keep, shared):
    """Config 5: forward + MSE + reverse pass on the 3,000-atom graph; loss and every gradient against the stored
    fp64 oracle results (weight gradients in full, input-feature gradient at sampled rows)."""
    import torch
    assert torch.cuda.is_available()
    path = os.path.join(GOLDEN, "config5_training.npz")
    assert os.path.exists(path), "run tests/golden/make_golden.py 5"
    gold = np.load(path)
    w = synth.workload(5)
    wt = U.model_weights(w)
    T = synth.normal(np.random.default_rng([w.seed, 99]), (int(gold["n_edges"]), w.n_orb, w.n_orb))
    res = U.gpu_training_step(w, wt, float(gold["agg"]), T, keep=keep, shared_rows=shared)
    assert res["n_edges"] == int(gold["n_edges"])
    print(f"loss gpu {res['loss']:.8f} oracle {float(gold['loss']):.8f}", flush=True)
    assert abs(res["loss"] / float(gold["loss"]) - 1) < 1e-5
    for k, v in res["grads"].items():
        if k == "x0":
            # input-feature gradient at the stored rows, every degree on its own scale
            err = max(rel_err_per_degree(v[gold["nodes"]].astype(np.float64), gold["x0_rows"], gold["x0_maxabs_l"], w.lmax))
        elif v.ndim == 3 and v.shape[0] == w.lmax + 1:
            # per-degree channel mixes [l][E][E]: each degree's matrix on its own scale
            err = max(U.rel_err(v[l], gold[k][l]) for l in range(w.lmax + 1))
        else:
            err = U.rel_err(v, gold[k])
        print(f"config 5 grad {k}: rel err {err:.2e}", flush=True)
        assert err < U.TOL, k


@pytest.mark.parametrize("what", ["layer", "so2"])
def test_fullsize_equivariance(what):
    """A property that holds at any size: rotating the structure and the features rotates the result.  Config 3's
    structure is made non-periodic for this (a cube is not invariant under a general rotation), which keeps ~400,000
    edges; the rotation matrices of the features come from the oracle's harmonics (fp64)."""
    import torch
    from oracle import egnn_oracle as O
    from paper_2507_03840_amd import binding as B
    B.load_library()
    w = synth.workload(3, check_cutoff=False)
    w.pbc = np.zeros(3, np.uint8)
    wt = U.model_weights(w)
    rng = np.random.default_rng(99)
    q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
    Q = q * np.sign(np.linalg.det(q))
    DQ = O.wigner_d_block(w.lmax, Q)
    centre = w.pos.astype(np.float64).mean(axis=0)
    pos2 = ((w.pos.astype(np.float64) - centre) @ Q.T + centre).astype(np.float32)
    x = wt["x0"].astype(np.float64)
    x2 = np.einsum("ab,nbc->nac", DQ, x).astype(np.float32)

    def run(pos_np, x_np):
        pos = B.to_device(pos_np)
        probe = B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, 1.0)
        g = probe.egnn_nlist(pos, w.n_owned, w.box, w.pbc)
        m = B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, 150.0)
        if what == "layer":
            ws = m.workspace(g)
            y = m.egnn_layer_forward(g, pos, w.box, B.to_device(x_np), B.to_device(wt["layers"][0]), ws)
        else:
            from oracle import so2_oracle as S
            W_e, W0, Wr, Wi = synth.so2_weights(np.random.default_rng([w.seed, 777]), w.lmax, w.channels, w.n_rbf)
            ws = torch.empty(m.egnn_so2_workspace_bytes(g.n_edges), dtype=torch.uint8, device="cuda")
            y = m.egnn_so2_message_sum(g, pos, w.box, B.to_device(x_np), B.to_device(W_e), B.to_device(S.so2_pack(W0, Wr, Wi)), ws)
        return g.n_edges, y.cpu().numpy().astype(np.float64)

    n1, y1 = run(w.pos, x.astype(np.float32))
    n2, y2 = run(pos2, x2)
    # pairs within a few ulp of the cutoff can flip when the positions are rotated in fp32; their messages carry the
    # envelope f_c ~ 1e-13, so they do not show in the result
    assert abs(n1 - n2) <= 4 and n1 > 300000
    err = np.abs(y2 - np.einsum("ab,nbc->nac", DQ, y1)).max() / np.abs(y1).max()
    print(f"{what}: {n1} edges, equivariance error {err:.2e} of scale", flush=True)
    assert err < 2e-5      # positions and features of the rotated copy are rounded to fp32 once more
