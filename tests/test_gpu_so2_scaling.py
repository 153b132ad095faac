"""SO(2) calls on operands of very different size: what is small beside something else that does not enter it keeps its
accuracy, and what no edge reads has no influence.  Every case has enough edges a node to mix its channels per node."""
import numpy as np
import pytest

from oracle import so2_oracle as S
from paper_2507_03840_amd import synth
from tests import gpu_util as U
from tests.test_gpu_so2_backward import check, unpack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def dense(lmax, E, n, n_owned, n_rbf, seed):
    """Every atom within the cutoff of every other."""
    w = synth.small_cluster(n, n_owned, lmax, E, n_rbf, 40.0, seed)
    rng = np.random.default_rng([n, lmax, E, seed])
    x = synth.node_features(rng, n, lmax, E)
    da = rng.standard_normal((n_owned, (lmax + 1) ** 2, E)).astype(np.float32)
    return w, x, da, synth.so2_weights(rng, lmax, E, n_rbf)


def times(weights, we, ws):
    W_e, W0, Wr, Wi = weights
    f = lambda v, s: (v * np.float32(s)).astype(np.float32)
    return f(W_e, we), f(W0, ws), [f(v, ws) for v in Wr], [f(v, ws) for v in Wi]


class Call:
    """The calls on one structure; the workspace holds garbage before each."""

    def __init__(self, B, w, agg=7.0):
        import torch
        self.B, self.w, self.m = B, w, B.Egnn(w.lmax, w.channels, w.n_rbf, w.r_cut, agg)
        self.pos = B.to_device(w.pos)
        self.graph = g = self.m.egnn_nlist(self.pos, w.n_owned, w.box, w.pbc)
        n = max(self.m.egnn_so2_backward_workspace_bytes(g.n_edges, g.n_owned), self.m.egnn_so2_blocks_workspace_bytes(g.n_edges),
                self.m.egnn_backward_workspace_bytes(g.n_edges, g.n_owned, g.n_total))
        self.ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        self.col_ptr, self.perm = self.m.egnn_graph_transpose(g, self.ws)

    def run(self, name, *args):
        self.ws.fill_(0xFF)
        return getattr(self.m, name)(*args, self.ws)

    def forward(self, x, weights):
        d = self.B.to_device
        return self.run("egnn_so2_message_sum", self.graph, self.pos, self.w.box, d(x), d(weights[0]), d(S.so2_pack(*weights[1:]))).cpu().numpy()

    def backward(self, x, weights, da):
        d = self.B.to_device
        out = self.run("egnn_so2_message_sum_backward", self.graph, self.col_ptr, self.perm, self.pos, self.w.box, d(x),
                       d(weights[0]), d(S.so2_pack(*weights[1:])), d(da))
        return [o.cpu().numpy() for o in out]

    def node_block(self, x, T, weights, w_att):
        d = self.B.to_device
        return self.run("egnn_so2_node_block", self.graph, self.pos, self.w.box, d(x), d(T), d(S.so2_pack(*weights[1:])), d(w_att)).cpu().numpy()


def named(out, lmax, E):
    g0, gr, gi = unpack(out[2], lmax, E)
    d = dict(dx=out[0], dW_e=out[1], dW0=g0)
    for i in range(lmax):
        d[f"dWr{i + 1}"], d[f"dWi{i + 1}"] = gr[i], gi[i]
    return d


# Features and the basis of the edge lengths grow or shrink together, as in test_so2_operand_scales (whose graphs have too few
# edges a node for this route), and one without the other.  Bound: as there.
@pytest.mark.parametrize("lmax,E,n,n_rbf", [(3, 16, 61, 6), (4, 32, 52, 16)])
@pytest.mark.parametrize("x_scale,we_scale,w_scale,da_scale", [
    (1e-7, 1e-7, 1e5, 1.0), (3e4, 3e4, 2e-6, 1e-9), (1e-12, 1e-12, 1e-9, 1e6), (5e8, 5e8, 40.0, 1e4), (1e-7, 1.0, 1.0, 1.0), (1.0, 1e-7, 1.0, 1.0)])
def test_operand_scales(B, lmax, E, n, n_rbf, x_scale, we_scale, w_scale, da_scale):
    print("case", lmax, E, n, x_scale, we_scale, w_scale, da_scale, flush=True)
    w, x, da, weights = dense(lmax, E, n, n - 4, n_rbf, 11)
    x, da = x * np.float32(x_scale), da * np.float32(da_scale)
    weights = times(weights, we_scale, w_scale)
    g = U.oracle_graph(w)
    c = Call(B, w)
    e = U.rel_err(c.forward(x, weights), S.so2_message_sum(g, w.pos, w.box, x, *weights, lmax, E, n_rbf, w.r_cut, 7.0))
    ref = S.so2_message_sum_backward(g, w.pos, w.box, x, *weights, lmax, E, n_rbf, w.r_cut, 7.0, da)
    want = dict(dx=ref[0], dW_e=ref[1], dW0=ref[2])
    for i in range(lmax):
        want[f"dWr{i + 1}"], want[f"dWi{i + 1}"] = ref[3][i], ref[4][i]
    got = named(c.backward(x, weights, da), lmax, E)
    eb = {k: float(np.abs(got[k].astype(np.float64) - want[k]).max() / np.abs(want[k]).max()) for k in want}
    print(f"  forward {e:.2e}, adjoint " + " ".join(f"{k} {v:.1e}" for k, v in eb.items()), flush=True)
    assert e < 1e-5
    check(got, want, 1e-5)


def with_loose_atoms(lmax, E, n, n_owned, n_rbf):
    """The dense structure with an owned atom and a halo atom beyond every cutoff."""
    w, x, da, weights = dense(lmax, E, n, n_owned, n_rbf, 12)
    far = np.array([[400.0, 0.0, 0.0]], np.float32)
    w.pos = np.concatenate([w.pos[:n_owned], far, w.pos[n_owned:], -far]).astype(np.float32)
    w.n_owned, w.n_total = n_owned + 1, n + 2
    row = np.zeros((1,) + x.shape[1:], np.float32)
    return w, np.concatenate([x[:n_owned], row, x[n_owned:], row]), np.concatenate([da, row]), weights, [n_owned, n + 1]


@pytest.mark.parametrize("lmax,E,n,n_owned", [(2, 16, 60, 50), (4, 32, 64, 60), (1, 64, 50, 45)])
@pytest.mark.parametrize("value", [1e30, float("inf"), float("nan")])
def test_rows_that_no_edge_reads(B, lmax, E, n, n_owned, value):
    """Features and gradients of atoms without neighbours: the results are those with zeros there, bit for bit."""
    print("case", lmax, E, n, n_owned, value, flush=True)
    w, x, da, weights, loose = with_loose_atoms(lmax, E, n, n_owned, 8)
    c = Call(B, w)
    n_edges = c.graph.n_edges
    assert n_edges == n_owned * (n - 1)
    T = np.random.default_rng(3).standard_normal((n_edges, (lmax + 1) ** 2, E)).astype(np.float32)
    w_att = synth.normal(np.random.default_rng(4), (E,)).astype(np.float32)
    x2, da2 = x.copy(), da.copy()
    x2[loose], da2[loose[0]] = value, value
    a, a2 = c.forward(x, weights), c.forward(x2, weights)
    b, b2 = c.node_block(x, T, weights, w_att), c.node_block(x2, T, weights, w_att)
    d, d2 = c.backward(x, weights, da), c.backward(x2, weights, da2)
    assert np.abs(a[:n_owned]).max() > 0 and not np.any(a[n_owned]) and not np.any(b[n_owned])
    for name, p, q in [("a", a, a2), ("node block", b, b2), ("dx", d[0], d2[0]), ("dW_e", d[1], d2[1]), ("dW", d[2], d2[2])]:
        assert np.array_equal(p, q), name


@pytest.mark.parametrize("lmax,E", [(4, 32), (2, 64)])
def test_rows_of_nodes_at_the_cutoff(B, lmax, E):
    """A node whose single neighbour lies just inside the cutoff (on an axis, so that its distance is a 32-bit number and the
    envelope exact to its last bits): a sum 1e-9 of the others' keeps its accuracy, a few roundings of 32 bits, and with a
    gradient as much larger it counts as much as the others in the weight gradients."""
    print("case", lmax, E, flush=True)
    w, x, da, weights = dense(lmax, E, 60, 50, 8, 13)
    w.pos -= w.pos[0]
    w.pos[1:] *= np.float32(0.25)
    w.pos[:, 0] = -np.abs(w.pos[:, 0])
    w.pos[1:, 0] -= np.float32(1.0)                                     # atom 0 is the one with the largest x
    w.pos = np.concatenate([[[w.r_cut - 3e-3, 0.0, 0.0]], w.pos]).astype(np.float32)    # the node at the cutoff comes first
    w.n_owned, w.n_total = w.n_owned + 1, w.n_total + 1
    x, da = np.concatenate([x[:1], x]), np.concatenate([da[:1] * np.float32(2e9), da])
    g = U.oracle_graph(w)
    assert np.sum(g[1] == 0) == 1
    c = Call(B, w)
    got, ref = c.forward(x, weights), S.so2_message_sum(g, w.pos, w.box, x, *weights, lmax, E, 8, w.r_cut, 7.0)
    size, e, rest = np.abs(ref[0]).max() / np.abs(ref).max(), U.rel_err(got[0], ref[0]), U.rel_err(got[1:], ref[1:])
    back, want = c.backward(x, weights, da), S.so2_message_sum_backward(g, w.pos, w.box, x, *weights, lmax, E, 8, w.r_cut, 7.0, da)
    want = dict(dx=want[0], dW_e=want[1], dW0=want[2], **{f"dWr{i + 1}": v for i, v in enumerate(want[3])},
                **{f"dWi{i + 1}": v for i, v in enumerate(want[4])})
    print(f"  row {size:.1e} of the largest: error {e:.1e}, other rows {rest:.1e}", flush=True)
    assert 1e-10 < size < 1e-8 and e < 2e-6 and rest < 2e-6
    print(f"  adjoint {check(named(back, lmax, E), want, 5e-6):.1e}", flush=True)


@pytest.mark.parametrize("lmax,E,n,n_owned,bound", [(4, 32, 210, 24, 2.2e-7), (4, 64, 48, 40, 2.5e-7)])
def test_running_sums(B, lmax, E, n, n_owned, bound):
    """The channel mixing adds a quarter of 1,632 (64 channels: 3,264) columns in a row, four columns to a rounding.  A sum that
    grows from zero and is rounded to 24 bits r times is off by about 2^-24 sqrt(r / 24) of its end value.  Correction products
    in the same sum would make that 2.1e-7 (3.0e-7); in a sum of their own, and the rest in two, it is 0.9e-7 (1.2e-7).  The
    sums over the edges add 1.5e-7 (0.7e-7), and everything else about 1e-7: 2.0e-7 (1.8e-7) against 2.8e-7 (3.3e-7)."""
    print("case", lmax, E, n, flush=True)
    w, x, da, weights = dense(lmax, E, n, n_owned, 8, 14)
    g = U.oracle_graph(w)
    ref = S.so2_message_sum(g, w.pos, w.box, x, *weights, lmax, E, 8, w.r_cut, 7.0)
    e = np.linalg.norm(Call(B, w).forward(x, weights) - ref) / np.linalg.norm(ref)
    print(f"  2-norm error {e:.2e}", flush=True)
    assert e < bound
