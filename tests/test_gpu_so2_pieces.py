"""GPU test of the half-precision pieces of the per-edge SO(2) products: with one non-zero product per result every value comes out to the 22
bits of its pieces, at halfway cases of half precision and far below the largest value too."""
import numpy as np
import pytest

from oracle import so2_oracle as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


def _values(rng, shape):
    """Largest below 2, so that the pieces are those of 2^13 times the value: ordinary values, halfway between two neighbouring halves, and
    down to 2^-18 of the largest."""
    h = rng.integers(0x3000, 0x7000, shape).astype(np.uint16)                   # 2^-3 .. 2^13
    ties = 0.5 * (h.view(np.float16).astype(np.float64) + (h + 1).astype(np.uint16).view(np.float16).astype(np.float64)) / 2.0 ** 13
    ties *= 1.0 + 2.0 ** -23 * rng.integers(-1, 2, shape)
    ordinary = rng.uniform(0.5, 1.9, shape)
    small = 2.0 ** rng.uniform(-18, 0, shape)
    kind = rng.integers(0, 3, shape)
    return (rng.choice([-1.0, 1.0], shape) * np.choose(kind, [ordinary, ties, small])).astype(np.float32)


def test_pieces(B):
    import torch
    E, n, n_rbf, r_cut = 32, 96, 6, 20.0
    rng = np.random.default_rng(3)
    pos = np.stack([1.3 * np.arange(n), 0.1 * rng.random(n), 0.1 * rng.random(n)], 1).astype(np.float32)
    box = np.array([400.0] * 3, np.float32)
    dst = np.arange(n - 1, dtype=np.int32)                                      # a chain: every node but the last hears its neighbour
    src = dst + 1
    row_ptr = np.minimum(np.arange(n + 1), n - 1).astype(np.int32)
    shift = np.zeros((n - 1, 3), np.int8)
    g = (src, dst, shift, row_ptr)
    x = _values(rng, (n, 1, E))
    x[5, 0, 3] = 1.9375
    W0 = np.zeros((E, 3 * E), np.float32)
    W0[np.arange(E), rng.permutation(E)] = 1.0                                  # the source's channels in another order
    W_e = np.zeros((E, n_rbf), np.float32)
    m = B.Egnn(0, E, n_rbf, r_cut, 1.0)
    graph = B.Graph(B.to_device(src), B.to_device(dst), B.to_device(row_ptr), B.to_device(shift), n, n)
    nbytes = max(m.egnn_so2_workspace_bytes(n - 1), m.egnn_so2_backward_workspace_bytes(n - 1, n), m.egnn_backward_workspace_bytes(n - 1, n, n))
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    dev = lambda *a: [B.to_device(v) for v in a]
    pos_d, x_d, We_d, W_d = dev(pos, x, W_e, W0.ravel())

    # pieces of 22 bits (2^-23 of the value, 2^-25 of the unit where the low one is subnormal); the envelope and the products 2^-22 more
    quantum = 2.0 ** -24 / 2.0 ** 13
    a = m.egnn_so2_message_sum(graph, pos_d, box, x_d, We_d, W_d, ws).cpu().numpy()
    ref = S.so2_message_sum(g, pos, box, x, W_e, W0, [], [], 0, E, n_rbf, r_cut, 1.0)
    over = (np.abs(a - ref) - quantum) / np.maximum(np.abs(ref), 1e-30)
    print(f"sum: {over.max():.2e}", flush=True)
    assert over.max() < 2.0 ** -21

    # the weights' gradient of a single edge: products of two values in pieces
    col_ptr, perm = m.egnn_graph_transpose(graph, ws)
    da = np.zeros((n, 1, E), np.float32)
    da[7] = _values(rng, (1, E))
    da[7, 0, 0] = 1.9375
    dx, _, dW = m.egnn_so2_message_sum_backward(graph, col_ptr, perm, pos_d, box, x_d, We_d, W_d, B.to_device(da), ws)
    ref = S.so2_message_sum_backward(g, pos, box, x, W_e, W0, [], [], 0, E, n_rbf, r_cut, 1.0, da)
    got = dW.cpu().numpy().reshape(E, 3 * E)
    over = (np.abs(got - ref[2]) - 4.0 * quantum) / np.maximum(np.abs(ref[2]), 1e-30)
    print(f"weights: {over.max():.2e}", flush=True)
    assert over.max() < 2.0 ** -20 and np.count_nonzero(ref[2]) > E * E
    over = (np.abs(dx.cpu().numpy() - ref[0]) - quantum) / np.maximum(np.abs(ref[0]), 1e-30)
    print(f"features: {over.max():.2e}", flush=True)
    assert over.max() < 2.0 ** -21
