"""Radial weights at row counts and widths where the column blocks are shared out differently over the workgroups."""
import numpy as np
import pytest

from oracle import egnn_oracle as O
from tests import gpu_util as U
from tests.test_gpu_w_fp16 import unpack_w16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    binding.load_library()
    return binding


# rows: one, a workgroup's 448 and one more, just under and over half of the 256 workgroups the chip holds; columns: a part of a
# block, one block, an odd and an even number, the widest row
@pytest.mark.parametrize("lmax,E,n", [(0, 8, 1), (0, 32, 449), (1, 16, 448), (2, 16, 1387), (3, 32, 3000), (4, 128, 65), (4, 32, 448 * 127),
                                      (2, 32, 448 * 129 + 5), (1, 8, 448 * 256 + 1)])
def test_radial_weights_shared_out(B, lmax, E, n):
    n_rbf, r_cut = 7, 5.0
    rng = np.random.default_rng(n)
    m = B.Egnn(lmax, E, n_rbf, r_cut, 1.0)
    d = (rng.random(n) * 5.0).astype(np.float32)
    rd = np.concatenate([np.zeros((n, 3), np.float32), d[:, None]], 1)
    W1 = (rng.standard_normal((64, n_rbf)) * n_rbf ** -0.5).astype(np.float32)
    W2 = (rng.standard_normal((m.n_paths * E, 64)) * 0.125).astype(np.float32)
    print("case", lmax, E, n, flush=True)
    args = (0, B.to_device(rd), B.to_device(W1), B.to_device(W2))
    w = m.egnn_radial_weights(*args).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(n, 70)), rng.integers(0, n, 200), np.arange(max(0, n - 70), n)]))
    ref = O.radial_weights(d[rows].astype(np.float64), W1, W2, m.paths, E, n_rbf, r_cut)
    assert U.rel_err(w[rows], ref) < 2e-6          # operands of 22 bits, 64 products and 7 Gaussians in 32 bits
    half = unpack_w16(m.egnn_radial_weights_f16(*args).cpu().numpy(), m.n_paths * E).reshape(w.shape)
    assert np.array_equal(half, w.astype(np.float16).astype(np.float64))
