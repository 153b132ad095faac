"""The loss over whole and part vectors, aligned and not, and columns whose own block falls anywhere among more than 64
sources, against the oracle.  Loss terms: sums in double of float differences, compared at a few float roundings."""
import numpy as np
import pytest

from oracle import hamiltonian_oracle as Hm
from paper_2507_03840_amd import synth
from tests import gpu_util as U
from tests.test_gpu_hamiltonian import SHELLS3, _blocks_case, _dev_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    return binding


@pytest.mark.parametrize("orb_l,shells", [([0, 0, 1, 1, 2], SHELLS3), ([0, 1], [[0, 1], [0], [1]]), ([0, 0, 0], [[0, 1], [2]])])
@pytest.mark.parametrize("n", [1, 3, 97, 1001])
@pytest.mark.parametrize("off_h,off_t", [(0, 0), (1, 0), (0, 2), (4, 4)])
def test_loss_vectors(B, orb_l, shells, n, off_h, off_t):
    import torch
    rng = np.random.default_rng([n, off_h, len(orb_l)])
    n_orb = sum(2 * l + 1 for l in orb_l)
    species = rng.integers(0, len(shells), 50).astype(np.int32)
    bits = Hm.species_orbital_bits(orb_l, shells)
    rows, cols = (rng.integers(0, 50, n).astype(np.int32) for _ in range(2))
    H, T = (synth.normal(rng, (n, n_orb, n_orb)).astype(np.float32) for _ in range(2))

    def at(x, off):
        buf = torch.empty(x.size + off, dtype=torch.float32, device="cuda")
        v = buf[off:].view(x.shape)
        v.copy_(B.to_device(x))
        return v

    m = B.Egnn(1, 8, 4, 3.0, 1.0, orb_l=orb_l)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    sp_d, bits_d, ra, ca = B.to_device(species), _dev_bits(B, bits), B.to_device(rows), B.to_device(cols)
    loss, dH = m.egnn_loss_l1l2(at(H, off_h), at(T, off_t), ra, ca, sp_d, bits_d, ws)
    ref_loss, ref_g = Hm.loss_l1l2(H, T, bits[species[rows]], bits[species[cols]])
    assert abs(float(loss[0]) - ref_loss) <= 1e-6 * max(ref_loss, 1e-30)
    assert U.rel_err(dH.cpu().numpy(), ref_g) < 1e-6
    only, none = m.egnn_loss_l1l2(at(H, off_h), at(T, off_t), ra, ca, sp_d, bits_d, ws, want_grad=False)
    assert none is None and torch.equal(only, loss)


def test_own_block_anywhere(B):
    w, g, species, bits, H_edge, H_node, m, gd = _blocks_case(B, 150, 150, False, 9, SHELLS3, 12.0)
    assert np.median(np.diff(g[3])) > 96          # most columns hold more than 64 sources on one side or both
    sp_d, bits_d = B.to_device(species), _dev_bits(B, bits)
    ws, plan = m.hamiltonian_workspace(gd)
    orb_off, col_ptr, nnz = m.egnn_hamiltonian_structure(gd, sp_d, bits_d, plan)
    row_idx, values = m.egnn_hamiltonian_fill(gd, sp_d, bits_d, orb_off, plan, B.to_device(H_edge), B.to_device(H_node), nnz)
    r_off, r_ptr, r_rows, r_vals = Hm.assemble_csc(g, species, bits, H_edge, H_node, 150, 150)
    assert np.array_equal(orb_off.cpu().numpy(), r_off) and np.array_equal(col_ptr.cpu().numpy(), r_ptr)
    assert np.array_equal(row_idx.cpu().numpy(), r_rows)
    assert np.array_equal(values.cpu().numpy().astype(np.float64), r_vals)
