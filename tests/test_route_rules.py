"""The rules that send a call to the kernels with the radial weights in registers or through a weight tensor, at the sizes where they
turn, asked of the library without a GPU.  Each line is one that measurements on both sides set; what they measured stands beside
the rules in edge_fused.hip, readout_fused.hip, tp_bins.hip and readout_adjoint.hip."""
import os

import pytest

from tests import gpu_util as U


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.load_library()
    return binding


def _layer(B, lmax, E, n_edges, n, n_total=None):
    return U.fused_route(B, B.Egnn(lmax, E, 16, 10.0, 20.0), "layer", n_edges, n, n_total or n)


@pytest.mark.parametrize("E", [32, 64])
def test_layer_lmax_1(B, E):
    """w is small at lmax 1: on many nodes or edges S3 and S4 are the faster ones as soon as the weights are kept."""
    nodes, edges = 800 * 32 // E, 46000 * 32 // E
    assert _layer(B, 1, E, 20 * nodes, nodes)
    assert not _layer(B, 1, E, 20 * nodes, nodes + 1)
    assert _layer(B, 1, E, edges, 300)
    assert not _layer(B, 1, E, edges + 1, 300)
    assert not _layer(B, 1, E, 524172, 2500) and not _layer(B, 1, 128, 3858, 200) and not _layer(B, 0, E, 3858, 200)


@pytest.mark.parametrize("lmax", [2, 3, 4])
@pytest.mark.parametrize("E", [8, 16, 32, 64, 128])
def test_layer_from_lmax_2(B, lmax, E):
    assert _layer(B, lmax, E, 524172, 2500) and _layer(B, lmax, E, 9000, 300) and _layer(B, lmax, E, 2000000, 12000, 20000)
    odd = lmax == 2 and E == 128                         # few edges on more than 300 nodes
    assert _layer(B, lmax, E, 60 * 301, 301) and _layer(B, lmax, E, 60 * 301 - 1, 301) != odd
    assert _layer(B, lmax, E, 60 * 799, 799) and _layer(B, lmax, E, 60 * 799 - 1, 799) != odd
    assert _layer(B, lmax, E, 25 * 800, 800) and _layer(B, lmax, E, 25 * 800 - 1, 800) != odd
    assert not _layer(B, lmax, E, 40, 30)                # (the scratch does not fit where w would lie)
    assert not _layer(B, lmax, E, 0, 30) and not _layer(B, lmax, E, 0, 0, 30)


SETS = {4: (0, 1), 5: (0, 0, 1), 7: (0, 1, 1), 8: (0, 0, 1, 1), 9: (0, 1, 2), 10: (0, 0, 1, 2), 12: (0, 1, 1, 2), 13: (0, 0, 1, 1, 2)}


def _readout(B, lmax, E, n_orb, n_edges):
    m = B.Egnn(lmax, E, 16, 10.0, 20.0, orb_l=SETS[n_orb])
    return U.fused_route(B, m, "readout", n_edges, 1200, 1200)


# (lmax, channels, orbitals, last or first edge count, whether it is taken there, one edge on)
@pytest.mark.parametrize("lmax,E,n_orb,n_edges,here,beyond", [
    (2, 64, 13, 149999, False, True), (4, 64, 12, 149999, False, True), (3, 64, 10, 149999, False, False), (1, 64, 9, 149999, False, True),
    (1, 64, 8, 149999, False, False), (2, 32, 8, 32768, True, False), (4, 32, 8, 32768, True, False), (4, 32, 8, 49152, False, True),
    (3, 32, 9, 49152, False, True), (3, 32, 8, 49152, False, False), (2, 32, 10, 49152, False, True), (2, 32, 9, 49152, False, False),
    (1, 32, 9, 49152, False, True), (4, 32, 12, 32768, True, False), (2, 32, 13, 32768, True, True), (4, 32, 13, 49152, True, True),
    (2, 32, 7, 20000, False, False), (2, 16, 4, 32768, True, False), (2, 16, 8, 32768, True, False), (2, 16, 9, 32768, True, True),
    (1, 16, 5, 32768, True, False), (1, 16, 8, 32768, True, True), (3, 16, 4, 32768, True, True), (4, 16, 4, 32768, True, True),
    (2, 8, 4, 32768, True, True), (4, 128, 13, 300000, False, False), (0, 32, 13, 32768, False, False)])
def test_readout(B, lmax, E, n_orb, n_edges, here, beyond):
    assert _readout(B, lmax, E, n_orb, n_edges) == here and _readout(B, lmax, E, n_orb, n_edges + 1) == beyond


@pytest.mark.parametrize("orb", [(0, 0, 0, 1, 1, 2), (0, 1, 2, 2), (0, 0, 1, 1, 1), (2, 2, 1)])
def test_readout_rows_of_v(B, orb):
    """Sets with more rows of V in a degree than the kernel has room for: the two kernels."""
    assert not U.fused_route(B, B.Egnn(3, 32, 16, 10.0, 20.0, orb_l=orb), "readout", 300000, 1200, 1200)


@pytest.mark.parametrize("lmax,E,first", [(1, 8, 12000), (2, 16, 12000), (3, 32, 12000), (4, 128, 12000), (3, 16, 30000), (4, 16, 30000),
                                          (3, 8, 60000), (4, 8, 60000)])
def test_weight_gradient_summed_as_it_is_made(B, lmax, E, first):
    m = B.Egnn(lmax, E, 16, 10.0, 20.0)
    assert U.tp_bins_route(m, first) and not U.tp_bins_route(m, first - 1)
    assert not U.tp_bins_route(B.Egnn(0, E, 16, 10.0, 20.0), 1000000)


@pytest.mark.parametrize("lmax,E,orb,first", [
    (1, 64, (0, 0, 1, 1, 2), 12000), (2, 32, (0, 0, 1, 1, 2), 12000), (3, 16, (0, 1, 1, 2), 12000), (4, 128, (0, 1, 1, 2), 12000),
    (4, 64, (0, 1), 12000), (4, 32, (0, 1), 40000), (4, 16, (0, 1, 2), 40000), (3, 128, (0, 1), 18000), (3, 64, (0, 0, 1, 1), 18000),
    (3, 32, (0, 1, 2), 40000), (3, 16, (0, 1), 40000)])
def test_readout_adjoint(B, lmax, E, orb, first):
    m = B.Egnn(lmax, E, 16, 10.0, 20.0, orb_l=orb)
    assert U.readout_adjoint_route(m, first) and not U.readout_adjoint_route(m, first - 1)


@pytest.mark.parametrize("lmax,E,orb", [(0, 32, (0, 0, 1, 1, 2)), (4, 8, (0, 0, 1, 1, 2)), (1, 32, (0, 0, 1, 1, 2)), (2, 16, (0, 0, 1, 1, 2)),
                                        (2, 64, (0, 1, 2)), (3, 64, (0, 1)), (3, 32, (0, 1)), (4, 64, (0, 0, 0, 1, 1, 1)), (4, 32, (0, 0, 0, 1, 1, 1, 2, 2))])
def test_readout_adjoint_never(B, lmax, E, orb):
    """Too few channels, no room for its own gradients of the collapsed values, few orbitals, more rows of V than there is room for."""
    assert not U.readout_adjoint_route(B.Egnn(lmax, E, 16, 10.0, 20.0, orb_l=orb), 1000000)
