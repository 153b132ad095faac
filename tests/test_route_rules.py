"""The rules that send a call to the kernels with the radial weights in registers or through a weight tensor, at the sizes where they
turn, asked of the library without a GPU.  Each line is one that measurements on both sides set; what they measured stands beside
the rules in edge_fused.hip and readout_fused.hip."""
import pytest

from tests import gpu_util as U


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
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
    assert _layer(B, lmax, E, 524172, 2500) and _layer(B, lmax, E, 12560, 300) and _layer(B, lmax, E, 2000000, 12000, 20000)
    assert not _layer(B, lmax, E, 40, 30)                # (the scratch does not fit where w would lie)
    assert not _layer(B, lmax, E, 0, 30) and not _layer(B, lmax, E, 0, 0, 30)
