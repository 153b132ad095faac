"""CPU-side checks of the C ABI library: it loads, exports every declared symbol, and its host logic
(path tables, readout widths, workspace sizes, argument checks) agrees with the oracle's definitions."""
import ctypes
import os
import re
import numpy as np
import pytest

from oracle import egnn_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def B():
    from paper_2507_03840_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.load_library()
    return binding


def test_every_declared_symbol_is_exported(B):
    header = open(os.path.join(ROOT, "include", "egnn.h")).read()
    declared = set(re.findall(r"\b(egnn_[a-z_0-9]+)\s*\(", header))
    declared -= {"egnn_workspace_bytes(...)"}
    assert declared == set(B.SYMBOLS), declared ^ set(B.SYMBOLS)
    lib = ctypes.CDLL(B.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name


def test_no_callback_that_allocates(B):
    """std::function may allocate, and throw through a C entry."""
    assert b"bad_function_call" not in open(B.LIB_PATH, "rb").read()


@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 4])
def test_path_tables_match_definition(B, lmax):
    m = B.Egnn(lmax, 32, 16, 8.0, 50.0)
    assert m.paths == O.tp_paths(lmax, lmax, lmax)
    assert m.paths_readout == O.tp_paths(lmax, lmax, 4)
    assert m.n_out == O.readout_slots((0, 0, 1, 1, 2))[1]
    m2 = B.Egnn(lmax, 8, 4, 8.0, 50.0, orb_l=(0, 1, 2, 2))
    assert m2.n_out == O.readout_slots((0, 1, 2, 2))[1]


def test_create_rejects_bad_descriptors(B):
    for kw in [dict(lmax=5), dict(channels=24), dict(n_rbf=1), dict(n_rbf=33), dict(r_cut=0.0), dict(agg_norm=-1.0),
               dict(orb_l=(0, 3)), dict(lmax_sh=2), dict(n_radial_hidden=32)]:
        args = dict(lmax=3, channels=32, n_rbf=16, r_cut=8.0, agg_norm=10.0)
        args.update(kw)
        with pytest.raises(B.EgnnError) as e:
            B.Egnn(**args)
        assert e.value.code == -1, kw


def test_transpose_asks_for_one_word_per_edge(B):
    """Nothing but the buckets lies in the workspace: whatever the number of atoms, a word per edge is not too small (EGNN_EWS), a byte less is."""
    m = B.Egnn(1, 8, 8, 4.0, 1.0)
    at, n_edges = ctypes.c_void_p(4096), 640
    g = B.GraphDesc(4096, 4096, 4096, None, n_edges, 100, 50000, None, 0, None, None)
    call = lambda n: m.lib.egnn_graph_transpose(m.ctx, ctypes.byref(g), at, at, at, ctypes.c_size_t(n), None)
    if not os.path.exists("/dev/kfd"):                      # (without a GPU nothing is launched)
        assert call(4 * n_edges) != -3
    assert call(4 * n_edges - 1) == -3


def test_workspace_bytes_cover_every_buffer(B):
    m = B.Egnn(4, 32, 16, 10.0, 200.0)
    n_e, n_o, n_t = 625_000, 3000, 3000
    need = n_e * 16 + n_t * 25 * 32 * 4 + n_o * 25 * 32 * 4 + n_e * 42 * 32 * 4
    got = m.egnn_workspace_bytes(n_e, n_o, n_t, True)
    assert need <= got <= need * 1.01 + 4096
    assert m.egnn_workspace_bytes(n_e, n_o, n_t, False) >= n_e * 16 + 2 * n_t * 25 * 32 * 4
    assert m.egnn_workspace_bytes(0, 0, 0, True) >= 0
