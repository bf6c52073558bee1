"""The C-ABI library loads on a machine without a GPU and exports every symbol include/obc.h declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "obc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(obc_[a-z0-9_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    from paper_2208_11580_amd import binding

    if not os.path.exists(binding.LIB_PATH):
        from paper_2208_11580_amd import build

        build.build_lib()
    return binding.load_library()


def test_header_declares_the_boundary():
    syms = _declared_symbols()
    for name in ("obc_hessian", "obc_invert", "obc_prune_rows", "obc_quant_rows", "obc_global_select"):
        assert name in syms


def test_library_exports_every_declared_symbol(lib):
    from paper_2208_11580_amd import binding

    syms = _declared_symbols()
    assert sorted(binding.EXPORTS) == syms
    for name in syms:
        assert hasattr(lib, name), name


def test_small_rows_hold_no_bulk_elimination(lib):
    """Up to 192 columns a row's workspace is two matrices, 128 vectors and its state, without the two 64 x 64
    fp64 blocks of the bulk elimination."""
    n = ctypes.c_size_t()
    for R, d in ((1000, 65), (1000, 100), (1, 192), (5000, 192)):
        assert lib.obc_rows_workspace_bytes(R, d, 2, ctypes.byref(n)) == 0
        assert n.value <= R * (2 * 4 * (d * d + 3) + 128 * 4 * (d + 4) + 25 * d + 32) + 20 * 256, (R, d)


def test_second_moment_workspaces_serve_smaller_batches(lib):
    """Calibration data arrives in batches, the last one ragged: what is enough for N samples is enough for
    fewer."""
    n = ctypes.c_size_t()
    for d in (16, 64, 200, 576, 768, 1283, 2304, 3072, 4608):
        most = 0
        for N in list(range(1, 3000, 7)) + list(range(3000, 60000, 233)) + [10 ** 6, 10 ** 7]:
            assert lib.obc_hessian_workspace_bytes(d, N, ctypes.byref(n)) == 0
            assert n.value >= most, (d, N)
            most = n.value
        assert most <= 64 * d * d * 4 + 256
    for d_row, d_col in ((1, 64), (16, 576), (256, 2304)):
        most = 0
        for N in range(1, 60000, 97):
            assert lib.obc_cross_workspace_bytes(d_row, d_col, N, ctypes.byref(n)) == 0
            assert n.value >= most, (d_row, d_col, N)
            most = n.value


def test_host_only_calls(lib):
    assert b"gfx950" in lib.obc_version()
    n = ctypes.c_size_t()
    assert lib.obc_rows_workspace_bytes(256, 2304, 1, ctypes.byref(n)) == 0
    assert n.value >= 256 * 2304 * 2304 * 4
    assert lib.obc_rows_workspace_bytes(16, 32, 0, ctypes.byref(n)) == 0 and n.value <= 4096
    assert lib.obc_rows_workspace_bytes(-1, 32, 0, ctypes.byref(n)) == -1
    assert lib.obc_rows_workspace_bytes(1, 32, 7, ctypes.byref(n)) == -1
    assert lib.obc_invert_workspace_bytes(0, ctypes.byref(n)) == -1
    assert lib.obc_invert_workspace_bytes(100, ctypes.byref(n)) == 0 and n.value >= 2 * 100 * 100 * 8
    assert lib.obc_hessian_workspace_bytes(576, 50000, ctypes.byref(n)) == 0 and n.value >= 576 * 576 * 4
    assert lib.obc_global_select_workspace_bytes(64, 576, ctypes.byref(n)) == 0 and n.value >= 64 * 576 * 4
    assert lib.obc_last_error(None) == b"null context"
    # widened entry points
    assert lib.obc_cross_workspace_bytes(256, 2304, 50000, ctypes.byref(n)) == 0 and n.value >= 256 * 2304 * 4
    assert lib.obc_cross_workspace_bytes(0, 2304, 50000, ctypes.byref(n)) == -1
    m = ctypes.c_size_t()
    assert lib.obc_invert_workspace_bytes(576, ctypes.byref(m)) == 0
    assert lib.obc_refit_workspace_bytes(576, 64, ctypes.byref(n)) == 0 and n.value >= m.value + 2 * 64 * 576 * 8
    assert lib.obc_refit_workspace_bytes(576, 0, ctypes.byref(n)) == -1
    # block pruning: blocks of 4 go to the deferred-update solver, other sizes to the rank-1 solver,
    # which cannot be forced to take what it does not do
    r1, rb = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.obc_rows_workspace_bytes(8, 576, 1, ctypes.byref(r1)) == 0
    assert lib.obc_rows_workspace_bytes(8, 576, 2, ctypes.byref(rb)) == 0
    assert lib.obc_blocks_workspace_bytes(8, 576, 4, 0, ctypes.byref(n)) == 0 and n.value == rb.value
    assert lib.obc_blocks_workspace_bytes(8, 576, 2, 0, ctypes.byref(n)) == 0 and n.value == r1.value
    assert lib.obc_blocks_workspace_bytes(8, 576, 2, 2, ctypes.byref(n)) == -1
    assert lib.obc_blocks_workspace_bytes(8, 576, 9, 0, ctypes.byref(n)) == -1


def test_binding_constants_match_the_header():
    from paper_2208_11580_amd import binding

    text = open(os.path.join(ROOT, "include", "obc.h")).read()
    defs = dict(re.findall(r"#define\s+(OBC_[A-Z0-9_]+)\s+\(?(-?\d+)\)?", text))
    assert int(defs["OBC_SELECT_STATIC_MAX_WEIGHTS"]) == binding.SELECT_STATIC_MAX_WEIGHTS
    assert int(defs["OBC_SELECT_STATIC_MAX_ROWS"]) == binding.SELECT_STATIC_MAX_ROWS
    for name in ("OBC_ERR_BAD_ARG", "OBC_ERR_BAD_SHAPE", "OBC_ERR_NOT_SPD", "OBC_ERR_WORKSPACE", "OBC_ERR_NUMERIC",
                 "OBC_ERR_HIP"):
        assert int(defs[name]) == getattr(binding, name)


def test_no_oracle_in_product_path():
    """The package never imports the oracle (the oracle is test infrastructure)."""
    pkg = os.path.join(ROOT, "paper_2208_11580_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), (dirpath, f)
