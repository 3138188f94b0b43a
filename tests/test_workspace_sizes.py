"""Workspace sizes without a GPU (the queries do not read the matrix): nothing is asked for launches that the options
or the shape rule out.  The constants are the requirements of one launch per step, by the sizes of their buffers."""
import ctypes

import pytest

import paper_2603_02207_amd as ld
from paper_2603_02207_amd import _native as nat

BIG = 10_000_000


def size(n, nnz, degree, n_matvec, grad=0, adaptive=False, dtype=nat.LD_F32, **options):
    c = nat.LdCsr()
    c.n, c.nnz, c.row_ptr, c.col_idx, c.val, c.dtype = n, nnz, 256, 256, 256, dtype
    o, b = ld.Options(**options).to_c(), ctypes.c_size_t(0)
    lib = nat.load()
    if adaptive:
        nat.check(lib.ld_adaptive_workspace_size(ctypes.byref(c), degree, n_matvec, ctypes.byref(o), ctypes.byref(b)), "size")
    else:
        nat.check(lib.ld_workspace_size(ctypes.byref(c), degree, n_matvec, grad, ctypes.byref(o), ctypes.byref(b)), "size")
    return b.value


def up(x):
    return -(-x // 256) * 256


def preparation(n, elem, csr_only=False):
    """ld_apply_log's workspace besides its blocks, at most: row list, counts, diagonal storage, info."""
    return up(4 * n) + up(4 * (n // 256 + 4)) + (0 if csr_only else up(9 * n * elem) + up(2 * n)) + 3 * 256


@pytest.mark.parametrize("cols,degree,options", [
    (16, 12, {}),                      # whole vectors, too many entries for a stencil
    (17, 3, {}),                       # padded copies do not pay for three steps
    (17, 12, {"block_cols": 4}),       # the caller's blocks keep V's own rows
])
def test_apply_asks_for_two_blocks(cols, degree, options):
    n = 1 << 20
    assert size(n, 15 * n, degree, -cols, **options) <= 2 * up(4 * n * cols) + preparation(n, 4)


def test_apply_stencil_options():
    n = 1 << 20
    plain = 2 * up(4 * n * 16)
    assert size(n, 5 * n, 12, -16) > plain + preparation(n, 4)   # three packed blocks
    assert size(n, 5 * n, 12, -16, tile_order=1) <= plain + preparation(n, 4)
    assert size(n, 5 * n, 12, -16, csr_only=1) <= plain + preparation(n, 4, csr_only=True)


@pytest.mark.parametrize("options", [{"tile_order": 1}, {"tile_order": 2}, {"csr_only": 1}])
def test_adaptive_asks_for_no_chunks_that_the_options_rule_out(options):
    chunk = up(4 * BIG * 20)
    assert size(BIG, 5 * BIG - 6, 12, -17, grad=1, **options) <= size(BIG, 5 * BIG - 6, 12, -17, grad=1) - 4 * chunk
    assert size(1 << 22, 5 << 22, 100, 32, adaptive=True, **options) < size(1 << 22, 5 << 22, 100, 32, adaptive=True)


def test_more_entries_than_a_stencil_ask_for_no_chunks():
    assert size(BIG, 5 * BIG + 1, 12, -17, grad=1) < size(BIG, 5 * BIG, 12, -17, grad=1)
