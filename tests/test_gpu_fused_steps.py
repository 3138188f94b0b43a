"""Several Newton steps per launch on constant five-point stencils, against the FP64 oracle and the
single-step launches (which an explicit tile order keeps).

Sizes: the shortest lines taken and a line just above, below and at whole strips; fewer lines than a wave's
chunk and one line more; a last line cut short; entries missing inside the grid.  Degrees that leave one
level, one launch exactly, and launches of unequal levels, for the sketch (up to 6 levels) and for the
quadratic forms (3 or 4).  Tolerances: the repository's bounds for estimates on stencils, 1e-10 relative in
FP64 and 2e-5 in FP32; between the two kinds of launch 1e-11 and 1e-5."""
import numpy as np
import pytest

import workloads as w
from oracle import bounds, hutchpp, newton
from tests.gpu_common import assert_cols_close, random_spd_csr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402


def stencil(width, lines, cut=0, holes=0, wrap=False):
    """0.3 I + five-point stencil on `lines` lines of `width` points, the last `cut` points left out, `holes`
    symmetric pairs of entries removed; `wrap` keeps the entries between the end of a line and the next's start."""
    n = width * lines - cut
    idx = np.arange(n)
    rng = np.random.default_rng(width + lines)
    rows, cols = [], []
    for off in (1, width):
        i = idx[: n - off]
        keep = np.ones(i.size, dtype=bool) if (off != 1 or wrap) else i % width != width - 1
        keep[rng.choice(i.size, min(holes, i.size), replace=False)] = False
        rows.append(i[keep])
        cols.append(i[keep] + off)
    u, v = np.concatenate(rows), np.concatenate(cols)
    o = np.full(u.size, -1.0)
    return w._assemble(n, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]),
                       np.concatenate([np.full(n, 4.3), o, o]))


CASES = [  # width, lines, cut, holes, wrap, degree, queries
    (128, 40, 0, 0, False, 6, 12),
    (128, 17, 5, 0, False, 1, 9),
    (129, 16, 0, 30, False, 7, 30),
    (156, 33, 100, 0, True, 19, 14),
    (208, 1 + 16 * 3, 0, 5, False, 24, 60),
    (1000, 3, 999, 0, False, 13, 3),
    (300, 300, 1, 200, True, 40, 33),
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("width,lines,cut,holes,wrap,degree,queries", CASES)
def test_fused_steps_against_oracle(width, lines, cut, holes, wrap, degree, queries, dtype):
    csr = stencil(width, lines, cut, holes, wrap)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=dtype)
    lo, hi = 0.25, 8.4
    vals = A.val.double().cpu().numpy()
    ref = hutchpp.logdet_estimate(w.to_scipy((csr[0], csr[1], vals, csr[3])), lo, hi, degree, queries, 3)
    tol, between = (1e-10, 1e-11) if dtype == torch.float64 else (2e-5, 1e-5)
    est, st = ld.logdet(A, lo, hi, degree, queries, 3, return_stats=True)
    one, st1 = ld.logdet(A, lo, hi, degree, queries, 3, options=ld.Options(tile_order=1), return_stats=True)
    assert st["dia_constant"] == 1 and st1["dia_constant"] == 1
    assert abs(est - ref) < tol * abs(ref)
    assert abs(est - one) < between * abs(ref)
    if st["dot_mode_used"] == ld.LD_DOT_SQUARED:   # fewer launches than steps
        assert degree == 1 or st["launches1"] < st1["launches1"]
    assert ld.logdet(A, lo, hi, degree, queries, 3) == est   # repeatable
    gauss = ld.Options(probe_dist=1)
    ref_g = hutchpp.logdet_estimate(w.to_scipy((csr[0], csr[1], vals, csr[3])), lo, hi, degree, queries, 3,
                                    probes="gaussian")
    assert abs(ld.logdet(A, lo, hi, degree, queries, 3, options=gauss) - ref_g) < tol * abs(ref_g)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind", ["fused", "stencil", "csr"])
def test_apply_log_column_counts(kind, dtype):
    """log(A) V at column counts around whole 16-byte vectors: launches of several steps on packed chunks (one
    chunk used in place, a misaligned V, several chunks), and padded copies of V elsewhere; a workspace too
    small for the packed blocks gives the same columns.  1e-12 / 2e-5 of a column's largest entry."""
    csr = {"fused": lambda: stencil(150, 31, 7, 3), "stencil": lambda: stencil(30, 40),
           "csr": lambda: random_spd_csr(1500, 3, density=0.01, long_rows=1)}[kind]()
    n = csr[3]
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), n, dtype=dtype)
    vals = A.val.double().cpu().numpy()
    lo, hi = (0.25, 8.4) if kind != "csr" else bounds.gershgorin((csr[0], csr[1], vals, n))
    Q = w.to_scipy((csr[0], csr[1], vals, n))
    rng = np.random.default_rng(1)
    tol = 1e-12 if dtype == torch.float64 else 2e-5
    for cols, degree in ((1, 9), (2, 4), (3, 5), (4, 8), (5, 3), (17, 12), (67, 4)):
        store = torch.tensor(rng.standard_normal(n * cols + 1), dtype=dtype, device="cuda")
        for shift in (0, 1):   # V at an odd element: rows on no vector boundary
            V = store[shift:shift + n * cols].view(n, cols)
            out = ld.apply_log(A, lo, hi, degree, V).double().cpu().numpy()
            ref = newton.apply_log(Q, V.double().cpu().numpy(), lo, hi, degree)
            assert_cols_close(out, ref, tol)
    # the size without packed blocks is still accepted
    import ctypes

    from paper_2603_02207_amd import _native as nat
    c, o = A.c_struct(), ld.Options().to_c()
    b = ctypes.c_size_t(0)
    nat.check(nat.load().ld_workspace_size(ctypes.byref(c), 12, -17, 0, ctypes.byref(o), ctypes.byref(b)), "size")
    elem = 8 if dtype == torch.float64 else 4
    pad = -(-(n * 20 if elem == 4 else n * 18) * elem // 256) * 256
    plain = b.value - 3 * pad + 2 * (-(-n * 17 * elem // 256) * 256)
    V = torch.tensor(rng.standard_normal((n, 17)), dtype=dtype, device="cuda")
    small, out = torch.empty(plain, dtype=torch.uint8, device="cuda"), torch.empty_like(V)
    args = (ctypes.byref(c), float(lo), float(hi), 12, ctypes.c_void_p(V.data_ptr()), ctypes.c_void_p(out.data_ptr()),
            17, ctypes.byref(o), ctypes.c_void_p(small.data_ptr()))
    assert nat.load().ld_apply_log(*args, plain, None) == nat.LD_OK
    torch.cuda.synchronize()
    assert_cols_close(out.double().cpu().numpy(), newton.apply_log(Q, V.double().cpu().numpy(), lo, hi, 12), tol)
    assert nat.load().ld_apply_log(*args, plain - 256, None) == nat.LD_EWORKSPACE


def test_bounds_of_the_cases():
    for width, lines, cut, holes, wrap, _, _ in CASES:
        lo, hi = bounds.gershgorin(stencil(width, lines, cut, holes, wrap))
        assert lo >= 0.25 and hi <= 8.4
