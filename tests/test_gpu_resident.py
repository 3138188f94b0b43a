"""Matrices small enough for a whole recurrence in one launch, against the FP64 oracle and the one-launch-per-step
path (which an explicit tile order keeps): row counts around a workgroup's threads and their multiples, the
largest matrix of either precision that fits and one that does not, rows without entries off the diagonal,
column counts around whole 16-byte vectors, FP64 column sums, Alg. 2's stopping degrees.  Bounds as elsewhere
for well-conditioned matrices: 1e-12 / 1e-5 for log(A) V, 1e-10 / 1e-5 for estimates; the two paths' recurrences
are the same bits, so their estimates differ by the grouping of FP64 sums only (1e-12)."""
import numpy as np
import pytest

import workloads as w
from oracle import hutchpp, newton
from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402


def band(n):
    """Tridiagonal part of a chain with a third of its links removed, plus a few long links; spectrum in [0.5, 6.5]."""
    rng = np.random.default_rng(n)
    idx = np.arange(n)
    u = idx[: n - 1][rng.random(n - 1) < 0.67]
    far = idx[: max(0, n - 40)][::97]
    u, v = np.concatenate([u, far]), np.concatenate([u + 1, far + 37])
    x = -rng.uniform(0.3, 0.9, u.size)
    diag = 0.6 + np.bincount(u, -x, n) + np.bincount(v, -x, n)
    return w._assemble(n, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]), np.concatenate([diag, x, x]))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [5, 64, 1023, 1024, 1025, 2049, 3700, 5200])
def test_one_launch_recurrences(n, dtype):
    csr = band(n)
    A = ld.CSR.from_arrays(csr[0], csr[1], csr[2], n, dtype=dtype)
    Q = w.to_scipy((csr[0], csr[1], A.val.double().cpu().numpy(), n))
    lo, hi = 0.5, 6.5
    steps = ld.Options(tile_order=1)
    tol, tol_est = (1e-12, 1e-10) if dtype == torch.float64 else (1e-5, 1e-5)
    for cols, degree in ((1, 1), (3, 17), (4, 30), (7, 40), (18, 25)):
        V = torch.tensor(np.random.default_rng(cols).standard_normal((n, cols)), dtype=dtype, device="cuda")
        out = ld.apply_log(A, lo, hi, degree, V)
        assert torch.equal(out, ld.apply_log(A, lo, hi, degree, V, steps))
        assert_cols_close(out.double().cpu().numpy(), newton.apply_log(Q, V.double().cpu().numpy(), lo, hi, degree), tol)
        for t in (0.0, 1e-4, 1e9):
            o1, d1 = ld.apply_log_adaptive(A, lo, hi, degree, t, V)
            o2, d2 = ld.apply_log_adaptive(A, lo, hi, degree, t, V, steps)
            assert (d1 == d2).all()
            assert_cols_close(o1.double().cpu().numpy(), o2.double().cpu().numpy(), tol)
    for m_vec, degree in ((3, 1), (14, 40), (15, 41), (60, 20)):
        if m_vec // 3 > n:
            continue
        for probes in (0, 1):
            opts = ld.Options(probe_dist=probes)
            if n == 5 and m_vec > 3 and not probes:   # the sketch is rank-deficient, refused either way
                for o in (opts, steps):
                    with pytest.raises(ld.NativeError, match="rank-deficient"):
                        ld.logdet(A, lo, hi, degree, m_vec, 7, options=o)
                continue
            est, st = ld.logdet(A, lo, hi, degree, m_vec, 7, options=opts, return_stats=True)
            one, st1 = ld.logdet(A, lo, hi, degree, m_vec, 7, options=ld.Options(probe_dist=probes, tile_order=1),
                                 return_stats=True)
            ref = hutchpp.logdet_estimate(Q, lo, hi, degree, m_vec, 7, probes="gaussian" if probes else "rademacher")
            assert abs(est - ref) < tol_est * max(abs(ref), 1.0), (m_vec, probes)
            assert abs(est - one) <= 1e-12 * max(abs(ref), 1.0) or n == 5
            if n <= 3700:
                assert st["launches1"] < st1["launches1"] or degree == 1
        if n == 5 and m_vec > 3:
            continue
        e1, d1 = ld.logdet_adaptive(A, lo, hi, degree, 1e-3, m_vec, 7)
        e2, d2 = ld.logdet_adaptive(A, lo, hi, degree, 1e-3, m_vec, 7, options=steps)
        assert (d1 == d2).all() and abs(e1 - e2) <= tol_est * max(abs(e1), 1.0)
