"""Rows at the edges of the long-row kernel's regimes (64 / 65 entries: row group / wave; 1024 / 1025:
wave / workgroup), at column counts that leave one to 64 row groups per wave, against the FP64 oracle.

Tolerances: log(A) V by the repository's FP64 and FP32 bounds of an irregular matrix (1e-12 and 2e-5 of a
column's largest entry), the estimate 1e-10 and 2e-5 relative."""
import math

import numpy as np
import pytest

import workloads as w
from oracle import bounds, hutchpp, newton
from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402

N = 2600
LENGTHS = {3: 64, 700: 65, 701: 127, 1500: 1024, 1501: 1025, 2599: 2400}   # row: stored entries


def long_row_matrix():
    """Symmetric diagonally dominant matrix whose named rows hold exactly the named number of entries."""
    rng = np.random.default_rng(5)
    special = np.array(sorted(LENGTHS))
    ordinary = np.setdiff1d(np.arange(N), special)
    pairs = {}
    for r, length in LENGTHS.items():   # partners among the ordinary rows, the diagonal is one more entry
        for c in rng.choice(ordinary, length - 1, replace=False):
            pairs[(min(r, c), max(r, c))] = rng.uniform(0.2, 1.0)
    u = np.array([p[0] for p in pairs])
    v = np.array([p[1] for p in pairs])
    x = -np.array(list(pairs.values()))
    diag = 0.5 + np.bincount(u, -x, N) + np.bincount(v, -x, N)
    idx = np.arange(N)
    csr = w._assemble(N, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]), np.concatenate([diag, x, x]))
    assert all(np.diff(csr[0])[r] == length for r, length in LENGTHS.items())
    return csr


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_long_rows_at_the_edges(dtype):
    csr = long_row_matrix()
    vals = np.asarray(csr[2], dtype=np.float32 if dtype == torch.float32 else np.float64)
    A = ld.CSR.from_arrays(csr[0], csr[1], vals, N, dtype=dtype)
    csr_v = (csr[0], csr[1], vals.astype(np.float64), N)
    lo, hi = bounds.gershgorin(csr_v)
    Q = w.to_scipy(csr_v)
    plan = newton.NewtonPlan(lo, hi, 20)
    plan.d = ld.divided_differences(plan.lo, plan.hi, 20)[0]   # the kernels alone are under test here
    for cols in (1, 4, 21, 64):
        V = torch.tensor(np.random.default_rng(cols).standard_normal((N, cols)), dtype=dtype, device="cuda")
        out = ld.apply_log(A, lo, hi, 20, V).double().cpu().numpy()
        ref = plan.apply_poly(Q, V.double().cpu().numpy()) + math.log(plan.sigma) * V.double().cpu().numpy()
        assert_cols_close(out, ref, 1e-12 if dtype == torch.float64 else 2e-5)
    for m_vec, mode in ((3, ld.LD_DOT_SQUARED), (64, ld.LD_DOT_FORWARD), (129, ld.LD_DOT_SQUARED)):
        est = ld.logdet(A, lo, hi, 20, m_vec, 1, options=ld.Options(dot_mode=mode))
        ref = hutchpp.logdet_estimate(Q, lo, hi, 20, m_vec, 1)
        assert abs(est - ref) < (1e-10 if dtype == torch.float64 else 2e-5) * abs(ref), (m_vec, mode)
