"""log(A) V on CSR rows whose staging decides whether V goes through padded copies and how many slices a row takes:
a band of 17 entries a row, enough rows for the rules of large matrices, column counts on both sides of each of
them, against the FP64 oracle and the same columns among others.  1e-12 / 2e-5 of a column's largest entry."""
import math

import numpy as np
import pytest

import workloads as w
from oracle import bounds, newton
from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_columns_around_the_padding_rule(dtype):
    n, degree = 44_100, 12
    rng = np.random.default_rng(4)
    idx = np.arange(n)
    u = np.concatenate([idx[: n - o] for o in range(1, 9)])
    v = np.concatenate([idx[o:] for o in range(1, 9)])
    x = -rng.uniform(0.2, 1.0, u.size)
    diag = 0.5 + np.bincount(u, -x, n) + np.bincount(v, -x, n)
    csr = w._assemble(n, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]), np.concatenate([diag, x, x]))
    A = ld.CSR.from_arrays(csr[0], csr[1], csr[2], n, dtype=dtype)
    csr_v = (csr[0], csr[1], A.val.double().cpu().numpy(), n)
    lo, hi = bounds.gershgorin(csr_v)
    plan = newton.NewtonPlan(lo, hi, degree)
    plan.d = ld.divided_differences(plan.lo, plan.hi, degree)[0]
    V = torch.tensor(rng.standard_normal((n, 31)), dtype=dtype, device="cuda")
    Vh = V.double().cpu().numpy()
    ref = plan.apply_poly(w.to_scipy(csr_v), Vh) + math.log(plan.sigma) * Vh
    tol = 1e-12 if dtype == torch.float64 else 2e-5
    for cols in (1, 3, 5, 6, 7, 9, 10, 11, 13, 17, 24, 31):
        out = ld.apply_log(A, lo, hi, degree, V[:, :cols].contiguous())
        assert_cols_close(out.double().cpu().numpy(), ref[:, :cols], tol)
