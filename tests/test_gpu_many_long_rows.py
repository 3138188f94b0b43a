"""More long rows than the long-row kernel shares out among workgroups (8192): a wave for each row at any column
count; one row of 900 entries among them.  Against the FP64 oracle, bounds as for the other irregular matrices:
1e-12 / 2e-5 of a column's largest entry, 1e-10 / 2e-5 of an estimate."""
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


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_a_wave_for_each_of_many_rows(dtype):
    n, half = 8400, 33
    rng = np.random.default_rng(9)
    idx = np.arange(n)
    far = np.arange(4000, 4000 + 833 * 5, 5)
    u = np.concatenate([idx[: n - o] for o in range(1, half + 1)] + [np.full(far.size, 100)])
    v = np.concatenate([idx[o:] for o in range(1, half + 1)] + [far])
    x = -rng.uniform(0.2, 1.0, u.size)
    diag = 0.5 + np.bincount(u, -x, n) + np.bincount(v, -x, n)
    csr = w._assemble(n, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]), np.concatenate([diag, x, x]))
    assert (np.diff(csr[0]) > 64).sum() > 8192 and np.diff(csr[0]).max() == 900
    A = ld.CSR.from_arrays(csr[0], csr[1], csr[2], n, dtype=dtype)
    csr_v = (csr[0], csr[1], A.val.double().cpu().numpy(), n)
    Q = w.to_scipy(csr_v)
    lo, hi = bounds.gershgorin(csr_v)
    plan = newton.NewtonPlan(lo, hi, 12)
    plan.d = ld.divided_differences(plan.lo, plan.hi, 12)[0]
    f64 = dtype == torch.float64
    for cols in (5, 64):
        V = torch.tensor(rng.standard_normal((n, cols)), dtype=dtype, device="cuda")
        Vh = V.double().cpu().numpy()
        ref = plan.apply_poly(Q, Vh) + math.log(plan.sigma) * Vh
        assert_cols_close(ld.apply_log(A, lo, hi, 12, V).double().cpu().numpy(), ref, 1e-12 if f64 else 2e-5)
    ref = hutchpp.logdet_estimate(Q, lo, hi, 12, 96, 1)
    assert abs(ld.logdet(A, lo, hi, 12, 96, 1) - ref) < (1e-10 if f64 else 2e-5) * abs(ref)
