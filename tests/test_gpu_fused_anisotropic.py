"""Launches of several steps on stencils whose x and y couplings differ, against the FP64 oracle and one launch per
step: a coupling taken for the other, or one not folded into its coefficient, is off by far more than the bounds.
Those of the equal couplings in FP64 (1e-10 of an estimate, 1e-12 and 1e-11 of a column's largest entry).  In FP32 the
y coupling, the diagonals' values times alpha, is an FP32 number by the choice of the basis, the x coupling rounds
(2^-25 at most): the estimate within 1e-7 (its rms over 16 matrices 1.5e-8; one launch per step 1.4e-7) and log(A) V
within 4e-7 in norm (1.0e-7; 1.3e-7)."""
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
from tests.test_gpu_adaptive_accuracy import grid  # noqa: E402


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("cx,cy", [(0.7, 1.3), (1.3, 0.7), (0.05, 1.0), (1.0, 0.05)])
def test_unequal_couplings(cx, cy, dtype):
    A, lo, hi = grid(140, 37, 1.3, 0.2, cx, cy)
    B = A.with_values(A.val.to(dtype))   # the FP32 values in either precision
    Q = w.to_scipy((A.row_ptr.cpu().numpy(), A.col_idx.cpu().numpy(), A.val.double().cpu().numpy(), A.n))
    f64 = dtype == torch.float64
    for degree, queries in ((13, 12), (40, 30)):
        ref = hutchpp.logdet_estimate(Q, lo, hi, degree, queries, 3)
        est, st = ld.logdet(B, lo, hi, degree, queries, 3, return_stats=True)
        one, st1 = ld.logdet(B, lo, hi, degree, queries, 3, options=ld.Options(tile_order=1), return_stats=True)
        assert st["dia_constant"] == 1 and st["launches1"] < st1["launches1"]
        assert abs(est - ref) < (1e-10 if f64 else 1e-7) * abs(ref)
        assert abs(est - one) < (1e-11 if f64 else 1e-6) * abs(ref)
    V = torch.tensor(np.random.default_rng(2).standard_normal((A.n, 9)), dtype=dtype, device="cuda")
    Vh = V.double().cpu().numpy()
    ref = newton.apply_log(Q, Vh, lo, hi, 30)
    out = ld.apply_log(B, lo, hi, 30, V).double().cpu().numpy()
    aout, deg = ld.apply_log_adaptive(B, lo, hi, 30, 0.0, V)
    assert (deg == 30).all()
    if f64:
        assert_cols_close(out, ref, 1e-12)
        assert_cols_close(aout.cpu().numpy(), ref, 1e-11)
    else:
        for x in (out, aout.double().cpu().numpy()):
            assert np.linalg.norm(x - ref) <= 4e-7 * np.linalg.norm(ref)


def test_estimate_of_equal_couplings_in_fp32():
    """400^2 points, degree 80, 60 queries: the coefficients' moved centres leave 2e-9 (one launch per step, whose
    alpha and beta round, 2e-7); 5e-8 fails without them."""
    A, lo, hi = grid(400, 400, 1.0, 0.1013, 1.0, 1.0)
    B = A.with_values(A.val.double())
    for seed in range(6):
        ref = ld.logdet(B, lo, hi, 80, 60, seed)
        assert abs(ld.logdet(A, lo, hi, 80, 60, seed) - ref) <= 5e-8 * abs(ref)
