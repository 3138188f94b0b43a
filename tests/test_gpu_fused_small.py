"""Launches of several steps on stencils too small to fill the device, where a wave takes as few as two lines: an odd
line left over, a last line cut short, one column and several chunks, against the FP64 oracle; and no slower than one
launch per step (an explicit tile order), which walks of 16 lines were (sketch steps of 4.6 us against 3.4; now 2.0).
Bounds as for the other stencils: 1e-10 of an estimate in FP64 and 2e-5 in FP32, 1e-12 and 2e-5 of a column's largest
entry."""
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
from tests.test_gpu_fused_steps import stencil  # noqa: E402


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("width,lines,cut", [(128, 63, 0), (128, 33, 50), (230, 101, 0)])
def test_short_walks_against_oracle(width, lines, cut, dtype):
    csr = stencil(width, lines, cut, holes=7)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=dtype)
    Q = w.to_scipy((csr[0], csr[1], A.val.double().cpu().numpy(), csr[3]))
    lo, hi, degree = 0.25, 8.4, 22
    f64 = dtype == torch.float64
    for queries in (9, 60):
        ref = hutchpp.logdet_estimate(Q, lo, hi, degree, queries, 5)
        assert abs(ld.logdet(A, lo, hi, degree, queries, 5) - ref) < (1e-10 if f64 else 2e-5) * abs(ref)
    V = torch.tensor(np.random.default_rng(2).standard_normal((csr[3], 9)), dtype=dtype, device="cuda")
    for cols in (1, 9):
        v = V[:, :cols].contiguous()
        ref = newton.apply_log(Q, v.double().cpu().numpy(), lo, hi, degree)
        assert_cols_close(ld.apply_log(A, lo, hi, degree, v).double().cpu().numpy(), ref, 1e-12 if f64 else 2e-5)
        out, deg = ld.apply_log_adaptive(A, lo, hi, degree, 0.0, v)
        assert (deg == degree).all()
        assert_cols_close(out.double().cpu().numpy(), ref, 1e-11 if f64 else 2e-5)


@pytest.mark.parametrize("width,lines", [(128, 128), (200, 40)])
def test_small_stencils_are_no_slower_than_single_steps(width, lines):
    csr = stencil(width, lines)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float32)
    ms = {}
    for name, opts in (("several", ld.Options()), ("single", ld.Options(tile_order=1))):
        runs = [ld.logdet(A, 0.25, 8.4, 60, 30, 1, options=opts, return_stats=True)[1] for _ in range(12)]
        ms[name] = (min(r["ms_steps1"] for r in runs), min(r["ms_steps23"] for r in runs))
    assert ms["several"][0] < ms["single"][0] and ms["several"][1] < ms["single"][1], ms
