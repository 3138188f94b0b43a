"""Alg. 2's loop with several steps per launch (constant five-point stencils), against the FP64 oracle and the
loop of one step per launch (which an explicit tile order keeps).

Column scales over ten orders make the columns stop everywhere: at degree 0, inside a launch, at its last step,
and never (the cap).  Caps below one launch's steps, at them, and of unequal launches; one column, part of a
16-byte chunk, chunks and a remainder, and more than the 64 columns of one mask.  Tolerances: the repository's
bounds for this entry point, 1e-11 in FP64 and 2e-5 in FP32 of each column; degrees are equal."""
import numpy as np
import pytest

import workloads as w
from oracle import newton
from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402
from tests.test_gpu_adaptive import clear_of_ties, e_sequence  # noqa: E402
from tests.test_gpu_fused_steps import stencil  # noqa: E402


@pytest.mark.parametrize("dtype,vtol", [(torch.float64, 1e-11), (torch.float32, 2e-5)])
@pytest.mark.parametrize("width,lines,cut,holes,wrap,cap,ncols", [
    (128, 17, 5, 0, False, 1, 3),
    (129, 16, 0, 30, False, 4, 1),
    (156, 33, 100, 0, True, 23, 8),
    (200, 40, 0, 5, False, 40, 17),
    (1000, 3, 999, 0, False, 30, 70),
    (2500, 2, 0, 0, False, 9, 64),
])
def test_fused_adaptive(width, lines, cut, holes, wrap, cap, ncols, dtype, vtol):
    csr = stencil(width, lines, cut, holes, wrap)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=dtype)
    Q = w.to_scipy((csr[0], csr[1], A.val.double().cpu().numpy(), csr[3]))
    lo, hi = 0.25, 8.4
    rng = np.random.default_rng(ncols)
    V = rng.standard_normal((csr[3], ncols)) * np.geomspace(1e-7, 1e3, ncols)[rng.permutation(ncols)]
    Vd = torch.tensor(V, dtype=dtype, device="cuda")
    Vin = Vd.double().cpu().numpy()
    e = e_sequence(newton.NewtonPlan(lo, hi, cap), Q, Vin)
    used = 0
    for tol in [0.0, *np.geomspace(3.0, 1e-4, 9), 1e30]:
        if tol > 0 and not clear_of_ties(e, tol, 1e-4):
            continue
        out, deg = ld.apply_log_adaptive(A, lo, hi, cap, float(tol), Vd)
        ref, rdeg = newton.apply_log_adaptive(Q, Vin, lo, hi, cap, float(tol))
        one, odeg = ld.apply_log_adaptive(A, lo, hi, cap, float(tol), Vd, options=ld.Options(tile_order=1))
        np.testing.assert_array_equal(deg, rdeg)
        np.testing.assert_array_equal(deg, odeg)
        assert_cols_close(out.double().cpu().numpy(), ref, vtol)
        assert_cols_close(out.double().cpu().numpy(), one.double().cpu().numpy(), vtol)
        again, _ = ld.apply_log_adaptive(A, lo, hi, cap, float(tol), Vd)
        assert torch.equal(out, again)
        used += 1
    assert used >= 4


def test_fused_adaptive_estimate():
    csr = stencil(160, 50, 3, 20)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float64)
    for tol in (1e-1, 1e-5):
        est, deg, st = ld.logdet_adaptive(A, 0.25, 8.4, 60, tol, 30, 2, return_stats=True)
        one, odeg, st1 = ld.logdet_adaptive(A, 0.25, 8.4, 60, tol, 30, 2, options=ld.Options(tile_order=1),
                                            return_stats=True)
        np.testing.assert_array_equal(deg, odeg)
        assert abs(est - one) <= 1e-11 * abs(one)
        assert st["launches1"] < st1["launches1"] and st["launches23"] < st1["launches23"]


def test_fused_adaptive_smaller_workspace():
    # a workspace without the four blocks of chunks takes one launch per step; one that is shorter still is refused
    import ctypes
    from paper_2603_02207_amd import _native as nat
    csr = stencil(160, 50, 3, 20)
    n, cols = csr[3], 17
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), n, dtype=torch.float64)
    V = torch.tensor(np.random.default_rng(3).standard_normal((n, cols)), device="cuda")
    want, wdeg = ld.apply_log_adaptive(A, 0.25, 8.4, 60, 1e-3, V)
    c, b = A.c_struct(), ctypes.c_size_t(0)
    nat.check(nat.load().ld_workspace_size(ctypes.byref(c), 60, -cols, 1, None, ctypes.byref(b)), "size")
    plain = b.value - 4 * ((n * 18 * 8 + 255) // 256 * 256)
    for size, refused in ((plain, False), (plain - 256, True)):
        ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        at = (ws.data_ptr() + 255) // 256 * 256
        out, deg = torch.empty_like(V), np.zeros(cols, dtype=np.int32)
        rc = nat.load().ld_apply_log_adaptive(
            ctypes.byref(c), 0.25, 8.4, 60, 1e-3, ctypes.c_void_p(V.data_ptr()), ctypes.c_void_p(out.data_ptr()), cols,
            None, ctypes.c_void_p(at), size, None, deg.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
        assert rc == (nat.LD_EWORKSPACE if refused else nat.LD_OK)
        if rc == nat.LD_OK:
            torch.cuda.synchronize()
            np.testing.assert_array_equal(deg, wdeg)
            assert_cols_close(out.cpu().numpy(), want.cpu().numpy(), 1e-11)
