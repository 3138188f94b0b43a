"""Alg. 2's loop on stencils where the columns stop after a few steps: the same degrees and columns as one launch per
step (an explicit tile order) wherever they stop, and, where all of them stop at the first step, the time of one
launch per step (launches of four steps with their repeat took 1.6 times that: 687 us against 433 on 1000^2 points,
32 columns; a tenth is left for the measurement)."""
import time

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

LO, HI = 0.25, 8.4


@pytest.mark.parametrize("dtype,vtol", [(torch.float64, 1e-11), (torch.float32, 2e-5)])
@pytest.mark.parametrize("scale", [1.0, 1e-3, 1e6])
def test_stops_anywhere(dtype, vtol, scale):
    csr = stencil(150, 40, 3, 5)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=dtype)
    rng = np.random.default_rng(8)
    V = torch.tensor(rng.standard_normal((csr[3], 6)) * scale * np.geomspace(1.0, 1e3, 6), dtype=dtype, device="cuda")
    seen = set()
    Q = w.to_scipy((csr[0], csr[1], A.val.double().cpu().numpy(), csr[3]))
    e = e_sequence(newton.NewtonPlan(LO, HI, 26), Q, V.double().cpu().numpy())
    for tol in scale * csr[3] ** 0.5 * np.geomspace(2e3, 2e-4, 29):
        if not clear_of_ties(e, tol, 1e-4):
            continue
        out, deg = ld.apply_log_adaptive(A, LO, HI, 26, float(tol), V)
        one, odeg = ld.apply_log_adaptive(A, LO, HI, 26, float(tol), V, options=ld.Options(tile_order=1))
        np.testing.assert_array_equal(deg, odeg)
        assert_cols_close(out.double().cpu().numpy(), one.double().cpu().numpy(), vtol)
        seen |= set(deg.tolist())
    assert {0, 1, 2, 3, 5, 26} <= seen


def test_non_finite_columns_stop_alone():
    csr = stencil(150, 40)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float64)
    V = torch.tensor(np.random.default_rng(1).standard_normal((csr[3], 3)), device="cuda")
    V[7, 1] = float("nan")
    V[9, 2] = float("inf")
    out, deg = ld.apply_log_adaptive(A, LO, HI, 20, 1e-3, V)
    one, odeg = ld.apply_log_adaptive(A, LO, HI, 20, 1e-3, V, options=ld.Options(tile_order=1))
    np.testing.assert_array_equal(deg, odeg)
    assert_cols_close(out[:, 0].cpu().numpy(), one[:, 0].cpu().numpy(), 1e-11)
    assert torch.equal(out[:, 1:].isfinite(), one[:, 1:].isfinite())


def test_one_step_is_no_slower_than_single_launches():
    csr = stencil(1000, 1000)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float32)
    V = torch.randn((csr[3], 32), generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    best = {}
    for name, opts in (("several", ld.Options()), ("single", ld.Options(tile_order=1))):
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            _, deg = ld.apply_log_adaptive(A, LO, HI, 60, 2e3, V, options=opts)
            torch.cuda.synchronize()
            best[name] = min(best.get(name, 1e9), time.perf_counter() - t)
            assert (deg == 1).all()
    assert best["several"] < 1.1 * best["single"], best
