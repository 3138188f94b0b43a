"""FP32 accuracy of the adaptive estimate on five-point stencils: several steps per launch are no less accurate than
one launch per step (an explicit tile order).  The error of each against the FP64 library on the same FP32 values, rms
over 48 matrices (scales and shifts as hyperparameter fitting meets them, equal and unequal couplings), in the same
probes; the bound is the single steps' rms and a fifth for the spread of two rms values over 48 samples
(1 / sqrt(2 * 48) each).  With d_0 rounded to FP32 the ratio is 1.3 to 1.55."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402


def grid(width, lines, tau, kappa2, cx, cy):
    """tau (kappa2 I + cx, cy five-point Laplacian), Dirichlet: CSR with FP32 values, its interval."""
    n = width * lines
    i = np.arange(n)
    x = i % width
    off = np.array([-width, -1, 0, 1, width])
    ok = np.stack([i >= width, x > 0, np.ones(n, bool), x < width - 1, i < n - width], 1)
    val = tau * np.array([-cy, -cx, 2 * cx + 2 * cy + kappa2, -cx, -cy])
    row_ptr = np.concatenate([[0], ok.sum(1).cumsum()])
    A = ld.CSR.from_arrays(row_ptr, (i[:, None] + off)[ok], np.broadcast_to(val, (n, 5))[ok], n, dtype=torch.float32)
    return A, 0.999 * tau * kappa2, tau * (kappa2 + 4 * cx + 4 * cy)


@pytest.mark.parametrize("cx,cy", [(1.0, 1.0), (0.7, 1.3)])
def test_several_steps_are_no_less_accurate(cx, cy):
    rng = np.random.default_rng(11)
    single = ld.Options(tile_order=1)
    err = {"several": [], "single": []}
    for s in range(48):
        A, lo, hi = grid(130, 40, 0.5 + 2.0 * rng.random(), 0.05 + 0.5 * rng.random(), cx, cy)
        tol = 1e-7 * A.n ** 0.5
        B = A.with_values(A.val.double())
        ref, _ = ld.logdet_adaptive(B, lo, hi, 60, tol, 30, s, options=single)
        for name, opts in (("several", None), ("single", single)):
            est, _ = ld.logdet_adaptive(A, lo, hi, 60, tol, 30, s, options=opts)
            err[name].append(est / ref - 1.0)
    rms = {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in err.items()}
    assert rms["several"] <= 1.2 * rms["single"], rms
