"""CSR rows dealt to slices of lanes: row lengths around whole batches of the slices (none, 1 to 9, 16, 17, 32,
33, 64 and, with the long rows, 65 entries), row counts around whole tiles, and column counts that give one to
16 lanes per slice or too many for slices.  Every entry point that steps, against the FP64 oracle with the
library's own coefficients: log(A) V to 1e-12 / 2e-5 of a column's largest entry, estimates 1e-10 / 2e-5."""
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

LENGTHS = (1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65)


def matrix(n, seed):
    """Symmetric, diagonally dominant; the first rows hold exactly LENGTHS entries, the others 10 to 40 on average."""
    rng = np.random.default_rng(seed)
    k = len(LENGTHS)
    pairs = set()
    for r, length in enumerate(LENGTHS):
        pairs |= {(r, int(c)) for c in rng.choice(np.arange(k, n), length - 1, replace=False)}
    u = rng.integers(k, n, 10 * n)
    v = rng.integers(k, n, 10 * n)
    pairs |= {(min(a, b), max(a, b)) for a, b in zip(u.tolist(), v.tolist()) if a != b}
    u, v = np.array(sorted(pairs)).T
    x = -rng.uniform(0.2, 1.0, u.size)
    idx = np.arange(n)
    diag = 0.5 + np.bincount(u, -x, n) + np.bincount(v, -x, n)
    csr = w._assemble(n, np.concatenate([idx, u, v]), np.concatenate([idx, v, u]), np.concatenate([diag, x, x]))
    assert tuple(np.diff(csr[0])[:k]) == LENGTHS and csr[1].size > 9 * n
    return csr


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [127, 128, 1025])
def test_slices_at_the_edges(n, dtype):
    csr = matrix(n, n)
    A = ld.CSR.from_arrays(csr[0], csr[1], csr[2], n, dtype=dtype)
    csr_v = (csr[0], csr[1], A.val.double().cpu().numpy(), n)
    Q = w.to_scipy(csr_v)
    lo, hi = bounds.gershgorin(csr_v)
    plan = newton.NewtonPlan(lo, hi, 24)
    plan.d = ld.divided_differences(plan.lo, plan.hi, 24)[0]
    tol, tol_est = (1e-12, 1e-10) if dtype == torch.float64 else (2e-5, 2e-5)
    for cols in (1, 4, 6, 16, 33, 64):
        V = torch.tensor(np.random.default_rng(cols).standard_normal((n, cols)), dtype=dtype, device="cuda")
        Vh = V.double().cpu().numpy()
        ref = plan.apply_poly(Q, Vh) + math.log(plan.sigma) * Vh
        assert_cols_close(ld.apply_log(A, lo, hi, 24, V).double().cpu().numpy(), ref, tol)
        out, deg = ld.apply_log_adaptive(A, lo, hi, 24, 0.0, V)
        assert (deg == 24).all()
        assert_cols_close(out.double().cpu().numpy(), ref, tol)
    for m_vec, mode in ((3, ld.LD_DOT_SQUARED), (14, ld.LD_DOT_FORWARD), (40, ld.LD_DOT_SQUARED), (100, ld.LD_DOT_SQUARED)):
        ref = hutchpp.logdet_estimate(Q, lo, hi, 24, m_vec, 2)
        for order in (1, 2):
            est = ld.logdet(A, lo, hi, 24, m_vec, 2, options=ld.Options(dot_mode=mode, tile_order=order))
            assert abs(est - ref) < tol_est * abs(ref), (m_vec, mode, order)
