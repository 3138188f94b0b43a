"""The spectral interval at its edges: Lanczos on the smallest matrices, at row counts around the kernels'
lane groups, past an invariant subspace and past the polling interval; and the CSR check on every kind of
broken structure.  Tolerance: the repository's 1e-8 between the device's Lanczos bound and the oracle's."""
import numpy as np
import pytest

import workloads as w
from oracle import bounds, rng
from tests.gpu_common import random_spd_csr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402


def diagonal(n, values):
    idx = np.arange(n)
    return w._assemble(n, idx, idx, np.resize(np.asarray(values, dtype=np.float64), n))


CASES = {
    "one row": (diagonal(1, [3.0]), 4),
    "identity": (diagonal(300, [2.0]), 20),
    "two values": (diagonal(65, [1.0, 5.0]), 20),
    "penta 2 lane groups": (w.pentadiagonal(65, 1), 12),
    "grid 63 rows": (w.grid_laplacian_2d(7, 0.5), 49),
    "mean row 20": (random_spd_csr(1000, 3, density=0.02), 20),
    "mean row 60": (random_spd_csr(1025, 5, density=0.06, long_rows=1), 20),
    "past one poll": (w.grid_laplacian_2d(200, 0.1), 100),
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", sorted(CASES))
def test_lanczos_edges(name, dtype):
    csr, steps = CASES[name]
    n = csr[3]
    vals = np.asarray(csr[2], dtype=np.float32 if dtype == torch.float32 else np.float64).astype(np.float64)
    A = ld.CSR.from_arrays(csr[0], csr[1], vals, n, dtype=dtype)
    csr_v = (csr[0], csr[1], vals, n)
    g_lo, g_hi = bounds.gershgorin(csr_v)
    _, upper = bounds.lanczos_upper(w.to_scipy(csr_v), steps, rng.rademacher(0, 2, n, 1)[:, 0])
    lo, hi = ld.spectral_bounds(A, lanczos_steps=steps)
    assert lo == pytest.approx(g_lo, rel=1e-12)
    assert hi == pytest.approx(min(upper, g_hi), rel=1e-8)
    assert ld.spectral_bounds(A, lanczos_steps=steps) == (lo, hi)   # repeatable


def valid(row_ptr, col_idx, n):
    nnz = len(col_idx)
    if row_ptr[0] != 0 or row_ptr[-1] != nnz or (np.diff(row_ptr) < 0).any() or (row_ptr < 0).any():
        return False
    if ((col_idx < 0) | (col_idx >= n)).any():
        return False
    return all((np.diff(col_idx[b:e]) > 0).all() for b, e in zip(row_ptr[:-1], row_ptr[1:]))


def test_csr_check_finds_every_break():
    csr = random_spd_csr(300, 7, density=0.03, long_rows=1)
    rp, ci, val, n = (np.array(x) if i < 3 else x for i, x in enumerate(csr))
    r = int(np.argmax(np.diff(rp)))
    b = rp[r]
    broken = []
    for at, to in ((b, -1), (b + 3, n), (b + 3, ci[b + 2]), (rp[5], ci[rp[5] + 1] + 1), (len(ci) - 1, -5)):
        c = ci.copy()
        c[at] = to
        broken.append((rp, c))
    for at, to in ((0, 1), (n, len(ci) - 1), (n, len(ci) + 1), (10, rp[11] + 4), (r + 1, rp[r] - 1), (r, -3),
                   (20, 2**31 - 1)):
        p = rp.copy()
        p[at] = to
        broken.append((p, ci))
    p, c = rp.copy(), ci.copy()    # a row's end moved into the next row: the same drops, at another place
    p[41] += 1
    broken.append((p, c))
    broken.append((rp, ci[::-1].copy()))
    for p, c in broken:
        assert not valid(p, c, n)
        A = ld.CSR.from_arrays(p, c, val, n, dtype=torch.float64)
        for call in (lambda: ld.spectral_bounds(A), lambda: ld.spectral_bounds(A, 5),
                     lambda: ld.logdet(A, 0.5, 60.0, 5, 6, 0)):
            with pytest.raises(ld.NativeError) as e:
                call()
            assert e.value.code == -2
    empty_rows = (np.array([0, 0, 2, 2, 3, 3], dtype=np.int32), np.array([0, 4, 1], dtype=np.int32))
    assert valid(*empty_rows, 5)
    A = ld.CSR.from_arrays(*empty_rows, np.ones(3), 5, dtype=torch.float64)
    lo, hi = ld.spectral_bounds(A)      # accepted; no diagonal, so the interval is not positive
    assert lo <= 0.0
