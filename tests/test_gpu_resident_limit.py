"""The largest matrix whose recurrences go in one launch (four rows for each of a workgroup's 1024 threads) and one
row more, which keeps a launch per step: log(A) V, its adaptive form and the estimate, against the launches per step
that an explicit tile order asks for.  The recurrences are the same bits; the sums of an estimate or a norm are
FP64 in another grouping: 1e-12 of the estimate, equal degrees."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402
from tests.test_gpu_resident import band  # noqa: E402


@pytest.mark.parametrize("n,one_launch", [(4096, True), (4097, False)])
def test_largest_matrix_in_one_launch(n, one_launch):
    csr = band(n)
    A = ld.CSR.from_arrays(csr[0], csr[1], csr[2], n, dtype=torch.float32)
    steps = ld.Options(tile_order=1)
    V = torch.tensor(np.random.default_rng(1).standard_normal((n, 7)), dtype=torch.float32, device="cuda")
    assert torch.equal(ld.apply_log(A, 0.5, 6.5, 30, V), ld.apply_log(A, 0.5, 6.5, 30, V, steps))
    o1, d1 = ld.apply_log_adaptive(A, 0.5, 6.5, 30, 1e-3, V)
    o2, d2 = ld.apply_log_adaptive(A, 0.5, 6.5, 30, 1e-3, V, steps)
    assert (d1 == d2).all() and torch.allclose(o1, o2, rtol=0, atol=1e-5)
    est, st = ld.logdet(A, 0.5, 6.5, 30, 30, 7, return_stats=True)
    one, st1 = ld.logdet(A, 0.5, 6.5, 30, 30, 7, options=steps, return_stats=True)
    assert abs(est - one) <= 1e-12 * abs(one)
    assert (st["launches1"] < st1["launches1"]) == one_launch
    assert ld.logdet_noalloc(A, 0.5, 6.5, 30, 30, 7) == est
