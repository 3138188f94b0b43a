"""log(A) V on a five-point stencil with more column chunks than a launch has workgroups in y (65535 of four
chunks; 2^20 columns are allowed): the first columns, those around the limit and the last ones are the columns
of narrow calls, whose results the other tests check.  Columns never interact and the launches' levels do not
depend on their number, so FP64 rounding is all that may differ: 1e-12."""
import pytest

from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import numpy as np  # noqa: E402

import paper_2603_02207_amd as ld  # noqa: E402
from tests.test_gpu_fused_steps import stencil  # noqa: E402


def test_more_chunks_than_one_grid():
    csr = stencil(128, 2)
    n, cols, degree = csr[3], 4 * 65535 * 2 + 11, 201   # a degree beyond the one-launch recurrences
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), n, dtype=torch.float64)
    V = torch.randn((n, cols), generator=torch.Generator("cuda").manual_seed(1), device="cuda", dtype=torch.float64)
    out = ld.apply_log(A, 0.25, 8.4, degree, V)
    limit = 4 * 65535 * 2
    for at in (slice(0, 7), slice(limit - 4, limit + 5), slice(cols - 3, cols)):
        ref = ld.apply_log(A, 0.25, 8.4, degree, V[:, at].contiguous())
        assert_cols_close(out[:, at].cpu().numpy(), ref.cpu().numpy(), 1e-12)
