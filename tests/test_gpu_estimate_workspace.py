"""ld_logdet_estimate in a workspace without room for the single column block that scattered matrices take: it keeps
the column blocks that follow the stored bytes, as the size of such a workspace (a constant of the shape below) was
the entry point's whole requirement before that block was introduced.  The blocks group FP64 sums differently and
nothing else: 1e-11.  A page less is refused."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_02207_amd as ld  # noqa: E402
from paper_2603_02207_amd import _native as nat  # noqa: E402

N, QUERIES, DEGREE, LEAST = 400_000, 96, 4, 607_607_040   # FP64, 17 entries a row


def circulant():
    """Eight pairs of neighbours far away from every row, weights 1, diagonal 20."""
    i = torch.arange(N, device="cuda")
    off = torch.tensor([s * (23_456 * k + 7) for k in range(1, 9) for s in (1, -1)], device="cuda")
    col = torch.cat([i[:, None], (i[:, None] + off[None, :]) % N], 1)
    val = torch.full((N, 17), -1.0, dtype=torch.float64, device="cuda")
    val[:, 0] = 20.0
    col, order = col.sort(1)
    row_ptr = torch.arange(N + 1, device="cuda", dtype=torch.int32) * 17
    return ld.CSR(row_ptr, col.flatten().to(torch.int32), val.gather(1, order).flatten(), N)


def test_smaller_workspace_keeps_several_blocks():
    A = circulant()
    o, c = ld.Options().to_c(), A.c_struct()
    need = ld.workspace_size(A, DEGREE, QUERIES)
    assert need > LEAST
    got = {}
    for size in (need, LEAST, LEAST - 4096):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out, st = ctypes.c_double(0.0), nat.LdStats()
        rc = nat.load().ld_logdet_estimate(
            ctypes.byref(c), 4.0, 36.0, DEGREE, QUERIES, ctypes.c_uint64(5), ctypes.byref(o),
            ctypes.c_void_p(ws.data_ptr()), ws.numel(), None, ctypes.byref(out), ctypes.byref(st))
        assert rc == (nat.LD_EWORKSPACE if size < LEAST else nat.LD_OK)
        got[size] = (out.value, st.as_dict()["block_cols1"])
    assert got[need][1] == QUERIES // 3 > got[LEAST][1]
    assert abs(got[need][0] - got[LEAST][0]) <= 1e-11 * abs(got[need][0])
