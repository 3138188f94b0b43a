"""Calls without a workspace, and through the binding where PyTorch has no memory for one: the library allocates what
the matrix needs and, where there is no memory for the launches of several steps, the blocks of one launch per step.
The device is filled but for the room of those.  Same columns and degrees: 1e-11 (FP64)."""
import pytest

from tests.gpu_common import assert_cols_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import numpy as np  # noqa: E402

import paper_2603_02207_amd as ld  # noqa: E402
from tests.test_gpu_fused_steps import stencil  # noqa: E402

LO, HI = 0.25, 8.4
GIB = 1 << 30


@pytest.mark.parametrize("shape", ["stencil", "pentadiagonal", "small"])
def test_binding_without_memory_for_the_workspace(shape, monkeypatch):
    """torch.empty refuses every workspace: all four entry points still return what they do with one."""
    csr = {"stencil": lambda: stencil(150, 40), "pentadiagonal": lambda: stencil(2, 3000), "small": lambda: stencil(20, 20)}[shape]()
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float64)
    V = torch.tensor(np.random.default_rng(5).standard_normal((csr[3], 7)), device="cuda")

    def results():
        out, deg = ld.apply_log_adaptive(A, LO, HI, 20, 1e-4, V)
        est, degs = ld.logdet_adaptive(A, LO, HI, 20, 1e-4, 12, 3)
        return ld.logdet(A, LO, HI, 20, 12, 3), est, degs, ld.apply_log(A, LO, HI, 20, V), out, deg

    want = results()

    def refuse(*args, **kwargs):
        raise torch.OutOfMemoryError("no room")

    monkeypatch.setattr(ld, "_workspace", refuse)
    got = results()
    assert got[0] == want[0] and got[1] == want[1]
    assert (got[2] == want[2]).all() and (got[5] == want[5]).all()
    assert torch.equal(got[3], want[3]) and torch.equal(got[4], want[4])
    with pytest.raises(torch.OutOfMemoryError):   # the gradient has no smaller form
        ld.logdet_with_grad(A, LO, HI, 20, 12, 3)


def test_full_device_takes_one_launch_per_step():
    csr = stencil(2000, 2000)
    A = ld.CSR.from_arrays(csr[0], csr[1], np.asarray(csr[2]), csr[3], dtype=torch.float64)
    V = torch.randn((csr[3], 32), generator=torch.Generator("cuda").manual_seed(2), device="cuda", dtype=torch.float64)
    want = ld.apply_log(A, LO, HI, 9, V)
    awant, dwant = ld.apply_log_adaptive(A, LO, HI, 9, 0.0, V)
    block = V.numel() * 8
    torch.cuda.empty_cache()
    # the result, and room for two more blocks and the rest of the workspaces, not for four
    keep = block + int(2.9 * block) + GIB // 4
    hog = torch.empty(torch.cuda.mem_get_info()[0] - keep, dtype=torch.uint8, device="cuda")
    try:
        got = ld.apply_log(A, LO, HI, 9, V)
        assert_cols_close(got[:, ::5].cpu().numpy(), want[:, ::5].cpu().numpy(), 1e-11)
        del got
        torch.cuda.empty_cache()
        got, deg = ld.apply_log_adaptive(A, LO, HI, 9, 0.0, V)
        assert (deg == dwant).all()
        assert_cols_close(got[:, ::5].cpu().numpy(), awant[:, ::5].cpu().numpy(), 1e-11)
    finally:
        del hog
        torch.cuda.empty_cache()
