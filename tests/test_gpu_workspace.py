"""What a call's workspace decides: nothing but the kernels that run.  Any
workspace that the plan's parts fit in is accepted, and what does not fit, or
cannot be addressed, is left to the kernels that need less."""
import ctypes
import sys

import pytest

from paper_1904_11563_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402


def _code(s):
    return bpx.Code.search(s.n, s.k, s.b, s.sigma, s.seed, s.restarts, s.iters, walk=s.walk)


def _ops(seed, M, K, N):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn((M, K), generator=g, device="cuda"),
            torch.randn((K, N), generator=g, device="cuda"))


def _raw(entry, plan, A, B, C, ptr, nbytes):
    """An entry point with a workspace given as a plain address and size."""
    st = getattr(bpx._lib, entry)(
        plan._h, ctypes.c_void_p(A.data_ptr()), plan.K, ctypes.c_void_p(B.data_ptr()), plan.N,
        ctypes.c_void_p(C.data_ptr()), plan.N, ctypes.c_void_p(ptr), nbytes,
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return st


# A plan whose parts are empty (an uncoded layout: every product goes straight
# into C, and no tile of 256 x 256 fits), with operands that would be packed: no
# workspace, or one off the alignment, is accepted whatever size is named
@pytest.mark.parametrize("entry", ["bpx_coded_gemm", "bpx_coded_matmul"])
def test_plan_without_parts_takes_any_workspace(entry):
    M, K, N = 630, 516, 260
    code = bpx.Code.identity(4, 8)
    plan = bpx.Plan(code, [0, 1, 2, 3], 0, bpx.MODE_STRAGGLER, M, K, N)
    need = plan.workspace_bytes()[0]
    assert plan.workspace_layout()[6] == 0 and need > 0 and not plan.fused()
    A, B = _ops(1, M, K, N)
    buf = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    outs = []
    for ptr, nbytes in ((0, 0), (0, need), (buf.data_ptr() + 16, need), (buf.data_ptr() + 4, need)):
        C = torch.full((M, N), float("nan"), device="cuda")
        print(entry, "workspace", "none" if ptr == 0 else ptr - buf.data_ptr(), nbytes,
              file=sys.stderr, flush=True)
        assert _raw(entry, plan, A, B, C, ptr, nbytes) == 0
        outs.append(C)
        assert bool((buf == 0xA5).all())      # a workspace that is not usable is left alone
    for C in outs[1:]:
        assert torch.equal(C, outs[0])
    R = A.double() @ B.double()
    assert float(torch.linalg.norm(outs[0].double() - R) / torch.linalg.norm(R)) <= 1e-5
    # the same size, aligned: the packed operands
    C = torch.full((M, N), float("nan"), device="cuda")
    assert _raw(entry, plan, A, B, C, buf.data_ptr(), need) == 0
    assert not bool((buf == 0xA5).all())
    assert float(torch.linalg.norm(C.double() - R) / torch.linalg.norm(R)) <= 1e-5
