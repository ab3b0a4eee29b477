"""What a call's workspace decides: nothing but the kernels that run.  Any
workspace that the plan's parts fit in is accepted, and what does not fit, or
cannot be addressed, is left to the kernels that need less."""
import ctypes
import functools
import sys

import pytest

from paper_1904_11563_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402


@functools.lru_cache
def _code():
    s = inputs.CODE_1284
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


def _run(entry, plan, A, B, ws=None):
    C = torch.full((plan.M, -(-plan.N // 4) * 4), float("nan"), device="cuda")[:, :plan.N]
    if entry == "noalloc":
        bpx.coded_matmul_noalloc(plan, A, B, C)
    else:
        bpx.coded_matmul(plan, A, B, C, ws)
    torch.cuda.synchronize()
    return C.clone()


def _err(X, R):
    return float(torch.linalg.norm(X.double() - R) / torch.linalg.norm(R))


def _view(x):
    r, c = x.shape
    t = torch.zeros((r, -(-c // 4) * 4), device="cuda")
    t[:, :c] = x
    return t[:, :c]


# Products whose packed operands fit in the library's 32 MiB, with and without all
# the room for partial tiles: the same kernels, the same bits
@pytest.mark.parametrize("prec", [bpx.PREC_F32, bpx.PREC_BF16X3, bpx.PREC_BF16])
@pytest.mark.parametrize("M,K,N", [(1024, 1024, 1024), (1100, 1028, 777), (419, 2052, 373)])
def test_library_scratch_holds_packed_operands(M, K, N, prec):
    arrival, _ = inputs.shifted_exp_arrival(0, 12)
    plan = bpx.Plan(_code(), arrival, 0, bpx.MODE_STRAGGLER, M, K, N, prec)
    plan.upload()
    A, B = _ops(2, M, K, N)
    A, B = _view(A), _view(B)
    full = torch.full((plan.workspace_bytes()[0],), 0xA5, dtype=torch.uint8, device="cuda")
    want = _run("matmul", plan, A, B, full)
    print("scratch", M, K, N, prec, len(full) >> 20, "MiB", file=sys.stderr, flush=True)
    assert torch.equal(_run("noalloc", plan, A, B), want)
    if prec == bpx.PREC_F32:      # not those of the kernels that read A and B directly
        direct = _run("matmul", plan, A, B, full[:plan.workspace_layout()[6]])
        assert not torch.equal(direct, want)


# Every size from the parts alone to all of it: exact on integers, FP32 accuracy
@pytest.mark.parametrize("prec", [bpx.PREC_F32, bpx.PREC_FP8])
@pytest.mark.parametrize("M,K,N", [(419, 3428, 373), (2048, 2048, 1024)])
def test_any_workspace_between(M, K, N, prec):
    arrival, _ = inputs.shifted_exp_arrival(0, 12)
    plan = bpx.Plan(_code(), arrival, 0, bpx.MODE_STRAGGLER, M, K, N, prec)
    most, least = plan.workspace_bytes()[0], plan.workspace_layout()[6]
    buf = torch.full((most,), 0xA5, dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    A = _view(torch.randint(-8, 9, (M, K), generator=g, device="cuda").float())
    B = _view(torch.randint(-8, 9, (K, N), generator=g, device="cuda").float())
    Af, Bf = map(_view, _ops(4, M, K, N))
    R = Af.double() @ Bf.double()
    sizes = [least, (least + most) // 2 // 256 * 256, most - (1 << 20), most - 256, most]
    for nbytes in sizes:
        if nbytes < least:
            continue
        print("workspace", M, K, N, prec, nbytes, "of", most, file=sys.stderr, flush=True)
        buf.fill_(0xA5)
        if prec == bpx.PREC_F32:
            assert torch.equal(_run("matmul", plan, A, B, buf[:nbytes]).double(),
                               A.double() @ B.double())
            assert _err(_run("matmul", plan, Af, Bf, buf[:nbytes]), R) <= 1e-5
        else:            # the codes are the same: only the MFMA's own summation differs
            got = _run("matmul", plan, Af, Bf, buf[:nbytes])
            direct = got if nbytes == least else direct
            # 1.5e-5 per product, times what the releases make of it
            assert _err(got, direct.double()) <= 1e-3
        assert bool((buf[nbytes:] == 0xA5).all())


# FP8 products past 2^31 multiply-adds: the documented codes and scales of B in a
# workspace of the parts alone, left alone in a larger one
def test_fp8_codes_in_a_workspace_of_the_parts():
    M, K, N = 2048, 2048, 1024
    arrival, _ = inputs.shifted_exp_arrival(0, 12)
    plan = bpx.Plan(_code(), arrival, 0, bpx.MODE_STRAGGLER, M, K, N,
                    bpx.PREC_FP8)
    off, most = plan.workspace_layout(), plan.workspace_bytes()[0]
    assert most > off[6]
    A, B = _ops(5, M, K, N)
    B = B * torch.logspace(-3, 3, K, device="cuda")[:, None]
    blocks = B.view(K // 128, 128, N // 128, 128).abs().amax(dim=(1, 3))
    scale = torch.exp2(torch.ceil(torch.log2(blocks.double() / 448)))
    want = (B.double() / scale.repeat_interleave(128, 0).repeat_interleave(128, 1)).float()
    want = want.to(torch.float8_e4m3fn).t().contiguous().view(torch.uint8)
    for nbytes in (off[6], most):
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        print("fp8 codes", nbytes, "of", most, file=sys.stderr, flush=True)
        C = torch.empty((M, N), device="cuda")
        bpx.coded_gemm(plan, A, B, C, ws)
        torch.cuda.synchronize()
        if nbytes == off[6]:
            assert torch.equal(ws[off[4]:off[4] + N * K].view(N, K), want)
            assert torch.equal(ws[off[5]:off[6]].view(torch.float32)[:scale.numel()].double(),
                               scale.flatten())
        else:
            assert bool((ws[off[1]:off[6]] == 0xA5).all())


# A tile table that names a shape for one product of a group: that product on the
# kernels that read A directly, the others on packed operands as without it
def test_named_shape_takes_only_its_product_off_packed_operands():
    from paper_1904_11563_amd import autotune
    shapes = [(2048, 1024, 2048)] * 4 + [(2304, 512, 1800), (2048, 4096, 2048)]
    plans = []
    for i, (M, K, N) in enumerate(shapes):
        arrival, _ = inputs.shifted_exp_arrival(i, 12)
        plans.append(bpx.Plan(_code(), arrival, 0, bpx.MODE_STRAGGLER, M, K, N,
                              bpx.PREC_BF16X3))
    base = sum(-(-p.workspace_layout()[6] // 256) * 256 for p in plans)
    nbytes = bpx.group_workspace_bytes(plans)
    assert nbytes > base
    ops = [_ops(20 + i, *s) for i, s in enumerate(shapes)]
    As, Bs = [a for a, _ in ops], [b for _, b in ops]

    def run(table, size, integers=False):
        A = [torch.round(a * 4) for a in As] if integers else As
        B = [torch.round(b * 4) for b in Bs] if integers else Bs
        Cs = [torch.full((M, N), float("nan"), device="cuda") for M, _, N in shapes]
        bpx.set_tile_table(table)
        try:
            ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
            group = bpx.Group(plans, A, B, Cs, ws)
        finally:
            bpx.set_tile_table(None)
        print("group with a table" if table else "group", size, file=sys.stderr, flush=True)
        for _ in range(2):
            group.launch()
        torch.cuda.synchronize()
        if integers:
            for a, b, c in zip(A, B, Cs):
                assert torch.equal(c.double(), a.double() @ b.double())
        del group
        return Cs

    named = 5
    table = [-1] * autotune.N_ENTRIES
    M, K, N = shapes[named]
    table[autotune.index(bpx.PREC_BF16X3, plans[named].info()["Mb"], N, K)] = 1
    packed, direct = run(None, nbytes), run(None, base)
    mixed = run(table, nbytes)
    for i in range(len(shapes)):
        assert _err(mixed[i], As[i].double() @ Bs[i].double()) <= 1e-4
        if i != named:
            assert torch.equal(mixed[i], packed[i]), i
    assert not torch.equal(mixed[named], packed[named])
    run(table, nbytes, integers=True)
    # named throughout: the direct kernels, whatever the workspace
    table = [4] * autotune.N_ENTRIES
    for got, want in zip(run(table, nbytes), direct):
        assert torch.equal(got, want)
