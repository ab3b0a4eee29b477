"""Peel programs of more steps than the LDS form's records name, which take the
forms with slots in registers and in LDS, and both sides of the register limit on
blocks large enough for register slots: exact on integers."""
import sys

import pytest

from paper_1904_11563_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402

REG_SLOTS = 12  # the most live slots the register form holds


def _chains(kb, stride):
    """kb data blocks in `stride` chains: block i is released by {i - stride, i},
    so about `stride` values are live at a time."""
    return bpx.Code.from_columns(2, 2, kb // 2, [
        [(i,) if i < stride else (i - stride, i) for i in range(kb)], [(i,) for i in range(kb)]])


def _check(plan, M, N, pad):
    inf = plan.info()
    Mb, kb = inf["Mb"], plan.code.info()["k"] * plan.code.info()["b"]
    sch, (_, sym_ptr, sym_data) = plan.schedule(), plan.code.csr()
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randint(-1000, 1001, (kb, Mb, N), generator=g, device="cuda").float()
    X.view(kb * Mb, N)[M:] = 0
    Y = torch.full((max(int((sch["dest"] >= 0).sum()), 1), Mb, N), float("nan"), device="cuda")
    C = torch.full((kb * Mb, -(-N // 4) * 4 + pad), float("nan"), device="cuda")
    for sym, d in zip(sch["computed"].tolist(), sch["dest"].tolist()):
        v = sum(X[int(u)] for u in sym_data[sym_ptr[sym]:sym_ptr[sym + 1]])
        if d >= 0:
            Y[d] = v
        else:
            C[(-1 - d) * Mb:(-d) * Mb, :N] = v
    # only the M rows of the matrix are the caller's
    buf = torch.full((M + 8, C.shape[1]), float("nan"), device="cuda")
    buf[:M] = C[:M]
    plan.upload()
    bpx.peel_decode(plan, Y.view(torch.uint8).flatten(), buf[:M, :N])
    torch.cuda.synchronize()
    assert torch.equal(buf[:M, :N], X.view(kb * Mb, N)[:M])
    assert bool(buf[M:].isnan().all()) and bool(buf[:, N:].isnan().all())


# four columns per thread and one (odd N), few live slots and more than registers
# hold, a ragged last block, an empty one
@pytest.mark.parametrize("stride", [1, 5, 20])
@pytest.mark.parametrize("Mb,cut,N", [(1, 0, 4), (5, 3, 36), (5, 7, 33), (40, 1, 260), (3, 0, 1)])
def test_long_programs_exact(stride, Mb, cut, N):
    kb = 300
    M = kb * Mb - cut
    plan = bpx.Plan(_chains(kb, stride), [0, 1], 0, bpx.MODE_STRAGGLER, M, 4, N)
    assert plan.info()["Mb"] == Mb
    prog = plan.peel_program()
    print("peel", stride, Mb, N, "steps", len(prog["steps"]), "slots", prog["n_slots"],
          file=sys.stderr, flush=True)
    assert len(prog["steps"]) >= 256
    assert (prog["n_slots"] > REG_SLOTS) == (stride > REG_SLOTS)
    _check(plan, M, N, 4)


# blocks of 2^19 elements and more, 17 to 255 steps: register slots up to the
# limit, the LDS form past it
@pytest.mark.parametrize("stride", [REG_SLOTS - 1, REG_SLOTS, REG_SLOTS + 1])
@pytest.mark.parametrize("Mb,N", [(256, 2048), (257, 2044), (1024, 512)])
def test_register_limit_on_large_blocks_exact(stride, Mb, N):
    kb = 40
    M = kb * Mb - 3
    plan = bpx.Plan(_chains(kb, stride), [0, 1], 0, bpx.MODE_STRAGGLER, M, 4, N)
    prog = plan.peel_program()
    print("peel", stride, Mb, N, "steps", len(prog["steps"]), "slots", prog["n_slots"],
          file=sys.stderr, flush=True)
    assert 16 < len(prog["steps"]) < 256 and Mb * N >= 524288
    _check(plan, M, N, 0)
