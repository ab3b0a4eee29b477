"""FP32 products on split planes at the ends of their range: how far a single
product may be off."""
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402


def _uncoded(M, K, N):
    """Every row of A on its own: no sums of blocks, no peel."""
    plan = bpx.Plan(bpx.Code.identity(2, 2), [0, 1], 0, bpx.MODE_STRAGGLER, M, K, N)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6]
    return plan


def _run(plan, A, B, tile=-1):
    C = torch.full((plan.M, plan.N), float("nan"), device="cuda")
    ws = torch.full((max(plan.workspace_bytes()[0], 256),), 0xA5, dtype=torch.uint8, device="cuda")
    bpx.force_tile(tile)
    try:
        bpx.coded_matmul(plan, A, B, C, ws)
        torch.cuda.synchronize()
    finally:
        bpx.force_tile(-1)
    return C


def _signed(lo, hi, shape, gen):
    """Magnitudes in [2^lo, 2^hi), spread over their exponents."""
    x = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
    s = torch.randint(0, 2, shape, generator=gen, device="cuda") * 2.0 - 1.0
    return (torch.exp2(x * (hi - lo) + lo) * s).float()


def _err(X, R):
    return float(torch.linalg.norm(X.double() - R) / torch.linalg.norm(R))


# One nonzero per row of A: every output is one product.  The planes leave out
# m.l, l.m and l.l, at most 2 2^-8 2^-17 + 2^-34 of the operands' powers of two;
# the matrix instruction cuts what it has summed at the last place of a larger
# product before it adds and rounds, so the last one, h.h, costs up to a unit,
# 2^-23 of the product, and those before it 2^-7 times as much together.
@pytest.mark.parametrize("ends", [(-1, 1), (-60, 30)])
def test_single_products(ends):
    M, K, N = 4096, 512, 4096
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.zeros((M, K), device="cuda")
    A[torch.arange(M, device="cuda"),
      torch.randint(0, K, (M,), generator=g, device="cuda")] = _signed(*ends, (M,), g)
    A[::2] *= 0.0
    # mantissas around 1 + 2^-8, where h rounds the furthest
    at = torch.randint(0, K, (M // 2,), generator=g, device="cuda")
    A[torch.arange(0, M, 2, device="cuda"), at] = 1 + 2.0 ** -8 * (
        0.5 + torch.rand((M // 2,), generator=g, device="cuda"))
    B = _signed(*ends, (K, N), g)
    B[:, ::2] = 1 + 2.0 ** -8 * (0.5 + torch.rand((K, N // 2), generator=g, device="cuda"))
    R = A.double() @ B.double()
    plan = _uncoded(M, K, N)
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    rel = lambda X: float(((X.double() - R) / R).abs().max()) * 2.0 ** 24
    print("single products", ends, "planes", rel(new), _err(new, R), "direct", rel(old),
          _err(old, R), file=sys.stderr, flush=True)
    assert rel(old) <= 1.001
    assert rel(new) <= 3.05
    # and exact where the other factor is a power of two
    A = torch.sign(A) * 0.125
    assert torch.equal(_run(plan, A, B).double(), A.double() @ B.double())
