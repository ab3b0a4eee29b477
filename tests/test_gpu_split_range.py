"""FP32 products on split planes at the ends of their range: how far a single
product may be off, operands down to the smallest subnormal number, and the
magnitude from which tiles go to the FP32 kernels."""
import sys

import pytest

from paper_1904_11563_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402


def _code(s):
    return bpx.Code.search(s.n, s.k, s.b, s.sigma, s.seed, s.restarts, s.iters, walk=s.walk)


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


def _both(plan, A, B):
    R = A.double() @ B.double()
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    d = lambda X: float(torch.linalg.norm(X.double() - R))
    return new, old, d(new), d(old)


# Values down to the smallest subnormal one run on the planes (the FP32 kernels
# sum in another order, so their bits differ) and are no further off than there
@pytest.mark.parametrize("ends_a,ends_b", [((-149, 0), (-2, 2)), ((-2, 2), (-149, 0)),
                                           ((-126, -100), (30, 40)), ((-149, -120), (20, 36))])
def test_small_values_stay_on_planes(ends_a, ends_b):
    M, K, N = 1100, 1028, 1100
    code = _code(inputs.CODE_642)
    arrival, _ = inputs.shifted_exp_arrival(0, 6)
    plan = bpx.Plan(code, arrival, 0, bpx.MODE_FULL, M, K, N)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6] and not plan.fused()
    g = torch.Generator(device="cuda").manual_seed(5)
    A, B = _signed(*ends_a, (M, K), g), _signed(*ends_b, (K, N), g)
    A[:, 5] = 0.0
    B[7, :] = -0.0
    new, old, dn, do = _both(plan, A, B)
    print("small values", ends_a, ends_b, dn, do, file=sys.stderr, flush=True)
    assert not torch.equal(new, old)
    assert dn <= do + 2.0 ** -149 * (M * N) ** 0.5


# (both operands spread over many powers of two: sums of a few products each,
# for which the bound of single products holds, 3.05 times the FP32 kernels')
def test_small_values_two_dimensional():
    M, K, N = 1100, 1028, 1040
    arrival, _ = inputs.shifted_exp_arrival(1, 5)
    plan = bpx.Plan(bpx.Code.table1(), arrival, 0, bpx.MODE_FULL, M, K, N, two_d=True)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6]
    g = torch.Generator(device="cuda").manual_seed(6)
    A, B = _signed(-149, 0, (M, K), g), _signed(-30, 0, (K, N), g)
    new, old, dn, do = _both(plan, A, B)
    print("small values 2-D", dn, do, file=sys.stderr, flush=True)
    assert not torch.equal(new, old)
    assert dn <= 3.05 * do + 2.0 ** -149 * (M * N) ** 0.5


# K = 1024 products of magnitudes under 2^42 fit the scaled sums' range; from
# there up the panel of 256 rows or columns goes to the FP32 kernels
@pytest.mark.parametrize("side", ["a", "b"])
def test_largest_value_on_planes(side):
    M, K, N = 1024, 1024, 1024
    plan = _uncoded(M, K, N)
    g = torch.Generator(device="cuda").manual_seed(7)
    below = 2.0 ** 42 * (1 - 2.0 ** -24)
    panel = (slice(512, 768), slice(None)) if side == "a" else (slice(None), slice(512, 768))
    for value, split in ((below, True), (-below, True), (2.0 ** 42, False), (-(2.0 ** 42), False),
                         (2.0 ** 112, False), (torch.finfo(torch.float32).max, False)):
        A, B = (torch.randn((M, K), generator=g, device="cuda"),
                torch.randn((K, N), generator=g, device="cuda") * 2.0 ** -8)
        if side == "a":
            A[600, 1023] = value
        else:
            B[0, 700] = value
        new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
        print("largest", side, value, split, file=sys.stderr, flush=True)
        # (the largest FP32 value overflows in FP32 arithmetic too)
        assert torch.equal(torch.isfinite(new), torch.isfinite(old)) and not new.isnan().any()
        assert torch.equal(new[panel], old[panel]) != split
        assert not torch.equal(new, old)            # the other panels stay on planes
    # every product at the edge, all of one sign
    A, B = torch.full((M, K), below, device="cuda"), torch.full((K, N), below, device="cuda")
    C = _run(plan, A, B)
    R = A.double() @ B.double()
    assert float(((C.double() - R) / R).abs().max()) <= 1e-6


# A captured call on operands with and without values for the FP32 kernels:
# the same finite values and the same infinities and NaN as the eager call
def test_flagged_panels_in_a_graph():
    M, K, N = 1473, 1000, 1280
    arrival, _ = inputs.shifted_exp_arrival(0, 12)
    plan = bpx.Plan(_code(inputs.CODE_1284), arrival, 0, bpx.MODE_STRAGGLER, M, K, N)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6] and not plan.fused()
    plan.upload()
    gen = torch.Generator(device="cuda").manual_seed(8)
    A = torch.randn((M, K), generator=gen, device="cuda")
    B = torch.randn((K, N), generator=gen, device="cuda")
    C = torch.empty((M, N), device="cuda")
    ws = bpx.alloc_workspace(plan)
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            bpx.coded_matmul(plan, A, B, C, ws)
    torch.cuda.current_stream().wait_stream(s)
    for what in ("none", "inf a", "nan b", "both", "none"):
        A[M - 1, 1] = float("inf") if what in ("inf a", "both") else 1.0
        B[3, 2] = float("nan") if what in ("nan b", "both") else 1.0
        want = _run(plan, A, B)
        C.fill_(float("nan"))
        ws.fill_(0xA5)
        g.replay()
        torch.cuda.synchronize()
        print("graph", what, int(want.isnan().sum()), int(want.isinf().sum()), file=sys.stderr,
              flush=True)
        assert torch.equal(C.isnan(), want.isnan())
        ok = ~want.isnan()
        assert torch.equal(C[ok], want[ok])
        assert bool(ok.all()) == (what == "none")
