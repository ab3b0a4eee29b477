"""Large products on operands split into BF16 planes: exact on integers at the
edges of tiles, stages and K pieces, FP32 results no further from float64 than
the FP32 kernels', and values the planes cannot hold left to those kernels."""
import sys

import numpy as np
import pytest

from paper_1904_11563_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1904_11563_amd import bpx  # noqa: E402


def _code(s):
    return bpx.Code.search(s.n, s.k, s.b, s.sigma, s.seed, s.restarts, s.iters, walk=s.walk)


def _plan(spec, M, K, N, prec, mode=bpx.MODE_STRAGGLER):
    arrival, _ = inputs.shifted_exp_arrival(0, spec.n)
    plan = bpx.Plan(_code(spec), arrival, 0, mode, M, K, N, prec)
    # above the size at which the operands are split
    inf = plan.info()
    assert inf["n_computed"] * inf["Mb"] * K * N > 2 ** 31
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6]
    return plan


def _plan2d(code, M, K, N, mode):
    n = code.info()["n"]
    arrival, _ = inputs.shifted_exp_arrival(1, n)
    plan = bpx.Plan(code, arrival, 0, mode, M, K, N, two_d=True)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6]
    return plan


def _view(x, pad):
    """x in a buffer whose rows are `pad` floats (rounded up to 4) longer."""
    r, c = x.shape
    t = torch.full((r, -(-(c + pad) // 4) * 4), float("nan"), device="cuda")
    t[:, :c] = x
    return t[:, :c]


def _run(plan, A, B, tile=-1, pad=0, ws=None):
    A, B = _view(A, pad), _view(B, pad)
    C = _view(torch.full((plan.M, plan.N), float("nan"), device="cuda"), pad)
    if ws is None:
        ws = torch.full((plan.workspace_bytes()[0],), 0xA5, dtype=torch.uint8, device="cuda")
    bpx.force_tile(tile)
    try:
        bpx.coded_matmul(plan, A, B, C, ws)
        torch.cuda.synchronize()
    finally:
        bpx.force_tile(-1)
    return C.clone()


def _ops(seed, M, K, N, integer):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if integer:
        return (torch.randint(-8, 9, (M, K), generator=g, device="cuda").float(),
                torch.randint(-8, 9, (K, N), generator=g, device="cuda").float())
    return (torch.randn((M, K), generator=g, device="cuda"),
            torch.randn((K, N), generator=g, device="cuda"))


def _err(X, R):
    return float(torch.linalg.norm(X.double() - R) / torch.linalg.norm(R))


# M, K, N: one k chunk and a granule past a chunk (the shortest loops), K a
# multiple of neither stage, blocks and columns of one past a tile, a last
# round split along K (few tiles) and one that is not (short K), odd N
SHAPES = [(6000, 16, 30000), (6000, 20, 25000), (6000, 44, 9001), (6000, 64, 7000),
          (2056, 1000, 1025), (999, 4100, 769), (4104, 1048, 2306)]
PRECS = [bpx.PREC_F32, bpx.PREC_BF16X3, bpx.PREC_BF16]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", SHAPES)
def test_split_planes_exact_and_accurate(shape, prec):
    M, K, N = shape
    plan = _plan(inputs.CODE_642, M, K, N, prec, bpx.MODE_FULL)
    A, B = _ops(1, M, K, N, True)
    print("planes", shape, prec, file=sys.stderr, flush=True)
    C = _run(plan, A, B, pad=8)
    # members' sums of at most 4 x 8 and K products of at most 32 x 8 are exact
    assert torch.equal(C.double(), A.double() @ B.double())
    A, B = _ops(2, M, K, N, False)
    R = A.double() @ B.double()
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    print("  error", _err(new, R), "direct kernels", _err(old, R), file=sys.stderr, flush=True)
    # The same splits in BF16*, so the same error up to the order of the sums
    # (1e-6 at K = 4100); FP32: dropped plane products (2^-26 of a product) and
    # fewer roundings than the FP32 matrix instruction's K / 4 per output.
    assert _err(new, R) <= _err(old, R) * (1.0 if K > 256 else 1.1) + 1e-7
    assert torch.equal(new, _run(plan, A, B))          # deterministic
    small = torch.empty(plan.workspace_layout()[6], dtype=torch.uint8, device="cuda")
    if prec == bpx.PREC_F32:   # a workspace without the planes: the direct kernels
        assert _err(_run(plan, A, B, ws=small), R) <= 1e-5


# every pass count and kind of symbol; blocks of whole tiles, blocks ragged in
# both directions, a K of a few chunks, and fewer tiles than CUs (all split)
@pytest.mark.parametrize("mode", [bpx.MODE_FULL, bpx.MODE_MIN])
@pytest.mark.parametrize("code,shape", [("1282", (4096, 512, 4096)), ("1282", (1100, 3004, 1040)),
                                        ("1282", (5000, 44, 13008)), ("table1", (3001, 1000, 2600)),
                                        ("table3", (2000, 1200, 1812))])
def test_split_planes_two_dimensional(code, shape, mode):
    M, K, N = shape
    lib = {"1282": lambda: _code(inputs.CODE_1282), "table1": bpx.Code.table1,
           "table3": bpx.Code.table3}[code]()
    plan = _plan2d(lib, M, K, N, mode)
    print("planes 2-D", code, shape, mode, file=sys.stderr, flush=True)
    A, B = _ops(5, M, K, N, True)
    assert torch.equal(_run(plan, A, B, pad=4).double(), A.double() @ B.double())
    A, B = _ops(6, M, K, N, False)
    R = A.double() @ B.double()
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    print("  error", _err(new, R), "direct kernels", _err(old, R), file=sys.stderr, flush=True)
    assert _err(new, R) <= _err(old, R) * (1.0 if K > 256 else 1.1) + 1e-7
    assert torch.equal(new, _run(plan, A, B))
    small = torch.empty(max(plan.workspace_layout()[6], 256), dtype=torch.uint8, device="cuda")
    assert _err(_run(plan, A, B, ws=small), R) <= 1e-5
    for t in (A, B):          # one block's panels go to the FP32 kernels
        t[t.shape[0] - 1, 3] = float("inf")
        new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
        fin = torch.isfinite(old)
        assert torch.equal(torch.isnan(new), torch.isnan(old))
        assert torch.equal(torch.isfinite(new), fin)
        d = torch.where(fin, new.double() - R, 0.0)
        assert float(torch.linalg.norm(d) / torch.linalg.norm(R)) <= 1e-5


@pytest.mark.parametrize("shape", [(2048, 1024, 2048), (1999, 1500, 1001)])
def test_split_planes_leave_out_of_range_values_to_fp32(shape):
    """Infinities, NaN and values outside the planes' range: the same
    non-finite outputs as the FP32 kernels and, elsewhere, FP32 accuracy."""
    M, K, N = shape
    plan = _plan(inputs.CODE_1284, M, K, N, bpx.PREC_F32)
    for what in ("inf a", "nan b", "tiny a", "huge b", "max"):
        A, B = _ops(3, M, K, N, False)
        if what == "inf a":
            A[M - 1, K - 1] = float("inf")
        elif what == "nan b":
            B[0, N - 1] = float("nan")
        elif what == "tiny a":                # below the smallest normal number
            A[5, :] *= 1e-39
        elif what == "huge b":
            B[:, 7] *= 2.0 ** 100
        else:                                 # rounds up to infinity in BF16
            A[3, 4] = torch.finfo(torch.float32).max
            B[:, 2] = 2.0 ** -10
        new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
        fin = torch.isfinite(old)
        print("planes range", shape, what, int((~fin).sum()), file=sys.stderr, flush=True)
        assert torch.equal(torch.isnan(new), torch.isnan(old)), what
        assert torch.equal(torch.isfinite(new), fin), what
        R = A.double() @ B.double()
        scale = torch.linalg.norm(torch.where(fin, R, 0.0), dim=0).clamp_min(1e-300)
        e = lambda X: float((torch.linalg.norm(torch.where(fin, X.double() - R, 0.0), dim=0) /
                             scale).max())
        # per column, since a huge column would hide the others; coded sums mix
        # rows, so a row with a huge element is as far off as the direct kernels'
        assert e(new) <= max(e(old) * 1.1, 1e-5), what


@pytest.mark.parametrize("exps", [(0, 0), (-60, -40), (-70, -68), (30, 30)])
def test_split_planes_scale_of_operands(exps):
    """Operands far from 1 (results down to subnormal numbers) are no further
    from float64 than the FP32 kernels' results plus one subnormal unit."""
    M, K, N = 2048, 1024, 2048
    plan = _plan(inputs.CODE_642, M, K, N, bpx.PREC_F32)
    A, B = _ops(4, M, K, N, False)
    A, B = A * 2.0 ** exps[0], B * 2.0 ** exps[1]
    R = A.double() @ B.double()
    d = lambda X: float(torch.linalg.norm(X.double() - R))
    new, old = d(_run(plan, A, B)), d(_run(plan, A, B, tile=1))
    print("planes scale", exps, new, old, file=sys.stderr, flush=True)
    assert new <= old + 2.0 ** -149 * np.sqrt(M * N)


@pytest.mark.parametrize("prec", [bpx.PREC_BF16X3, bpx.PREC_BF16])
def test_grouped_split_planes_exact_and_like_direct_kernels(prec):
    """A group with enough 256 x 256 tiles for every CU (more tiles than CUs,
    so a workgroup takes several; K of one stage to many, ragged rows, columns
    and K): exact on integers, and on floats as accurate as the same group on
    the direct kernels, which a workspace without the planes gets."""
    specs = {4: _code(inputs.CODE_642), 8: _code(inputs.CODE_1282)}
    shapes = inputs.batch_shapes(7, 40, lo=256, hi=2048, mult=4)
    shapes += [(2000, 4, 700, 4), (300, 28, 4, 8), (8, 64, 2050 * 2, 4), (1, 36, 1028, 8)]
    plans, base = [], 0
    for i, (M, K, N, k) in enumerate(shapes):
        n = specs[k].info()["n"]
        arrival, _ = inputs.erasure_arrival(i, n, n - k)
        plans.append(bpx.Plan(specs[k], arrival, 0, bpx.MODE_STRAGGLER, M, K, N, prec))
        base += -(-plans[-1].workspace_layout()[6] // 256) * 256
    full = bpx.group_workspace_bytes(plans)
    assert full > base                       # the group runs on split planes
    for integer in (True, False):
        ops = [_ops(20 + i, M, K, N, integer) for i, (M, K, N, _) in enumerate(shapes)]
        As, Bs = [a for a, _ in ops], [b for _, b in ops]
        outs = []
        for nbytes in (full, base):
            Cs = [torch.full((M, N), float("nan"), device="cuda") for M, _, N, _ in shapes]
            ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
            g = bpx.Group(plans, As, Bs, Cs, ws)
            print("grouped planes", prec, integer, nbytes, file=sys.stderr, flush=True)
            for _ in range(2):
                g.launch()
            torch.cuda.synchronize()
            outs.append(Cs)
            del g
        for i, (a, b) in enumerate(ops):
            R = a.double() @ b.double()
            if integer:
                assert torch.equal(outs[0][i].double(), R), shapes[i]
            else:
                # the same splits, summed in another order
                new, old = _err(outs[0][i], R), _err(outs[1][i], R)
                assert new <= old * 1.1 + 1e-6, (shapes[i], new, old)


# M, K, N: blocks of 40 and of 300 rows (several symbols in one fragment, a
# block over three scale blocks), ragged columns and K, the shortest K (two
# stages) and K of 2, 3 and 5 scale blocks, tiles split along K and not
@pytest.mark.parametrize("prec", [bpx.PREC_FP8X2, bpx.PREC_FP8])
@pytest.mark.parametrize("code,shape", [("moj", (5000, 1000, 2001)), ("642", (2400, 500, 3000)),
                                        ("642", (9000, 100, 8200)), ("642", (9000, 200, 6000)),
                                        ("642", (2048, 4100, 513)), ("moj", (1500, 640, 2304))])
def test_packed_fp8_like_direct_kernels(code, shape, prec):
    """The codes and scales are those of the direct kernels (checked there
    against the oracle), so the products differ by the MFMA's own summation
    only: within 1e-4 of them (1.5e-5 measured between that and float64), far
    below what a wrong row, scale or plane gives."""
    M, K, N = shape
    lib = _code(inputs.CODE_642) if code == "642" else bpx.Code.mojette(16, 8, 24, 0)
    n = lib.info()["n"]
    arrival, _ = inputs.shifted_exp_arrival(3, n)
    mode = bpx.MODE_FULL if code == "642" else bpx.MODE_STRAGGLER
    plan = bpx.Plan(lib, arrival, 0, mode, M, K, N, prec)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6]
    A, B = _ops(8, M, K, N, False)
    # rows and columns of very different scale, so that a scale applied to
    # another row or column shows
    A = A * torch.logspace(-3, 3, M, device="cuda")[torch.randperm(M, device="cuda")][:, None]
    B = B * torch.logspace(-3, 3, -(-N // 128), device="cuda").repeat_interleave(128)[:N]
    print("packed fp8", code, shape, prec, file=sys.stderr, flush=True)
    ws = torch.full((plan.workspace_bytes()[0],), 0xA5, dtype=torch.uint8, device="cuda")
    base = torch.empty(plan.workspace_layout()[6], dtype=torch.uint8, device="cuda")
    Av, Bv = _view(A, 8), _view(B, 8)
    dest = plan.schedule()["dest"]
    Mb, ny = plan.info()["Mb"], int((dest >= 0).sum())
    prods = []
    for w in (ws, base):
        C = _view(torch.zeros((M, N), device="cuda"), 8)
        bpx.coded_gemm(plan, Av, Bv, C, w)
        torch.cuda.synchronize()
        Y = w[:ny * Mb * N * 4].view(torch.float32).view(ny, Mb, N)
        prods.append((Y.clone(), C.clone()))
    for new, old in zip(prods[0], prods[1]):
        if new.numel() == 0:
            continue
        # per product and column block, the granularity of the scales
        d = new.double() - old.double()
        for n0 in range(0, N, 128):
            num = torch.linalg.norm(d[..., n0:n0 + 128])
            den = torch.linalg.norm(old[..., n0:n0 + 128].double())
            assert float(num) <= 1e-4 * float(den), n0
    again = _view(torch.zeros((M, N), device="cuda"), 8)
    bpx.coded_gemm(plan, Av, Bv, again, ws)
    assert torch.equal(again, prods[0][1])


def _identity_y(plan, X):
    """Y slots and C as the coded products leave them for blocks X (float64
    sums rounded to FP32)."""
    sch, Mb, kb = plan.schedule(), plan.info()["Mb"], X.shape[0]
    col_ptr, sym_ptr, sym_data = plan.code.csr()
    ny = int((sch["dest"] >= 0).sum())
    Y = torch.full((max(ny, 1), Mb, X.shape[2]), float("nan"), device="cuda")
    C = torch.full((kb * Mb, X.shape[2]), float("nan"), device="cuda")
    for g, d in zip(sch["computed"].tolist(), sch["dest"].tolist()):
        s = sum(X[int(u)] for u in sym_data[sym_ptr[g]:sym_ptr[g + 1]])
        if d >= 0:
            Y[d] = s
        else:
            C[(-1 - d) * Mb:(-d) * Mb] = s
    return Y, C


# programs: one step, chains past depth 4 (FP64), degrees past the four and the
# eight subtrahends held in a record, 64 and more steps, blocks already in C
# only; sizes: one element, odd columns, four columns per lane and not, large
# blocks on both sides of the register form, a ragged last block, an empty one
@pytest.mark.parametrize("code,M,N", [
    ("table1", 4, 1), ("table3", 9 * 40 - 3, 333), ("642", 2048, 513), ("1284", 32 * 63 - 17, 1001),
    ("1284", 32 * 256, 2048), ("1284", 32 * 256 - 5, 1024), ("moj", 5000, 500), ("moj", 128 * 3 - 2, 68),
    ("wide", 20 * 9, 130), ("wide", 20 * 512, 512)])
def test_peel_forms_exact(code, M, N):
    if code == "wide":       # releases by one symbol that covers everything
        lib = bpx.Code.from_columns(3, 2, 10, [
            [(i,) for i in range(10)], [(i, i + 1) for i in range(9, 18)] + [tuple(range(20))],
            [(i,) for i in range(19)]])
    else:
        lib = {"table1": bpx.Code.table1, "table3": bpx.Code.table3,
               "642": lambda: _code(inputs.CODE_642), "1284": lambda: _code(inputs.CODE_1284),
               "moj": lambda: bpx.Code.mojette(16, 8, 24, 0)}[code]()
    inf = lib.info()
    seen = 0
    for seed in range(3):
        arrival, _ = inputs.shifted_exp_arrival(seed, inf["n"])
        lost, mode = 0, bpx.MODE_STRAGGLER
        if code == "wide":
            arrival = [0, 1, 2]
        elif code == "moj":
            (arrival, lost), mode = inputs.erasure_arrival(seed, inf["n"], inf["n"] // 3), bpx.MODE_ERASURE
        plan = bpx.Plan(lib, arrival, lost, mode, M, 4, N)
        if not plan.decodable:
            continue
        kb, Mb = inf["k"] * inf["b"], plan.info()["Mb"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        # integers: every sum and difference is exact
        X = torch.randint(-1000, 1001, (kb, Mb, N), generator=g, device="cuda").float()
        X.view(kb * Mb, N)[M:] = 0
        Y, C = _identity_y(plan, X)
        Cv = _view(C[:M], 4)
        plan.upload()
        prog = plan.peel_program()
        print("peel", code, M, N, "steps", len(prog["steps"]), "slots", prog["n_slots"],
              file=sys.stderr, flush=True)
        before = Cv._base.clone()
        bpx.peel_decode(plan, Y.view(torch.uint8).flatten(), Cv)
        torch.cuda.synchronize()
        assert torch.equal(Cv, X.view(kb * Mb, N)[:M])
        assert torch.equal(Cv._base[:, N:].isnan(), before[:, N:].isnan())  # nothing past N
        seen += 1
    assert seen


# 256-wide and 128-wide tiles: all whole, all in K pieces, a last round in
# pieces; rows, columns and K that fit neither
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", [(4700, 4100, 2560), (4100, 516, 2050), (2600, 2052, 1100),
                                   (1000, 4100, 777), (3001, 516, 2050)])
def test_split_planes_tile_sizes(shape, prec):
    M, K, N = shape
    plan = _plan(inputs.CODE_642, M, K, N, prec, bpx.MODE_FULL)
    print("tiles", shape, prec, file=sys.stderr, flush=True)
    A, B = _ops(7, M, K, N, True)
    assert torch.equal(_run(plan, A, B, pad=4).double(), A.double() @ B.double())
    A, B = _ops(8, M, K, N, False)
    R = A.double() @ B.double()
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    assert _err(new, R) <= _err(old, R) + 1e-7      # fewer roundings, as above
    if prec == bpx.PREC_F32:  # the panels of one element go to the FP32 kernels
        A[M - 1, 3] = float("inf")
        B[5, N // 2] = float("nan")
        new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
        fin = torch.isfinite(old)
        assert torch.equal(torch.isnan(new), torch.isnan(old))
        assert torch.equal(torch.isfinite(new), fin)
        d = torch.where(fin, new.double() - R, 0.0)
        assert float(torch.linalg.norm(d) / torch.linalg.norm(R)) <= 1e-5


# Small products on packed operands: long K on few tiles (all in pieces), the
# smallest K and sizes that are packed, and codes the fused form does not run
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("code,mode,shape", [
    ("642", bpx.MODE_FULL, (419, 3428, 373)), ("1284", bpx.MODE_FULL, (330, 196, 301)),
    ("1284", bpx.MODE_STRAGGLER, (1473, 1000, 1277)), ("moj", bpx.MODE_MIN, (1000, 212, 90)),
    ("table3", bpx.MODE_FULL, (768, 1024, 769))])
def test_small_products_on_planes(code, mode, shape, prec):
    M, K, N = shape
    lib = {"642": lambda: _code(inputs.CODE_642), "1284": lambda: _code(inputs.CODE_1284),
           "moj": lambda: bpx.Code.mojette(8, 4, 12, 1), "table3": bpx.Code.table3}[code]()
    arrival, _ = inputs.shifted_exp_arrival(0, lib.info()["n"])
    plan = bpx.Plan(lib, arrival, 0, mode, M, K, N, prec)
    assert plan.workspace_bytes()[0] > plan.workspace_layout()[6] and not plan.fused()
    print("small planes", code, shape, prec, file=sys.stderr, flush=True)
    A, B = _ops(9, M, K, N, True)
    assert torch.equal(_run(plan, A, B, pad=4).double(), A.double() @ B.double())
    A, B = _ops(10, M, K, N, False)
    R = A.double() @ B.double()
    new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
    print("  error", _err(new, R), "direct kernels", _err(old, R), file=sys.stderr, flush=True)
    assert _err(new, R) <= _err(old, R) * (1.0 if K > 256 else 1.1) + 1e-7
    small = torch.empty(max(plan.workspace_layout()[6], 256), dtype=torch.uint8, device="cuda")
    if prec == bpx.PREC_F32:
        assert _err(_run(plan, A, B, ws=small), R) <= 1e-5
        A[3, 5] = float("inf")
        new, old = _run(plan, A, B), _run(plan, A, B, tile=1)
        assert torch.equal(torch.isfinite(new), torch.isfinite(old))
        assert torch.equal(torch.isnan(new), torch.isnan(old))


# The library's own scratch (which holds the first plan's packed operands, not
# the second's: that one reads A and B directly) and a captured graph, replayed
# with other work in between; the last one sends a panel to the FP32 kernels
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("M,K,N,fits", [(419, 1028, 373, True), (2100, 2052, 1100, False)])
def test_planes_in_scratch_and_in_a_graph(M, K, N, fits, prec):
    arrival, _ = inputs.shifted_exp_arrival(0, inputs.CODE_1284.n)
    plan = bpx.Plan(_code(inputs.CODE_1284), arrival, 0, bpx.MODE_STRAGGLER, M, K, N, prec)
    print("scratch and graph", M, K, N, prec, file=sys.stderr, flush=True)
    assert (plan.workspace_bytes()[0] <= 32 << 20) == fits
    plan.upload()
    A, B = _ops(11, M, K, N, False)
    A, B = _view(A, 0), _view(B, 0)
    want = _run(plan, A, B)
    C = _view(torch.full((M, N), float("nan"), device="cuda"), 0)
    bpx.coded_matmul_noalloc(plan, A, B, C)
    torch.cuda.synchronize()
    R = A.double() @ B.double()
    assert torch.equal(C, want) if fits else _err(C, R) <= _err(want, R) * 4 + 1e-6
    ws = bpx.alloc_workspace(plan)
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            bpx.coded_matmul(plan, A, B, C, ws)
    torch.cuda.current_stream().wait_stream(s)
    for rep in range(4):
        if rep == 3:
            A[M - 1, 1] = float("inf")
            want = _run(plan, A, B)
        C.fill_(float("nan"))
        ws.fill_(0xA5)
        torch.matmul(A, B)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.nan_to_num(C), torch.nan_to_num(want)), rep
