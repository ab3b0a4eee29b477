"""Performance cases of the coded product: the calls a program that uses the
library makes, from the smallest product to the full-size workloads.

A case is a plain dict.  Its "call" says which entry point it takes:
  matmul    bpx.coded_matmul, plan and workspace kept between calls
  noalloc   bpx.coded_matmul_noalloc, the library's own scratch array
  two_d     bpx.coded_matmul with a two-dimensional plan (A by rows, B by columns)
  batch     bpx.Group.launch, many products of uneven shapes in one sequence
"code", "mode" and "arrival" give the code, the decode mode and the seed of the
columns' arrival order (a plan is made once per arrival order and kept, as a
program that serves many products of one arrival does); "prec" the precision;
"dist" how the operands are distributed.
"""
import math

import torch

from paper_1904_11563_amd import bpx, inputs

DEVICE = "cuda"

_SEARCHED = {"642": inputs.CODE_642, "1284": inputs.CODE_1284, "1282": inputs.CODE_1282}
_MOJETTE = {"moj": inputs.CODE_MOJ, "mojb": inputs.CODE_MOJ_B}
_codes = {}


def _code(name):
    """The code handle of a case (a search of seconds at most; one per process)."""
    if name not in _codes:
        if name in _SEARCHED:
            s = _SEARCHED[name]
            _codes[name] = bpx.Code.search(s.n, s.k, s.b, s.sigma, s.seed, s.restarts, s.iters,
                                           walk=s.walk)
        elif name in _MOJETTE:
            s = _MOJETTE[name]
            _codes[name] = bpx.Code.mojette(s.k, s.b, s.n, s.qe)
        elif name == "table1":
            _codes[name] = bpx.Code.table1()
        elif name == "table3":
            _codes[name] = bpx.Code.table3()
        else:
            raise ValueError(name)
    return _codes[name]


def _case(name, call, code, mode, arrival, prec, dist, M, K, N):
    return {"name": name, "call": call, "code": code, "mode": mode, "arrival": arrival,
            "prec": prec, "dist": dist, "M": M, "K": K, "N": N}


def listed():
    return [
        # the smallest use: Table I's worked code in a serving loop that may
        # not allocate; launches and latency are all there is
        _case("tiny_f32_noalloc", "noalloc", "table1", "straggler", 0, "f32", "uniform",
              64, 64, 64),
        # the 512^3 workloads: one product too small to fill the chip
        _case("small_f32", "matmul", "642", "erasure:2", 0, "f32", "uniform", 512, 512, 512),
        _case("small_bf16x3", "matmul", "642", "erasure:2", 0, "bf16x3", "rowscaled",
              512, 512, 512),
        # a middling product whose sizes fit no tile (odd N, K a multiple of
        # 4 only, a ragged last block)
        _case("ragged_f32", "matmul", "1284", "straggler", 1, "f32", "normal", 1999, 1500, 1001),
        # the headline workload
        _case("large_f32", "matmul", "1284", "straggler", 0, "f32", "normal", 8192, 8192, 4096),
        # Construction B at the headline's shape, a third of the columns
        # erased: nearly twice the products of an uncoded multiplication
        _case("mojette_b_f32", "matmul", "mojb", "erasure:4", 0, "f32", "normal",
              8192, 8192, 4096),
        # the two-dimensional form's workload (gray symbols included)
        _case("grid_f32", "two_d", "1282", "straggler", 0, "f32", "normal", 8192, 8192, 8192),
        # the headline's shape for a caller that takes split BF16
        _case("large_bf16x3", "matmul", "1284", "straggler", 0, "bf16x3", "normal",
              8192, 8192, 4096),
        # plain BF16, every virtual worker computed, sizes that fit no tile
        _case("ragged_bf16", "matmul", "642", "full", 0, "bf16", "normal", 3000, 2060, 1530),
        # the block-scaled FP8 workload and a ragged product of the one-term form
        _case("mojette_fp8x2", "matmul", "moj", "erasure:8", 0, "fp8x2", "normal",
              16384, 16384, 8192),
        _case("ragged_fp8", "matmul", "moj", "erasure:8", 1, "fp8", "normal", 5000, 3000, 2000),
        # the batch workload: 256 products, each with its own code and arrival
        {"name": "batch_bf16x3", "call": "batch", "prec": "bf16x3", "count": 256, "shapes": 0},
    ]


def _log_int(rng, lo, hi, mult=1):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(x / mult) * mult, -(-lo // mult) * mult), hi // mult * mult)


def draw(rng):
    kind = rng.choice(["f32", "f32", "bf16x3", "bf16", "fp8", "two_d", "batch", "tiny"])
    arrival = rng.randrange(1000)
    if kind == "batch":
        return {"call": "batch", "prec": rng.choice(["bf16x3", "bf16x3", "bf16"]),
                "count": _log_int(rng, 16, 256), "shapes": rng.randrange(1000)}
    if kind == "tiny":
        c = _case("", "noalloc", rng.choice(["table1", "table3", "642"]), "straggler", arrival,
                  rng.choice(["f32", "bf16x3", "bf16"]), "uniform", _log_int(rng, 32, 640),
                  _log_int(rng, 32, 640, 4), _log_int(rng, 32, 640))
    elif kind == "two_d":
        c = _case("", "two_d", rng.choice(["table1", "1282"]),
                  rng.choice(["straggler", "straggler", "min"]), arrival, "f32", "normal",
                  _log_int(rng, 512, 8192), _log_int(rng, 512, 8192, 4),
                  _log_int(rng, 512, 8192, 16))
    elif kind == "fp8":
        c = _case("", "matmul", "moj", "erasure:8", arrival, rng.choice(["fp8", "fp8x2"]),
                  "normal", _log_int(rng, 2048, 16384), _log_int(rng, 1024, 16384, 4),
                  _log_int(rng, 1024, 8192))
    else:
        code = rng.choice(["642", "1284", "1284", "mojb"])
        mode = "erasure:4" if code == "mojb" else rng.choice(["straggler", "straggler", "full",
                                                              "min"])
        c = _case("", "matmul", code, mode, arrival, kind,
                  rng.choice(["normal", "uniform", "rowscaled"]), _log_int(rng, 300, 8192),
                  _log_int(rng, 300, 8192, 4), _log_int(rng, 300, 4096))
    del c["name"]
    return c


# --------------------------------------------------------------- operands --

def _random(dist, shape, gen, rows=False):
    if dist == "normal":
        return torch.randn(shape, generator=gen, device=DEVICE)
    x = torch.rand(shape, generator=gen, device=DEVICE) * 2 - 1
    if dist == "rowscaled" and rows:   # rows scaled log-uniformly over [1e-3, 1e3]
        e = torch.rand((shape[0], 1), generator=gen, device=DEVICE) * 2 - 1
        x = x * torch.exp(e * math.log(1e3))
    return x


def _aligned(x):
    """x as a view whose row stride is a multiple of 4 (the library's rule)."""
    r, c = x.shape
    if c % 4 == 0:
        return x
    buf = torch.zeros((r, -(-c // 4) * 4), device=DEVICE)
    buf[:, :c] = x
    return buf[:, :c]


def _empty(M, N):
    return torch.empty((M, -(-N // 4) * 4), device=DEVICE)[:, :N]


def _operands(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    A = _random(case["dist"], (case["M"], case["K"]), gen, rows=True)
    B = _random(case["dist"], (case["K"], case["N"]), gen)
    return A, B


def _batch_shapes(case):
    return inputs.batch_shapes(case["shapes"], case["count"])


def _batch_operands(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    for M, K, N, _ in _batch_shapes(case):
        yield (torch.randn((M, K), generator=gen, device=DEVICE),
               torch.randn((K, N), generator=gen, device=DEVICE))


# ------------------------------------------------------------------ plans --

def _plan(case):
    code = _code(case["code"])
    n = code.info()["n"]
    mode, lost = case["mode"], 0
    if mode.startswith("erasure:"):
        mode, lost = "erasure", int(mode.split(":")[1])
        arrival, _ = inputs.erasure_arrival(case["arrival"], n, lost)
    else:
        arrival, _ = inputs.shifted_exp_arrival(case["arrival"], n)
    return bpx.Plan(code, arrival, lost, bpx.MODE_NAMES[mode], case["M"], case["K"], case["N"],
                    bpx.PREC_NAMES[case["prec"]], two_d=case["call"] == "two_d")


def _batch_plans(case):
    plans = []
    for i, (M, K, N, k) in enumerate(_batch_shapes(case)):
        code = _code("642" if k == 4 else "1282")
        n = code.info()["n"]
        arrival, _ = inputs.erasure_arrival(case["shapes"] * 1000 + i, n, n - k)
        plans.append(bpx.Plan(code, arrival, 0, bpx.MODE_STRAGGLER, M, K, N,
                              bpx.PREC_NAMES[case["prec"]]))
    return plans


def prepare(case, seed):
    if case["call"] == "batch":
        plans = _batch_plans(case)
        ops = list(_batch_operands(case, seed))
        As, Bs = [a for a, _ in ops], [b for _, b in ops]
        # the results of a batch share one buffer, product after product
        out = torch.empty(sum(p.M * p.N for p in plans), device=DEVICE)
        Cs, at = [], 0
        for p in plans:
            Cs.append(out[at:at + p.M * p.N].view(p.M, p.N))
            at += p.M * p.N
        ws = torch.empty(bpx.group_workspace_bytes(plans), dtype=torch.uint8, device=DEVICE)
        return {"call": "batch", "group": bpx.Group(plans, As, Bs, Cs, ws), "out": out}
    plan = _plan(case)
    plan.upload()
    A, B = _operands(case, seed)
    state = {"call": case["call"], "plan": plan, "A": _aligned(A), "B": _aligned(B),
             "C": _empty(case["M"], case["N"])}
    if case["call"] != "noalloc":
        state["ws"] = bpx.alloc_workspace(plan)
    return state


def run(state):
    if state["call"] == "batch":
        state["group"].launch()
        return state["out"]
    if state["call"] == "noalloc":
        bpx.coded_matmul_noalloc(state["plan"], state["A"], state["B"], state["C"])
    else:
        bpx.coded_matmul(state["plan"], state["A"], state["B"], state["C"], state["ws"])
    return state["C"]


# ---------------------------------------------------------- work and exact --

def _passes(plan, code):
    """Products over K of a two-dimensional plan: a symbol whose members share
    neither an A block nor a B block takes one pass per member."""
    grid, _ = plan.grid()
    _, sym_ptr, sym_data = code.csr()
    total = 0
    for g in plan.schedule()["computed"].tolist():
        ids = [int(x) for x in sym_data[sym_ptr[g]:sym_ptr[g + 1]]]
        one = len({s // grid for s in ids}) == 1 or len({s % grid for s in ids}) == 1
        total += 1 if one else len(ids)
    return total


def _product_work(plan, products, M, K, N, width):
    return {"bytes": 4 * (M * K + K * N + M * N),
            "flops": 2 * plan.info()["Mb"] * K * width * products}


def work(case):
    """A, B and C once each; the coded products of every computed symbol."""
    if case["call"] == "batch":
        total = {"bytes": 0, "flops": 0}
        for plan in _batch_plans(case):
            w = _product_work(plan, plan.info()["n_computed"], plan.M, plan.K, plan.N, plan.N)
            total = {k: total[k] + w[k] for k in total}
        return total
    plan = _plan(case)
    M, K, N = case["M"], case["K"], case["N"]
    if case["call"] == "two_d":
        return _product_work(plan, _passes(plan, _code(case["code"])), M, K, N, plan.grid()[1])
    return _product_work(plan, plan.info()["n_computed"], M, K, N, N)


def exact(case, seed):
    """A.B in float64."""
    if case["call"] == "batch":
        return torch.cat([(a.double() @ b.double()).flatten()
                          for a, b in _batch_operands(case, seed)])
    A, B = _operands(case, seed)
    return A.double() @ B.double()
