"""Sizes of the workspace (host only): packed operands ask for their own bytes,
for the partial tiles their split takes and, at most as much again, for those of
a card with fewer CUs, and not for the parts they do not use."""
import functools

import pytest

from paper_1904_11563_amd import bpx, inputs


def _up(x, m):
    return -(-x // m) * m


@functools.lru_cache
def _code():
    s = inputs.CODE_1284
    return bpx.Code.search(s.n, s.k, s.b, s.sigma, s.seed, s.restarts, s.iters, walk=s.walk)


def _plan(M, K, N, prec):
    arrival, _ = inputs.shifted_exp_arrival(0, 12)
    return bpx.Plan(_code(), arrival, 0, bpx.MODE_STRAGGLER, M, K, N, prec)


@pytest.mark.parametrize("prec,width", [(bpx.PREC_F32, 6), (bpx.PREC_BF16X3, 4),
                                        (bpx.PREC_BF16, 2)])
@pytest.mark.parametrize("shape", [(8192, 8192, 4096), (1999, 1500, 1001), (1024, 1024, 1024),
                                   (419, 3428, 373), (4096, 300, 8192)])
def test_packed_operands_ask_for_what_they_use(shape, prec, width):
    M, K, N = shape
    plan = _plan(M, K, N, prec)
    inf, off = plan.info(), plan.workspace_layout()
    rows = _up(inf["n_computed"] * inf["Mb"], 256) + _up(N, 256)
    packed = rows * _up(K, 32) * width
    own = off[6] if prec == bpx.PREC_F32 else off[1]   # Y, and FP32's partial tiles
    # one word per pack block and tile, alignment
    flags = 4 * (rows // 32 * (K // 64 + 2)) + 16 * (rows // 256) ** 2 + 8192
    ws = plan.workspace_bytes()[0]
    assert ws > off[6]
    assert ws <= own + packed + min(packed, 64 << 20) + flags


def test_groups_do_not_reserve_both_forms():
    plans = [_plan(2048, 2048, 2048, bpx.PREC_BF16X3) for _ in range(8)]
    need = 0
    for p in plans:
        inf, off = p.info(), p.workspace_layout()
        rows = _up(inf["n_computed"] * inf["Mb"], 256) + 2048
        need += off[1] + rows * 2048 * 4 + 512
    base = sum(_up(p.workspace_layout()[6], 256) for p in plans)
    assert base < bpx.group_workspace_bytes(plans) <= need


# Two-dimensional products on either side of the line from which they are packed:
# K over a symbol's passes, and multiply-adds
@pytest.mark.parametrize("code,mode,shape,packed", [
    ("uncoded", bpx.MODE_STRAGGLER, (1035, 256, 1568), False),
    ("uncoded", bpx.MODE_STRAGGLER, (2191, 128, 1256), False),
    ("uncoded", bpx.MODE_STRAGGLER, (649, 448, 464), True),
    ("uncoded", bpx.MODE_STRAGGLER, (5116, 128, 1744), True),
    ("uncoded", bpx.MODE_STRAGGLER, (5116, 124, 1744), False),
    ("table1", bpx.MODE_FULL, (700, 148, 704), True),     # two passes: 296
    ("table1", bpx.MODE_FULL, (700, 144, 704), False)])
def test_two_dimensional_products_are_packed_where_it_pays(code, mode, shape, packed):
    lib = bpx.Code.identity(2, 2) if code == "uncoded" else bpx.Code.table1()
    n = lib.info()["n"]
    plan = bpx.Plan(lib, list(range(n)), 0, mode, *shape, two_d=True)
    assert (plan.workspace_bytes()[0] > plan.workspace_layout()[6]) == packed
