"""The choices of the host code (which tile, which form of a stage), asked through the testing header: no device."""
import itertools
import random
import types

import pytest
import torch

import paper_2604_17709_amd as dn
from gpu_util import RAW_ROWS

CUS = 256
DTYPES = {"f32": dn.F32, "bf16": dn.BF16, "f16": dn.F16}
WIDE = {(64, 64), (32, 64)}
SMALL = {(64, 32), (32, 32), (16, 32), (16, 16)}


def raw(M, N, K, dtype="f32", rows4=True, dual=False, cus=CUS):
    return dn.deinfer_plan_raw_tile(M, N, K, DTYPES[dtype], rows4, dual, cus)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows4,dual", [(True, False), (False, False), (True, True)])
def test_every_raw_tile_is_taken_somewhere(dtype, rows4, dual):
    rng = random.Random(5)
    seen = {raw(rng.randint(1, 2048), rng.randint(1, 4096), rng.randint(1, 4096), dtype, rows4, dual)[:2] for _ in range(4000)}
    assert seen == SMALL | (WIDE if rows4 and not dual else set())


def test_raw_tile_of_measured_products():
    """The fastest tile of products that were timed with each of the six."""
    assert raw(201, 1638, 4096) == (64, 32, 4)
    assert raw(201, 1638, 1638) == (64, 32, 4)
    assert raw(201, 4096, 1638) == (64, 64, 4)
    assert raw(201, 4096, 4096) == (64, 64, 4)
    assert raw(1024, 300, 4096) == (64, 32, 4)
    assert raw(512, 819, 4096, rows4=False) == (64, 32, 4)
    assert raw(201, 1638, 1638, "bf16") == (16, 32, 4)
    # 16 wavefronts per tile: from k = 4096 on, few tiles
    assert raw(16, 300, 1638) == (16, 16, 4) and raw(16, 300, 700) == (16, 16, 4)
    assert raw(1, 64, 4096) == (16, 16, 16) and raw(16, 300, 4096, "bf16") == (16, 16, 16)
    assert raw(16, 1638, 4096, "bf16")[2] == 4


def test_rows_of_the_raw_tile_test_take_every_tile():
    for dtype in ("f32", "bf16"):
        first, second, pairs = set(), set(), set()
        for (T, d_in, r, d_out), pad in itertools.product(RAW_ROWS, (0, 3)):
            rows4 = lambda n: pad == 0 and n % 4 == 0
            first.add(raw(T, r, d_in, dtype, rows4(r)))
            second.add(raw(T, d_out, r, dtype, rows4(d_out)))
            pairs.add(raw(T, d_out, r, dtype, rows4(d_out), dual=True))
        small = {t + (4,) for t in SMALL} | {(16, 16, 16)}
        assert first | second == small | {t + (4,) for t in WIDE}
        assert (16, 16, 16) in first and (16, 16, 16) in second
        assert pairs == small


def first_stage_parts(T, d_in, r):
    """k-parts of the first stage of a T > 128 call on one packed pair, from the workspace it asks for."""
    f = dn.Factors()
    f.U, f.V, f.d_in, f.d_out, f.r, f.dtype, f.layout = 1 << 28, 1 << 29, d_in, 4096, r, dn.BF16, dn.LAYOUT_PACKED
    up = lambda v, m: -(-v // m) * m
    part = dn.deinfer_workspace_bytes(T, [types.SimpleNamespace(desc=f)]) - 256 - up(up(T, 256) * up(r, 32) * 2, 256)
    one = -(-T // 256) * 256 * -(-up(r, 32) // 256) * 256 * 4
    assert part % one == 0
    return part // one


@pytest.mark.skipif(torch.cuda.is_available(), reason="sized for the 256 compute units that a machine without a device assumes")
def test_first_stages_are_split_where_that_was_faster():
    # timed with every number of parts (us whole, us in parts)
    assert first_stage_parts(1024, 2048, 1228) == 0         # 30.0, 43.1 in 5
    assert first_stage_parts(1536, 2048, 614) == 0          # 25.5, 37.8 in 5
    assert first_stage_parts(2048, 2048, 256) == 0          # 22.8, 32.7 in 8
    assert first_stage_parts(512, 2048, 2548) == 0          # 40.7, 51.3 in 5
    assert first_stage_parts(2048, 4096, 1228) == 0         # 44.4, 53.8 in 5
    assert first_stage_parts(4096, 4096, 4096) == 0         # 128.9, 182.0 in 2
    assert first_stage_parts(512, 11008, 1638) >= 10        # 99.7, 55.6 in 16
    assert first_stage_parts(1024, 28672, 3072) in (4, 5)   # 270.9, 184.6 in 4
    assert first_stage_parts(384, 4096, 1228) >= 8          # 47.8, 40.0 in 16
