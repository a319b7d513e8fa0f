"""The choices of the host code (which tile, which form of a stage), asked through the testing header: no device."""
import itertools
import random

import pytest

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
