"""The choices of the host code (which tile, which form of a stage), asked through the testing header: no device."""
import ctypes
import itertools
import random
import types

import pytest
import torch

import paper_2604_17709_amd as dn
from gpu_util import RAW_ROWS, workspace_of_eight_ranges

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


def stage(k, features, T, glu=False):
    return dn.deinfer_plan_decode_stage(T, -(-features // 32), -(-k // 32), glu, CUS)


def test_form_of_measured_decode_stages():
    """Stages that were timed in every form (us: split / one / two token blocks per workgroup)."""
    # 33 .. 64 tokens, just above 128 blocks: one round of two-block workgroups
    for k, f, T in ((1024, 4128, 48), (1024, 4480, 64), (2048, 4128, 64), (2048, 4480, 48), (1240, 4128, 40), (1240, 4480, 40)):
        assert stage(k, f, T) == 2                      # 2048 x 4480, 64 tokens: 14.4 / 14.4 / 13.1; 1240 x 4480, 40: 11.6 / 13.6 / 9.9
    assert stage(1640, 4128, 64) == 0                   # 13.4 / 15.6 / 14.0
    assert stage(256, 8192, 64) == 2                    # 11.8 / 7.1 / 5.8
    assert stage(1640, 4096, 128) == 2                  # 17.9 / 15.1 / 13.5
    assert stage(1024, 8192, 128) == 2                  # 18.4 / 15.5 / 13.9
    assert stage(512, 4096, 64) == 1                    # 12.1 / 5.7 / 6.2
    assert stage(1024, 4480, 128) == 1                  # 17.7 / 11.8 / 13.1
    assert stage(1640, 1024, 128) == 1                  # 11.5 / 8.7 / 12.4
    assert stage(4096, 2048, 128) == 1                  # 14.9 / 12.9 / 19.5
    # a last token block that is nearly empty
    assert stage(4096, 3072, 40) == 0                   # 13.2 / 14.1 / 17.2
    for k, f in ((1640, 2048), (1640, 3072), (1800, 2560), (2560, 2048), (2560, 3072)):
        assert stage(k, f, 40, glu=True) == 0           # 1640 x 3072: 12.8 / 14.7 / 16.4
    # GLU
    assert stage(512, 3584, 64, glu=True) == 1          # 12.4 / 6.3 / 8.2
    assert stage(512, 3584, 128, glu=True) == 2         # 17.4 / 8.8 / 8.1
    assert stage(1024, 4480, 64, glu=True) == 2         # 14.0 / 13.6 / 12.2
    assert stage(1640, 2048, 128, glu=True) == 1        # 18.2 / 13.5 / 20.4
    assert stage(2560, 2048, 128, glu=True) == 1        # 19.3 / 16.5 / 26.6
    assert stage(1024, 6000, 96, glu=True) == 0         # 16.6 / 18.0 / 19.7


def test_every_form_of_a_decode_stage_is_taken_by_the_rows_of_its_test():
    """... without tiles, and (where the stage chooses) by a row that is not left to tiles."""
    from test_gpu_parity import DECODE_STAGE_ROWS
    forms, chosen = set(), set()
    for T, (_, r, d_out), glu in itertools.product((9, 17, 33, 64, 65, 97, 128), DECODE_STAGE_ROWS, (False, True)):
        form = (glu, stage(r, d_out, T, glu), T > 64)
        forms.add(form)
        if dn.deinfer_plan_decode_tile(T, [d_out], -(-r // 32), glu, CUS) is None:
            chosen.add(form)
    every = {(g, f, late) for g in (False, True) for f in (0, 1, 2) for late in (False, True)}
    assert forms >= every and chosen >= every, every - chosen


def test_second_stages_that_run_as_tiles():
    """Upward projections that were timed in every form (us: other forms / tiles)."""
    def tile(k, features, T, glu=False):
        return dn.deinfer_plan_decode_tile(T, features if isinstance(features, list) else [features], -(-k // 32), glu, CUS)
    assert tile(1640, 8192, 128) == (64, 64, 2)              # 21.5 / 14.4
    assert tile(1640, [8192, 1024, 1024], 128) == (64, 96, 1)   # 23.1 / 15.7
    assert tile(512, 10240, 64) in ((32, 96, 1), (64, 128, 1))  # 13.0 / 7.6, 7.8
    assert tile(1640, 8192, 64) == (32, 64, 2)               # 15.4 / 11.8
    assert tile(1640, 8192, 128, True) == (64, 64, 1)        # 29.4 / 20.2
    assert tile(2392, 11008, 8, True) == (32, 64, 1)         # 22.2 / 21.5
    assert tile(3824, 11344, 32, True) is None               # 32.5 / 34.2
    assert tile(1968, 8748, 13) == (32, 64, 2)               # 13.0 / 11.6
    assert tile(2368, 11604, 2) == (32, 64, 2)               # 15.2 / 13.4
    assert tile(3440, 10240, 64) is None                     # 21.9 / 22.2
    assert tile(3440, 2048, 32) is None                      # 9.4 / 11.8
    assert tile(3440, 5504, 64, True) is None                # 22.3 / 27.7
    assert tile(197, 18336, 128) is None                     # 12.4 / 14.8
    assert tile(4890, 12208, 80) == (64, 96, 1)              # 49.3 / 34.2
    # one k-range per workgroup: tiles in more than one round, or whose last token block is nearly empty
    assert tile(4777, 28592, 24) is None                     # 44.1 / 49.0
    assert tile(672, 15944, 24) is None                      # 13 % slower as 32 x 64 tiles
    assert tile(1000, 13480, 37) is None                     # 10.1 / 11.4
    assert tile(736, 16024, 37) is None                      # 14 % slower as 64 x 64 tiles
    assert tile(8440, 15840, 65) is None                     # 69.6 / 84.7
    # the wide GLU form is not left, and no longer k than was timed
    assert tile(8858, 27336, 64, True) == (64, 128, 1)       # 178.9 / 194.1
    assert tile(10048, 8192, 128) is None


def test_decode_tile_query_by_compute_units():
    """The form that tiles are weighed against is planned for the compute units that are asked about, and the wide GLU form is
    among the answers."""
    def tile(features, T, k, cus):
        return dn.deinfer_plan_decode_tile(T, [features], -(-k // 32), True, cus)
    assert tile(2048, 17, 2072, 128) is None and tile(2048, 40, 2072, 128) is None      # against a split for 256 units: 32 x 32
    assert tile(28672, 128, 300, 256) == (128, 128, 1)       # 224 workgroups of 128 features


def decode_tile_call(form, kind):
    """Return code of a call of 64 tokens with the form forced, on pointers that are not real."""
    f = dn.Factors()
    f.U, f.V, f.d_in, f.d_out, f.r, f.dtype, f.layout = 1 << 28, 1 << 29, 1024, 512, 256, dn.BF16, dn.LAYOUT_PACKED
    a = ctypes.byref(f)
    L = dn.lib()
    dn.deinfer_set_decode_tile(form)
    try:
        if kind == "glu":
            return L.deinfer_lowrank_gateup_silu(1 << 30, 64, 1024, a, a, 1 << 31, 512, 1 << 32, 1 << 30, None)
        return L.deinfer_lowrank_linear(1 << 30, 64, 1024, a, 1 << 31, 512, 1 << 32, 1 << 30, None)
    finally:
        dn.deinfer_set_decode_tile(0)


def test_decode_tile_forms_that_are_not_built_are_refused():
    """... before anything is enqueued (without a device a launch would fail for that reason)."""
    if torch.cuda.is_available():
        pytest.skip("the pointers are not real")
    linear, glu = {112, 121, 122, 131, 222, 231, 241}, {111, 121, 141, 221, 241, 441}
    for form in sorted(linear | glu | {1, 12, 99, 100, 101, 110, 132, 212, 300, 331, 411, 999, 1112, 2 ** 31 - 1}):
        assert decode_tile_call(form, "linear") == (dn.ERR_DEVICE if form in linear else dn.ERR_UNSUPPORTED), form
        assert decode_tile_call(form, "glu") == (dn.ERR_DEVICE if form in glu else dn.ERR_UNSUPPORTED), form


def test_the_static_scratch_entry_takes_a_split_that_fits():
    """First stages whose best split needs more than the static array, while a smaller one (or none) fits it: not refused for
    lack of scratch (without a device the call then fails for that reason, with one it is not made here)."""
    if torch.cuda.is_available():
        pytest.skip("the pointers are not real")
    for T, d_in, r in ((375, 5608, 1249), (142, 3040, 3040), (131, 3560, 3560), (519, 5688, 522)):
        f = dn.Factors()
        f.U, f.V, f.d_in, f.d_out, f.r, f.dtype, f.layout = 1 << 28, 1 << 29, d_in, 64, r, dn.BF16, dn.LAYOUT_PACKED
        assert dn.deinfer_workspace_bytes(T, [types.SimpleNamespace(desc=f)]) > dn.STATIC_SCRATCH_BYTES
        rc = dn.lib().deinfer_lowrank_linear_static(1 << 30, T, d_in, ctypes.byref(f), 1 << 31, 64, None)
        assert rc == dn.ERR_DEVICE, dn.last_error()


def few_group_ranges(T, d_in, ranks):
    """k-ranges of the first stage of a T <= 128 call on packed pairs of few features, from the workspace it asks for: the
    partial sums against those of a short k, which takes eight."""
    def part(k):
        fs = []
        for r in ranks:
            f = dn.Factors()
            f.U, f.V, f.d_in, f.d_out, f.r, f.dtype, f.layout = 1 << 28, 1 << 29, k, 16, r, dn.BF16, dn.LAYOUT_PACKED
            fs.append(types.SimpleNamespace(desc=f))
        rows = 32 if T <= 32 else 64 if T <= 64 else 128
        return dn.deinfer_workspace_bytes(T, fs) - 256 - -(-rows * sum(-(-r // 32) * 32 for r in ranks) * 2 // 256) * 256
    assert 8 * part(d_in) % part(1024) == 0
    return 8 * part(d_in) // part(1024)


@pytest.mark.skipif(torch.cuda.is_available(), reason="sized for the 256 compute units that a machine without a device assumes")
def test_k_ranges_of_first_stages_of_few_feature_groups():
    from test_gpu_parity import FEW_GROUP_ROWS
    for T, d_in, ranks in FEW_GROUP_ROWS:
        assert few_group_ranges(T, d_in, ranks) > 8, (T, d_in, ranks)
    assert few_group_ranges(128, 8232, (400, 260)) == 8         # seven groups
    # timed with 64, 48, 32, 24, 16 and 12 k-blocks per range (us: eight ranges / as many as are taken)
    assert few_group_ranges(128, 8192, (297,)) == 16            # 15.0 / 13.7
    assert few_group_ranges(128, 11008, (299,)) == 16           # 18.6 / 15.7
    assert few_group_ranges(128, 14336, (640,)) == 16           # 21.2 / 17.4
    assert few_group_ranges(32, 14336, (640,)) == 14            # 14.8 / 13.4
    assert few_group_ranges(32, 8192, (638,)) == 8              # 11.5, 12.0 in 16
    # fewer than twelve: (9 ranges) 9.2, 10.0; 10.4, 11.2; (11) 9.1, 9.4
    assert few_group_ranges(32, 4904, (19,)) == 8
    assert few_group_ranges(33, 4960, (22, 22)) == 8
    assert few_group_ranges(9, 5912, (140,)) == 8
    assert few_group_ranges(128, 6144, (40,)) == 12 and few_group_ranges(128, 6112, (40,)) == 8


@pytest.mark.parametrize("T", [32, 64, 128])
def test_a_workspace_of_eight_ranges_is_taken(T):
    """Few feature groups and a long k: more than eight k-ranges where the workspace holds their sums, eight in a smaller one
    (without a device the call then fails for that reason; one byte less is refused)."""
    if torch.cuda.is_available():
        pytest.skip("the pointers are not real")
    f = dn.Factors()
    f.U, f.V, f.d_in, f.d_out, f.r, f.dtype, f.layout = 1 << 28, 1 << 29, 8192, 64, 297, dn.BF16, dn.LAYOUT_PACKED
    n = workspace_of_eight_ranges(dn, T, types.SimpleNamespace(desc=f))
    call = lambda ws: dn.lib().deinfer_lowrank_linear(1 << 30, T, 8192, ctypes.byref(f), 1 << 31, 64, 1 << 32, ws, None)
    assert call(n) == dn.ERR_DEVICE, dn.last_error()
    assert call(n - 1) == dn.ERR_WORKSPACE
