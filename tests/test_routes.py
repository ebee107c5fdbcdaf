"""Which kernels long bf16 launches take (no GPU): a launch of many short heads is long as a whole, but its workgroups walk one head at a
time, and the second pass with the keys in registers is the slower one there (figures at its rule)."""
import pytest

from paper_2510_20707_amd import binding as B
from tests import routes
from tests import test_gpu_gather as gather

UNITS = 1024


def _second(tiles, d, n, units=UNITS):
    p = B.make_params("bf16", units // 8, 4 * tiles, 4, d, n, 32, 64)
    return routes.passes(p, 2)[1]


@pytest.mark.parametrize("tiles,d,least", [(2, 128, 4096), (3, 128, 4096), (4, 128, 1536), (5, 128, 1536), (6, 128, 1536), (7, 128, 4096),
                                           (8, 128, 1024), (3, 64, 1536), (8, 64, 1536), (9, 64, 512), (13, 64, 512), (16, 64, 512)])
def test_heads_too_short_for_keys_in_registers(tiles, d, least):
    # every launch here is beyond 16 chunks per compute unit, and no wave of it idle if blocks were dealt over the whole launch
    for n in (320, 384, 512, 550, 640, 704, 768, 1024, 1536, 2048, 3072, 4096, 8192):
        units = UNITS * max(2, 1024 // n)
        # a second round of the eight waves with one or two 64-key blocks
        idle = d == 64 and (tiles > 12 and n == 550 or tiles > 14 and n == 640)
        assert _second(tiles, d, n, units) == ("kst_attn" if n >= least and not idle else "attn"), n


def test_few_tiles_need_longer_launches():
    # 4096 keys per head, 16 and 24 chunks of 128 keys per compute unit
    assert _second(3, 128, 4096, 128) == "attn" and _second(3, 128, 4096, 192) == "kst_attn"
    assert _second(4, 128, 4096, 128) == "kst_attn"
    # 6 tiles, 30 blocks of 64 keys per head: from 32 chunks on; 31 blocks: from 16 on
    assert _second(6, 128, 1900, 512) == "attn" and _second(6, 128, 1900, 1024) == "kst_attn"
    assert _second(6, 128, 1970, 512) == "kst_attn"


def test_only_shapes_the_kernels_are_written_for():
    assert _second(9, 128, 8192) == "attn"
    for dtype, hq, d, want in (("f32", 28, 128, ("stats", "attn")), ("bf16", 4, 128, ("ks_stats", "ks_attn")), ("bf16", 36, 128, ("stats", "attn"))):
        assert routes.passes(B.make_params(dtype, 16, hq, 4, d, 8192, 32, 64), 8) == want
    p = B.make_params("bf16", 16, 28, 4, 128, 8192, 32, 64)
    assert routes.passes(p, 8) == ("qs_stats", "kst_attn")
    assert routes.passes(p, 8, stride_n=1 << 25)[0] == "stats"          # the first pass forms 32-bit offsets inside a tile


@pytest.mark.parametrize("dtype,most", [("bf16", 32), ("f32", 8)])
def test_decode_rows_read_by_several_workgroups_stay_cached(dtype, most):
    # up to `most` query heads per KV head one workgroup serves them all and the rows are read once
    for g in (1, 7, most, most + 1, 2 * most, 2 * most + 1, 256):
        assert routes.decode_reads_once(g, dtype) == (g <= most), g


@pytest.mark.parametrize("dtype,d,alone", [("bf16", 64, 256), ("f32", 64, 256), ("f32", 128, 256), ("bf16", 128, 180)])
def test_keys_that_the_second_pass_reads_again_stay_cached(dtype, d, alone):
    # one query tile, eight layers; keys and values from 180 MB on, keys alone from `alone` MB on
    row = d * (2 if dtype == "bf16" else 4)
    for mb in (170, 190, 220, 250, 260, 300):
        units = round(mb * 1e6 / (1000 * row * 8))
        make = lambda n, intrinsic: B.make_params(dtype, units, 1, 1, d, n, 32, 64, intrinsic=intrinsic)  # noqa: E731
        assert routes.few_rows_read_once(make(1000, "knorm"), 8) == (mb > alone), mb
        assert routes.few_rows_read_once(make(500, "vnorm"), 8) == (mb > 180), mb
    units = round(200e6 / (400 * row * 8))               # short heads
    assert not routes.few_rows_read_once(B.make_params(dtype, units, 1, 1, d, 400, 32, 64, intrinsic="none"), 8)


def test_gather_cases_are_on_the_side_that_they_are_meant_for():
    for want, cases, tables in ((False, gather.INSIDE, gather.TABLE_INSIDE), (True, gather.APART, gather.TABLE_APART)):
        for dtype, d, n, w, hkv, budget in cases:
            assert routes.gathers_apart(B.make_params(dtype, 1, hkv, hkv, d, n, w, budget), 1, budget) == want, (dtype, d, budget)
        for hkv, budget, top in tables:
            assert routes.gathers_apart(B.make_params("bf16", 1, hkv, hkv, 64, 2000, 8, budget), 1, top) == want, (hkv, top)
