"""How the launches of a call are cut up (mlora_kernel_plan; CPU only)."""
import ctypes

import pytest

from tests import form_cases
from tests.test_host_abi import _problem, mb  # noqa: F401  (mb is a fixture)


def plan(mb, T, h, d, tokens, ranks, lead=0, f32=False):  # noqa: F811
    off = [lead]
    for t in tokens:
        off.append(off[-1] + t)
    p = _problem(mb, T=T, h=h, d=d, off=tuple(off), ranks=tuple(ranks), s=(1.0,) * len(ranks))
    if f32:
        p.c.dtype = mb.MLORA_F32
    return p.kernel_plan()


def test_plan_query(mb):  # noqa: F811
    p = _problem(mb, T=512, h=256, d=320, off=(0, 256, 512), ranks=(8, 16))
    out = (ctypes.c_int32 * len(mb.PLAN_FIELDS))()
    assert mb.lib.mlora_kernel_plan(ctypes.byref(p.c), out) == 0
    assert mb.lib.mlora_kernel_plan(ctypes.byref(p.c), None) == 1
    assert mb.lib.mlora_kernel_plan(None, out) == 1
    tiles = (ctypes.c_int32 * len(mb.PLAN_TILES))()
    assert mb.lib.mlora_kernel_plan_tiles(ctypes.byref(p.c), tiles) == 0
    assert mb.lib.mlora_kernel_plan_tiles(ctypes.byref(p.c), None) == 1
    assert mb.lib.mlora_kernel_plan_tiles(None, tiles) == 1
    bad = _problem(mb, off=(0, 40, 30))
    assert mb.lib.mlora_kernel_plan(ctypes.byref(bad.c), out) == 3
    assert mb.lib.mlora_kernel_plan_tiles(ctypes.byref(bad.c), tiles) == 3
    old = mb.set_kernel_path(1)      # general base products, aligned low-rank kernels
    try:
        q = p.kernel_plan()
        assert q["Y"] in ("skinny", "64", "128") and q["Z_rows"] >= 32
    finally:
        mb.set_kernel_path(old)
    assert plan(mb, 1100, 1024, 4096, [500, 600], [8, 16])["Y"] in ("whole", "halves", "mixed")


def group_plan(mb, T, h, ds, tokens, ranks, lead):  # noqa: F811
    off = [lead]
    for t in tokens:
        off.append(off[-1] + t)
    return mb.Group([_problem(mb, T=T, h=h, d=d, off=tuple(off), ranks=tuple(r), s=(1.0,) * len(r))
                     for d, r in zip(ds, ranks)]).kernel_plan()


def test_group_plan_query(mb):  # noqa: F811
    ps = [_problem(mb, T=512, h=256, d=d, off=(0, 256, 512), ranks=(8, 16)) for d in (320, 64)]
    g, out = mb.Group(ps), (ctypes.c_int32 * len(mb.PLAN_GROUP))()
    assert mb.lib.mlora_kernel_plan_group(g.c, 2, out) == 0
    assert mb.lib.mlora_kernel_plan_group(g.c, 2, None) == 1
    assert mb.lib.mlora_kernel_plan_group(None, 2, out) == 1
    assert mb.lib.mlora_kernel_plan_group(g.c, 0, out) == 2
    # a group of one is the plain call
    one = mb.Group(ps[:1]).kernel_plan()
    assert one == {k: ps[0].kernel_plan()[k] for k in one}


@pytest.mark.parametrize("case", form_cases.GROUPS)
def test_groups_of_the_gpu_tests_take_their_forms(mb, case):  # noqa: F811
    *sizes, want = case
    got = group_plan(mb, *sizes)
    assert {k: got[k] for k in want} == want


# features that are multiples of 64 or not, aligned or general: a name means one kernel
@pytest.mark.parametrize("dtype,sizes,form,rows", [
    ("bf16", (1100, 1024, 1024), "ring", 64), ("bf16", (600, 1016, 520), "ring", 64), ("bf16", (600, 1018, 518), "64", 64),
    ("f32", (900, 1024, 1024), "64", 64), ("bf16", (128, 256, 256), "skinny", 16), ("f32", (128, 256, 256), "skinny", 16),
    ("bf16", (1100, 2048, 5632), "halves", 128), ("bf16", (2000, 2056, 5640), "whole", 256)])
def test_form_names(mb, dtype, sizes, form, rows):  # noqa: F811
    got = plan(mb, *sizes, [sizes[0]], [8], f32=dtype == "f32")
    assert (got["Y"], got["Y_rows"]) == (form, rows)


@pytest.mark.parametrize("T,h,d,tokens,ranks,want", [
    # full rounds of whole tiles, nothing cut
    (32768, 5120, 5120, [2048] * 16, [8, 16, 32, 64] * 4,
     dict(Y="whole", dX="whole", Y_parts=1, dX_parts=1, Z_rows=128, Z_parts=1, G_rows=128, G_parts=1, grads=1)),
    # a few short prompts: small tiles, whatever the size of the weight
    (100, 4096, 4096, [37, 20, 43], [16] * 3, dict(Y="ring", dX="ring", Z_rows=32, Z_parts=1)),
    (32, 4096, 11008, [32], [16], dict(Y="ring", dX="ring")),
    (8, 2048, 8192, [8], [16], dict(Y="ring", dX="ring")),
    (30, 9752, 6144, [14, 16], [64, 8], dict(Y="ring", dX="ring")),
    (25, 1824, 10296, [12, 13], [16, 16], dict(Y="ring", dX="ring")),
    # ... half tiles in ranges for more rows
    (256, 11008, 4096, [85, 85, 86], [16] * 3, dict(Y="halves")),
    (300, 13824, 5120, [100] * 3, [32] * 3, dict(Y="halves", dX="halves")),
    (512, 4096, 4096, [170, 170, 172], [16] * 3, dict(Y="halves", dX="halves")),
    # ... also with features that are multiples of 8, whose ranges have room in the workspace as well
    (366, 6496, 11920, [73, 293], [2, 2], dict(dX="halves", dX_parts=2)),
    (500, 4104, 4104, [200, 300], [16, 16], dict(Y="halves", Y_parts=2, dX="halves", dX_parts=2)),
    (700, 8200, 2056, [300, 400], [16, 16], dict(Y="halves", Y_parts=4)),
    # small tiles beyond 64 tiles of 256 x 256
    (2740, 368, 1600, [130, 123, 21, 273, 336, 190, 92, 125, 379, 551, 105, 415], [16, 64, 32] * 4, dict(Y="ring")),
    (3191, 504, 1232, [1600, 1591], [32, 16], dict(Y="ring")),
    (3000, 512, 2944, [3000], [16], dict(Y="whole")),
    # between three and four small tiles per CU: the general kernel's, unless the features are multiples of 64
    (641, 200, 4504, [200, 200, 241], [64, 8, 16], dict(Y="64")),
    (1500, 392, 2136, [500] * 3, [64, 16, 32], dict(Y="64")),
    (1500, 456, 2136, [500] * 3, [64, 16, 32], dict(Y="ring")),
    (641, 192, 4544, [200, 200, 241], [64, 8, 16], dict(Y="ring")),
    (300, 200, 8008, [100] * 3, [64, 8, 16], dict(Y="ring")),
    (4291, 64, 1536, [656, 69, 1776, 1044, 16, 411, 319], [67, 3, 1, 5, 2, 81, 9], dict(Y="halves")),
])
def test_plans_of_known_calls(mb, T, h, d, tokens, ranks, want):  # noqa: F811
    got = plan(mb, T, h, d, tokens, ranks)
    assert {k: got[k] for k in want} == want


def test_tiles_of_the_aligned_products(mb):  # noqa: F811
    def tiles(*a):
        p = plan(mb, *a)
        return p["Y"], p["Y_whole"], p["Y_tiles"]
    assert tiles(16384, 4096, 4096, [16384], [16]) == ("whole", 1024, 1024)
    assert tiles(1100, 1024, 4096, [1100], [16]) == ("halves", 0, 80)
    assert tiles(4300, 1024, 4096, [2100, 2050], [16, 24], 50) == ("mixed", 256, 288)


@pytest.mark.parametrize("T,inner,rank,parts", [
    (16384, 512, 64, 1), (12288, 1024, 8, 1), (8192, 3072, 64, 1),     # shallow: the ranges' sums outweigh them
    (16384, 4096, 8, 1),
    (8192, 4096, 16, 4), (16448, 11008, 64, 4), (2048, 11008, 32, 8),  # deep
    (2048, 512, 128, 1), (16384, 1024, 128, 1),                        # ranks above 64, shallow
    (2048, 1024, 128, 4), (3072, 4096, 128, 8), (8192, 2048, 128, 4),
])
def test_contraction_ranges_of_low_rank_rows(mb, T, inner, rank, parts):  # noqa: F811
    assert plan(mb, T, inner, 64, [T], [rank])["Z_parts"] == parts
    assert plan(mb, T, 64, inner, [T], [rank])["G_parts"] == parts


@pytest.mark.parametrize("T,h,d,K,form", [
    (4000, 4, 2000, 4, "128"), (700, 4, 2000, 1, "64"),     # more blocks than a round: tiles
    (300, 4, 2000, 4, "skinny"), (128, 256, 256, 2, "skinny"),
    (40000, 50, 50, 1, "skinny"),                           # ... but one column block
])
def test_forms_of_shallow_base_products(mb, T, h, d, K, form):  # noqa: F811
    assert plan(mb, T, h, d, [T // K] * K, [4] * K, f32=True)["Y"] == form
    assert plan(mb, T, d, h, [T // K] * K, [4] * K, f32=True)["dX"] == form


@pytest.mark.parametrize("dtype,T,inner,outer,rank,parts", [
    # 64 x 64 tiles: contraction ranges on both sides of the estimate
    ("f32", 500, 2048, 2048, 8, 2), ("f32", 600, 2048, 2048, 8, 3), ("f32", 800, 2048, 2048, 8, 1),
    ("f32", 300, 1024, 1024, 8, 6), ("f32", 600, 1024, 1024, 8, 3), ("f32", 800, 1024, 1024, 8, 1),
    ("bf16", 150, 3000, 300, 2, 10), ("bf16", 900, 2050, 1500, 8, 1), ("bf16", 512, 1500, 2050, 8, 1),
    # high ranks, whose LoRA terms share the CUs of the last ranges
    ("f32", 500, 1000, 1000, 16, 4), ("f32", 500, 1000, 1000, 128, 2), ("f32", 500, 2000, 700, 128, 5),
    ("bf16", 300, 1500, 1500, 128, 1),
])
def test_contraction_ranges_of_general_products(mb, dtype, T, inner, outer, rank, parts):  # noqa: F811
    want = ("64", parts)
    got = plan(mb, T, inner, outer, [T], [rank], f32=dtype == "f32")
    assert (got["Y"], got["Y_parts"]) == want and got["Y_whole"] == got["Y_tiles"]
    got = plan(mb, T, outer, inner, [T], [rank], f32=dtype == "f32")
    assert (got["dX"], got["dX_parts"]) == want and got["dX_whole"] == got["dX_tiles"]


def test_short_tasks_keep_one_range(mb):  # noqa: F811
    assert plan(mb, 4096, 4096, 4096, [64] * 64, [8] * 64)["Z_parts"] == 1
    assert plan(mb, 4096, 4096, 4096, [128] * 32, [8] * 32)["Z_parts"] == 4


@pytest.mark.parametrize("dtype,case,want", [(t, c, w) for c, w in form_cases.GENERAL for t in ("f32", "bf16")] +
                         form_cases.QUARTERS + form_cases.EDGE_QUARTERS +
                         [("bf16", c, w) for c, w in form_cases.HALVES + form_cases.SPLIT_ROWS + form_cases.WHOLE_TILES +
                          form_cases.LANES] +
                         [(t, c, w) for t, c, w, _ in form_cases.ISOLATION])
def test_sizes_of_the_gpu_tests_take_their_forms(mb, dtype, case, want):  # noqa: F811
    T, h, d, tokens, ranks, lead = case
    got = plan(mb, T, h, d, tokens, ranks, lead, f32=dtype == "f32")
    assert {k: got[k] for k in want} == want
