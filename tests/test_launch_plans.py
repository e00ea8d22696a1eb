"""How the launches of a call are cut up (mlora_kernel_plan; CPU only)."""
import ctypes

import pytest

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
    bad = _problem(mb, off=(0, 40, 30))
    assert mb.lib.mlora_kernel_plan(ctypes.byref(bad.c), out) == 3
    old = mb.set_kernel_path(1)      # general base products, aligned low-rank kernels
    try:
        q = p.kernel_plan()
        assert q["Y"] in ("skinny", "64", "128") and q["Z_rows"] >= 32
    finally:
        mb.set_kernel_path(old)
    assert plan(mb, 512, 256, 320, [256, 256], [8, 16])["Y"] in ("whole", "halves", "mixed")


@pytest.mark.parametrize("T,h,d,tokens,ranks,want", [
    # full rounds of whole tiles, nothing cut
    (32768, 5120, 5120, [2048] * 16, [8, 16, 32, 64] * 4,
     dict(Y="whole", dX="whole", Y_parts=1, dX_parts=1, Z_rows=128, Z_parts=1, G_rows=128, G_parts=1, grads=1)),
    # a few short prompts: half tiles in contraction ranges
    (100, 4096, 4096, [37, 20, 43], [16] * 3, dict(Y="halves", dX="halves", Y_parts=7, Z_rows=32, Z_parts=1)),
])
def test_plans_of_known_calls(mb, T, h, d, tokens, ranks, want):  # noqa: F811
    got = plan(mb, T, h, d, tokens, ranks)
    assert {k: got[k] for k in want} == want
