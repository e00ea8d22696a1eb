"""bf16 base products in small tiles, and with a last, partial contraction tile (features that are multiples of 8
but not of 64), and low-rank products of few rows in contraction ranges, at the sizes of small_tile_cases.py."""
import pytest
import torch

from tests.small_tile_cases import APART, CASES, PACKED, ROWS, SMALL_BACK
from tests.test_host_abi import mb  # noqa: F401  (a fixture)
from tests.test_launch_plans import plan


@pytest.mark.parametrize("case,want", CASES)
def test_sizes_take_their_forms(mb, case, want):  # noqa: F811
    T, h, d, tokens, ranks, lead = case
    got = plan(mb, T, h, d, tokens, ranks, lead)
    assert {k: got[k] for k in want} == want


@pytest.mark.parametrize("dtype,case,want", ROWS + PACKED)
def test_few_rows_sizes_take_their_forms(mb, dtype, case, want):  # noqa: F811
    T, h, d, tokens, ranks, lead = case
    got = plan(mb, T, h, d, tokens, ranks, lead, f32=dtype == "f32")
    assert {k: got[k] for k in want} == want


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,case", [(t, c) for t, c, _ in ROWS + PACKED])
def test_few_rows_forms(dtype, case):
    from tests.parity_util import TOL, check_full, run_hip
    from tests.test_gpu_general import _inputs
    T, h, d, tokens, ranks, lead = case
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    inp = _inputs(T, h, d, tokens, ranks, dt, lead=lead, seed=93)
    check_full(inp, run_hip(inp), TOL[dt], label=f"few rows {dtype} {case[:3]}")


@pytest.mark.gpu
@pytest.mark.parametrize("case", [c for c, _ in CASES])
def test_small_tile_forms(case):
    from tests.parity_util import TOL, check_full, run_hip
    from tests.test_gpu_general import _inputs
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=90)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"small tiles {case}")


# one task's adapter and rows are not finite: every other task's results keep their bits (the task whose rows
# share tiles with two neighbours)
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (2900, 704, 192, [31, 33, 95, 97, 160, 2461], [8, 16, 33, 127, 5, 128], 17),
    (220, 1920, 2688, [22] * 9 + [21], [64] * 10, 0),
    (600, 1016, 520, [63, 65, 1, 300], [8, 32, 33, 64], 3),
    (128, 256, 256, [20, 20, 20, 60], [8, 64, 16, 9], 4),
    (9268, 1032, 136, [4000, 33, 5000], [128, 8, 33], 20),
    PACKED[0][1], PACKED[5][1],
])
def test_small_tile_isolation(case):
    from tests.parity_util import run_hip
    from tests.test_gpu_general import _inputs
    T, h, d, tokens, ranks, lead = case
    k = 1
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=91)
    ref = run_hip(inp)
    lo, hi = inp.seg_offsets[k], inp.seg_offsets[k + 1]
    inp.A[k].fill_(float("nan"))
    inp.B[k].fill_(float("inf"))
    for big, value in ((inp.X, "nan"), (inp.dY, "inf")):
        big[lo:hi:2] = float(value)
        big[lo + 1:hi:2] = -float("inf")
    out = run_hip(inp)
    for name in ("Y", "dX"):
        a, b = ref[name].view(torch.int16), out[name].view(torch.int16)
        assert torch.equal(a[:lo], b[:lo]) and torch.equal(a[hi:], b[hi:]), name
    for name in ("dA", "dB"):
        for i in range(len(ranks)):
            assert i == k or torch.equal(ref[name][i], out[name][i]), (name, i)


# projections that share their input: the summed dX in small tiles of two and four operand pairs, with partial
# contraction tiles
@pytest.mark.gpu
@pytest.mark.parametrize("h,ds", [(512, [512, 256]), (520, [712, 264, 1000, 72]), (1024, [512, 512, 1032])])
def test_small_tile_groups(h, ds):
    from tests.test_gpu_groups import _group_inputs, check_group, run_group
    from tests.parity_util import TOL
    ins = _group_inputs(500, h, ds, [100, 197, 170], [[16, 8, 64]] * len(ds), torch.bfloat16, lead=3, seed=92)
    check_group(ins, run_group(ins), TOL[torch.bfloat16])


# ... of packed rows in the general kernel
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_packed_group(dtype):
    from tests.test_gpu_groups import _group_inputs, check_group, run_group
    from tests.parity_util import TOL
    T, _, _, tokens, _, lead = PACKED[2][1]
    ins = _group_inputs(T, 1001, [385, 1500], tokens, [[1 + k % 9 for k in range(len(tokens))]] * 2, dtype, lead=lead, seed=94)
    check_group(ins, run_group(ins), TOL[dtype])


@pytest.mark.parametrize("dtype,case,want", SMALL_BACK + APART)
def test_small_backward_takes_its_form(mb, dtype, case, want):  # noqa: F811
    T, h, d, tokens, ranks, lead = case
    got = plan(mb, T, h, d, tokens, ranks, lead, f32=dtype == "f32")
    assert {k: got[k] for k in want} == want


# small backward calls, whose dX and gradients share a launch; overwriting, and adding to the gradients
# groups of such projections, whose gradients share launches in pairs: one range, several, projections in larger tiles
# between them, ranks above the others'
GROUPS = [
    ("f32", 500, 300, [700, 120, 1001], [100, 0, 390], [[17, 4, 8], [3, 16, 1], [64, 9, 30]]),
    ("bf16", 913, 999, [1500, 300], [300, 77, 513], [[8, 10, 16], [40, 3, 64]]),
    ("bf16", 1300, 512, [512, 4096, 64, 128], [700, 590], [[8, 32], [16, 3], [20, 20], [1, 5]]),
    ("bf16", 400, 704, [640, 5120, 128], [200, 196], [[8, 16], [16, 16], [9, 30]]),
]


@pytest.mark.parametrize("dtype,T,h,ds,tokens,ranks", GROUPS)
def test_small_groups_share_launches(mb, dtype, T, h, ds, tokens, ranks):  # noqa: F811
    plans = [plan(mb, T, h, d, tokens, r, 3, f32=dtype == "f32") for d, r in zip(ds, ranks)]
    assert sum(p["shared"] for p in plans) > 1, [(p["shared"], p["grads"]) for p in plans]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,T,h,ds,tokens,ranks", GROUPS)
def test_small_groups(dtype, T, h, ds, tokens, ranks):
    """The gradients against the oracle, bit for bit those of single calls, and added to what is there."""
    from tests.parity_util import TOL, run_hip
    from tests.test_gpu_groups import _group_inputs, check_group, run_group
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    ins = _group_inputs(T, h, ds, tokens, ranks, dt, lead=3, seed=96)
    out = run_group(ins)
    check_group(ins, out, TOL[dt], label=f"small group {ds}")
    acc = run_group(ins, accumulate=True, preset=(0.5, -1.5))
    for p, i in enumerate(ins):
        one = run_hip(i)
        for k in range(len(tokens)):
            assert torch.equal(one["dA"][k], out["dA"][p][k]) and torch.equal(one["dB"][k], out["dB"][p][k]), (p, k)
            assert torch.equal(acc["dA"][p][k], out["dA"][p][k] + 0.5) and torch.equal(acc["dB"][p][k], out["dB"][p][k] - 1.5), (p, k)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,case", [(t, c) for t, c, _ in SMALL_BACK])
def test_small_backward(dtype, case):
    from paper_2312_02515_amd import binding as hip
    from tests.parity_util import TOL, check_full, run_hip
    from tests.test_gpu_general import _inputs
    T, h, d, tokens, ranks, lead = case
    dtype = torch.float32 if dtype == "f32" else torch.bfloat16
    inp = _inputs(T, h, d, tokens, ranks, dtype, lead=lead, seed=95)
    out = run_hip(inp)
    check_full(inp, out, TOL[dtype], label=f"small backward {case}")
    # added to what is there: one fp32 addition behind the same sums
    pre = [[torch.randn_like(t) for t in out[n]] for n in ("dA", "dB")]
    acc = run_hip(inp, accumulate=True, preset_grads=pre)
    for n, ps in zip(("dA", "dB"), pre):
        for a, b, p in zip(acc[n], out[n], ps):
            assert torch.equal(a, p + b), n
    # dX in the place of X: the gradients still read X
    prob = hip.Problem(T, h, d, inp.W, inp.seg_offsets, inp.ranks, inp.scalings, inp.A, inp.B)
    saved, ws, X = prob.alloc_saved(), prob.alloc_workspace(), inp.X.clone()
    Y = torch.empty_like(out["Y"])
    hip.mlora_lora_fwd(prob, X, Y, saved, ws)
    dA, dB = prob.alloc_grads()
    hip.mlora_lora_bwd(prob, X, inp.dY, saved, X, dA, dB, False, ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, out["Y"])
    for a, b in zip(dA + dB, out["dA"] + out["dB"]):
        assert torch.equal(a, b)
    # (dX's ranges are planned with the whole scratch there: the sums may come in another order)
    err = (X.double() - out["dX"].double()).norm() / out["dX"].double().norm()
    assert err <= TOL[dtype]
    # dX in the place of the saved Z, which the gradients still read
    n = X.numel() * X.element_size()
    buf = torch.empty(max(n, prob.saved_bytes()), dtype=torch.uint8, device=X.device)
    saved, dX = buf[:prob.saved_bytes()], buf[:n].view(dtype).view(T, h)
    hip.mlora_lora_fwd(prob, inp.X, Y, saved, ws)
    dA, dB = prob.alloc_grads()
    hip.mlora_lora_bwd(prob, inp.X, inp.dY, saved, dX, dA, dB, False, ws)
    torch.cuda.synchronize()
    for a, b in zip(dA + dB, out["dA"] + out["dB"]):
        assert torch.equal(a, b)
    err = (dX.double() - out["dX"].double()).norm() / out["dX"].double().norm()
    assert err <= TOL[dtype]
