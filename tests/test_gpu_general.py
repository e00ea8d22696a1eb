"""The general kernels (fp32, and bf16 sizes or addresses the aligned kernels do not take) at the
sizes where their tiles, splits and tails change form, against the CPU fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2312_02515_amd import binding as mb
from paper_2312_02515_amd import workloads as wl
from tests import form_cases
from tests.parity_util import TOL, check_full, run_hip
from tests.test_gpu_groups import _group_inputs, check_group, run_group
from tests.test_gpu_parity import _others_identical

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _inputs(T, h, d, tokens, ranks, dtype, lead=0, seed=0):
    off = [lead]
    for t in tokens:
        off.append(off[-1] + t)
    assert off[-1] <= T
    return wl.make_inputs(T, h, d, off, ranks, [0.5 + 0.25 * (k % 4) for k in range(len(ranks))], dtype, device=DEV,
                          seed=seed, sigma_w=1.0 / np.sqrt(h))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("case", [
    # T, h, d, tokens, ranks, lead
    (40, 1, 1, [17, 20], [1, 3], 2),                      # rows of one element
    (70, 3, 5, [33, 30], [2, 8], 1),                      # rows shorter than one 16-byte piece
    (33, 8, 4, [33], [128], 0),                           # exactly one piece; 8 column groups of 16
    (65, 31, 33, [31, 34], [16, 17], 0),                  # 16 x 64 blocks: tails of one element
    (90, 127, 129, [90], [33], 0),                        # ... a column block of one column
    (100, 2050, 70, [60, 37], [5, 20], 2),                # few tiles, deep: forward split over the contraction
    (100, 70, 3001, [60, 37], [5, 20], 2),                # the same for the input gradient
    (2200, 136, 2101, [1000, 0, 1150], [7, 64, 32], 25),  # 128 x 128 tiles forward, odd stride
    (16500, 41, 24, [9000, 7000], [4, 40], 300),          # many 16-row blocks (501 blocks of 32 rows are too few)
    (700, 70, 514, [640], [9], 13),                       # token ranges; column groups of 64 that end early
    (150, 515, 67, [20, 101], [100, 17], 12),             # 16-row blocks: runs, single groups and a tail
    (49, 1021, 4, [16, 17], [1, 128], 3),                 # ... exactly one piece of columns
])
def test_general_kernel_edges(case, dtype):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, dtype, lead=lead, seed=71)
    if h == 1:
        # every gradient is one sum over tokens, sum_t x_t g_t with g_t rounded to 8 bits: its error is
        # up to 2^-9 sum |x_t g_t|, which is 2^-9 of the result only where the terms do not cancel
        inp.X.abs_()
        inp.dY.abs_()
    check_full(inp, run_hip(inp), TOL[dtype], label=f"general {case}")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("case", [c for c, _ in form_cases.GENERAL])
def test_general_kernel_forms(case, dtype):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, dtype, lead=lead, seed=80)
    check_full(inp, run_hip(inp), TOL[dtype], label=f"general {case}")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,h,d", [(1500, 520, 1024 + r) for r in range(1, 9)] + [   # 64 x 64 tiles, every remainder of a piece
    (2200, 139, 2113), (2200, 139, 2175), (2200, 139, 2167),                         # 128 x 128
    (100, 2050, 67), (100, 4200, 1)])                                                # ranges; rows shorter than a piece
def test_last_columns_of_general_tiles(dtype, T, h, d):
    """The piece of columns that crosses the right edge, with ranks and rows of no task beside it; an Inf in
    the last column of W stays there."""
    inp = _inputs(T, h, d, [T // 2, T // 3], [9, 24], dtype, lead=5, seed=83)
    check_full(inp, run_hip(inp), TOL[dtype], label=f"last columns {T, h, d}")
    inp.W[0, -1] = float("inf")
    inp.X[:, 0] = 1.0
    Y = run_hip(inp)["Y"]
    assert torch.isinf(Y[:, -1]).all() and torch.isfinite(Y[:, :-1]).all()


@pytest.mark.parametrize("dtype,case", [(t, c) for t, c, _ in form_cases.QUARTERS])
def test_general_quarters(dtype, case):
    T, h, d, tokens, ranks, lead = case
    dtype = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    inp = _inputs(T, h, d, tokens, ranks, dtype, lead=lead, seed=84)
    check_full(inp, run_hip(inp), TOL[dtype], label=f"quarters {case}")


@pytest.mark.parametrize("dtype,case", [(t, c) for t, c, _ in form_cases.EDGE_QUARTERS])
def test_columns_of_a_tile_are_summed_alike(dtype, case):
    """Columns of one 128 x 128 tile that hold the same values come out with the same bits, also those that the
    piece of columns at the right edge (of the next tile, which is summed in ranges) covers again."""
    T, h, d, tokens, ranks, lead = case
    dtype = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    inp = _inputs(T, h, d, tokens, ranks, dtype, lead=lead, seed=88)
    V = 16 // inp.X.element_size()
    p = d // 128 * 128                     # first column of the last tile
    again, other = slice(d - V, p), slice(d - V - 2 * V, p - 2 * V)
    for M in [inp.W] + inp.B:
        M[:, again] = M[:, other]
    out = run_hip(inp)
    assert torch.equal(out["Y"][:, again], out["Y"][:, other])
    check_full(inp, out, TOL[dtype], label=f"right edge {case}")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("h,d,tokens,ranks", [
    (61, 66, [31, 32, 33, 1], [16, 17, 8, 33]),           # around a run's tokens; edges inside and between lanes' pieces
    (259, 7, [63, 64, 65, 0], [65, 4, 64, 128]),          # ranks on either side of each group count
    (3, 513, [97, 130], [5, 40], ),                       # rows shorter than a piece; one column in the last block
    (70, 1027, [1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 28], [128, 17, 64, 1, 33, 65, 16, 128, 40, 66, 32, 8]),   # tokens around
                                                          # the groups of one run, in the body for each rank
])
def test_general_gradients_add_to_what_is_there(dtype, h, d, tokens, ranks):
    """A column that two lanes load is stored, and in accumulate mode added, once."""
    inp = _inputs(sum(tokens) + 9, h, d, tokens, ranks, dtype, lead=4, seed=85)
    got = run_hip(inp)
    check_full(inp, got, TOL[dtype], label=f"gradients {h, d}")
    pre = [[torch.full_like(g, 0.5 + k) for k, g in enumerate(got[n])] for n in ("dA", "dB")]
    acc = run_hip(inp, accumulate=True, preset_grads=pre)
    for n, p in zip(("dA", "dB"), pre):
        for g, was, now in zip(got[n], p, acc[n]):
            assert torch.equal(now, was + g)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_general_group_sum_in_large_tiles(dtype):
    """The summed input gradient in 128 x 128 tiles (2200 x 2101 outputs)."""
    ins = _group_inputs(2200, 2101, [139, 320], [1000, 1150], [[7, 64], [32, 5]], dtype, lead=25, seed=81)
    check_group(ins, run_group(ins), TOL[dtype], label="general group, large tiles")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,h,d", [(300, 128, 192), (1500, 520, 1032), (2200, 256, 2112)])   # 16 x 64, 64 x 64, 128 x 128
def test_general_kernels_take_misaligned_buffers(dtype, T, h, d):
    """Activations and weight one element off a 16-byte boundary: same results as aligned copies."""
    inp = _inputs(T, h, d, [100, 150], [8, 16], dtype, lead=5, seed=72)

    def off_by_one(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
        buf[1:].copy_(t.reshape(-1))
        return buf[1:].view(t.shape)

    inp.X, inp.dY, inp.W = off_by_one(inp.X), off_by_one(inp.dY), off_by_one(inp.W)
    inp.A, inp.B = [off_by_one(t) for t in inp.A], [off_by_one(t) for t in inp.B]
    check_full(inp, run_hip(inp), TOL[dtype], label="misaligned")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ds", [[72, 2051], [35, 130, 900, 1]])
def test_general_group_sum(ds, dtype):
    """dX of a group in one launch: operand pairs of unequal depth, split over the contraction."""
    ranks = [[3, 16 + p] for p in range(len(ds))]
    ins = _group_inputs(150, 52, ds, [80, 61], ranks, dtype, lead=4, seed=73)
    check_group(ins, run_group(ins), TOL[dtype], label=f"general group {ds}")


@pytest.mark.parametrize("case", [
    # T, h, d, tokens, ranks, lead: bf16, h and d multiples of 64, ranks that are no multiple of 8
    (300, 64, 64, [300], [9], 0),                                  # the LoRA tile right behind one base tile
    (1000, 192, 320, [100, 0, 333, 500], [7, 24, 127, 66], 7),     # beside whole-chunk ranks; two LoRA tiles
    (500, 1024, 1088, [77, 200, 223], [3, 20, 30], 0),             # contraction split over a block's waves
    (500, 1024, 1088, [77, 200, 223], [3, 36, 64], 0),
    (17000, 64, 128, [9000, 8000], [5, 12], 0),                    # 64-row low-rank blocks
    (33100, 128, 64, [16500, 16500], [1, 44], 60),                 # 128-row low-rank blocks
])
def test_ragged_ranks_on_aligned_shapes(case):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=74)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"ragged ranks {case}")


@pytest.mark.parametrize("case", [c for c, _ in form_cases.LANES])
def test_tasks_searched_by_all_lanes(case):
    """Around the number of tasks from which a wave's lanes search for a row's task: empty tasks at either
    end and in between, tasks of one row, rows of no task before and after."""
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=86)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"tasks {T, h, d, len(tokens)}")


@pytest.mark.parametrize("h,d,rank", [(2048, 192, 128), (192, 2112, 77), (4160, 64, 65)])
def test_short_tasks_of_high_rank_in_ranges(h, d, rank):
    """64 tasks of up to 32 rows, ranks above 64 among them: low-rank rows in blocks of 32 rows and ranges."""
    tokens = [(13 * k) % 33 for k in range(64)]
    inp = _inputs(sum(tokens) + 21, h, d, tokens, [rank if k % 3 == 0 else 1 + k for k in range(64)], torch.bfloat16, lead=9,
                  seed=87)
    plan = mb.Problem(sum(tokens) + 21, h, d, inp.W, inp.seg_offsets, inp.ranks, inp.scalings, inp.A, inp.B).kernel_plan()
    side = "Z" if h > d else "G"
    assert plan[side + "_rows"] == 32 and plan[side + "_parts"] > 1, plan
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"short tasks {h, d, rank}")


@pytest.mark.parametrize("h,d", [(256, 320), (5120, 1088)])
def test_gradients_of_high_ranks(h, d):
    """Ranks above 64 with at most 256 gradient blocks (three ring stages) and with more (two): tasks around whole
    64-token tiles, long enough to go round the ring, overwriting and adding."""
    tokens, ranks = [0, 1, 64, 65, 700, 449], [128, 65, 72, 100, 127, 128]
    assert (len(tokens) * ((h + 127) // 128 + (d + 127) // 128) > 256) == (h == 5120)
    inp = _inputs(sum(tokens) + 7, h, d, tokens, ranks, torch.bfloat16, lead=3, seed=89)
    got = run_hip(inp)
    check_full(inp, got, TOL[torch.bfloat16], label=f"high ranks {h, d}")
    pre = [[torch.full_like(g, 0.5 + k) for k, g in enumerate(got[n])] for n in ("dA", "dB")]
    acc = run_hip(inp, accumulate=True, preset_grads=pre)
    for n, p in zip(("dA", "dB"), pre):
        for g, was, now in zip(got[n], p, acc[n]):
            assert torch.equal(now, was + g)


@pytest.mark.parametrize("P", [2, 3, 4])
def test_ragged_ranks_in_a_group(P):
    ranks = [[5 + p, 12, 8] for p in range(P)]
    if P == 2:
        ranks[1] = [100, 33, 64]      # four 32-column groups
    ins = _group_inputs(420, 128, [64 * (p + 1) for p in range(P)], [90, 201, 100], ranks, torch.bfloat16, lead=6, seed=75)
    check_group(ins, run_group(ins), TOL[torch.bfloat16], label=f"ragged group {P}")


@pytest.mark.parametrize("case", [
    # T, h, d, tokens, ranks, lead: bf16 base products in small tiles ...
    (100, 4096, 512, [37, 20, 40], [16, 7, 128], 3),        # one row tile whose lower half is empty; many ranges
    (300, 512, 2048, [140, 0, 131], [64, 33, 8], 20),       # a task across half tiles; ranks 33..64
    (520, 1088, 448, [33, 31, 450], [1, 100, 32], 6),
] + [c for c, _ in form_cases.HALVES])                      # ... and cut into half tiles and contraction ranges
def test_half_tiles_and_contraction_ranges(case):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=76)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"half tiles {case}")
    inp.W.zero_()      # the LoRA terms alone
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"half tiles, W = 0 {case}")


@pytest.mark.parametrize("case", [
    # T, h, d, tokens, ranks, lead: low-rank rows whose contraction is cut into ranges over blocks
    (700, 512, 2048, [300, 0, 390], [128, 8, 70], 4),       # four column groups, rows before and after the tasks
    (8500, 256, 320, [4000, 4400], [16, 33], 60),           # more than 256 blocks of 32 rows: not split
    (1100, 8192, 64, [500, 560], [24, 9], 10),              # deep contraction of few rows (forward)
    (1100, 64, 8256, [500, 560], [24, 8], 10),              # ... and of s dy B^T; ranges of unequal length
])
def test_contraction_split_low_rank_rows(case):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=77)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"split rows {case}")
    inp.W.zero_()
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"split rows, W = 0 {case}")


@pytest.mark.parametrize("case", [c for c, _ in form_cases.SPLIT_ROWS])
def test_contraction_ranges_of_low_rank_rows(case):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=82)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"ranges {case}")
    inp.W.zero_()
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"ranges, W = 0 {case}")


@pytest.mark.parametrize("case", [c for c, _ in form_cases.WHOLE_TILES])
def test_whole_tiles_of_several_tasks(case):
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, torch.bfloat16, lead=lead, seed=84)
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"whole tiles {case[:3]}")
    inp.W.zero_()
    check_full(inp, run_hip(inp), TOL[torch.bfloat16], label=f"whole tiles, W = 0 {case[:3]}")


@pytest.mark.parametrize("what", ["A", "B", "X", "dY"])
@pytest.mark.parametrize("dtype,case,j", [(t, c, j) for t, c, _, j in form_cases.ISOLATION])
def test_isolation_from_non_finite_values_in_every_form(dtype, case, j, what):
    """A diverged task (NaN or Inf in its adapter or its rows) leaves its neighbours' results finite and
    bit-identical, also in ragged ranks, split launches and the general tiles."""
    T, h, d, tokens, ranks, lead = case
    inp = _inputs(T, h, d, tokens, ranks, {"f32": torch.float32, "bf16": torch.bfloat16}[dtype], lead=lead, seed=83)
    a = run_hip(inp)
    lo, hi = inp.seg_offsets[j], inp.seg_offsets[j + 1]
    flat = {"A": inp.A[j], "B": inp.B[j], "X": inp.X[lo:hi], "dY": inp.dY[lo:hi]}[what].view(-1)
    flat[0::3] = float("nan")
    flat[1::3] = float("inf")
    flat[2::3] = -float("inf")
    b = run_hip(inp)
    _others_identical(a, b, inp, j)
    for name in ("Y", "dX"):
        assert torch.isfinite(b[name][:lo]).all() and torch.isfinite(b[name][hi:]).all()


@pytest.mark.parametrize("case", [
    # T, h, d per projection, tokens, ranks, lead: a group's summed input gradient in small tiles ...
    (T, h, ds, tokens, [[(8, 64, 24)[(p + k) % 3] + (p == 1) for k in range(len(tokens))] for p in range(len(ds))], lead)
    for T, h, ds, tokens, lead in [
        (100, 512, [4096, 64, 1088], [37, 40], 5),       # contraction ranges that cross and skip operand pairs
        (300, 640, [512, 2048], [130, 0, 160], 3),
        (700, 1088, [1024, 1024, 256, 64], [300, 333], 60)]
] + [c[:-1] for c in form_cases.GROUPS])                 # ... in half tiles, whole tiles, partial contraction tiles
def test_group_sum_in_every_form(case):
    T, h, ds, tokens, ranks, lead = case
    ins = _group_inputs(T, h, ds, tokens, ranks, torch.bfloat16, lead=lead, seed=78)
    check_group(ins, run_group(ins), TOL[torch.bfloat16], label=f"group {case[:3]}")
    for i in ins:
        i.W.zero_()
    check_group(ins, run_group(ins), TOL[torch.bfloat16], label=f"group, W = 0 {case[:3]}")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("h,d", [(256, 72), (257, 131), (64, 4104), (2085, 40), (3000, 7),
                                 (161, 4104), (81, 65544), (160, 72)])
def test_weight_coder_over_row_ranges(h, d, dtype):
    """Row ranges of unequal length, 16-byte pieces and single columns, a zero column: codes and scales
    bit for bit against the oracle."""
    from oracle import w8_oracle as w8
    from paper_2312_02515_amd import binding as mb
    W = torch.randn((h, d), generator=torch.Generator().manual_seed(h + d)) * torch.logspace(-6, 3, d)
    W[:, d // 2] = 0
    W = W.to(dtype)
    Wq, c = mb.mlora_w8_quantize(W.to(DEV))
    ref_q, ref_c = w8.quantize_w8(W.to(torch.float32).numpy())
    assert np.array_equal(c.cpu().numpy(), ref_c) and np.array_equal(Wq.cpu().numpy(), ref_q)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_one_workspace_for_every_batch(dtype):
    """A workspace of the largest batch's size serves the smaller ones, whose launches are cut into more
    ranges: the same bits as with a workspace of their own, and the oracle's values."""
    from paper_2312_02515_amd import binding as mb
    h, d, ranks = 1024, 1088, [16, 64]
    batches = [_inputs(T, h, d, [T // 2, T - T // 2], ranks, dtype, seed=79) for T in (8192, 600, 64)]
    probs = [mb.Problem(i.X.shape[0], h, d, i.W, i.seg_offsets, i.ranks, i.scalings, i.A, i.B) for i in batches]
    ws = probs[0].alloc_workspace()
    for inp, prob in zip(batches[1:], probs[1:]):
        T = inp.X.shape[0]
        ref = run_hip(inp)
        check_full(inp, ref, TOL[dtype], label=f"T = {T}")
        ws.fill_(0xFF)
        Y, dX = torch.empty((T, d), dtype=dtype, device=DEV), torch.empty((T, h), dtype=dtype, device=DEV)
        (dA, dB), saved = prob.alloc_grads(), prob.alloc_saved()
        mb.mlora_lora_fwd(prob, inp.X, Y, saved, ws)
        mb.mlora_lora_bwd(prob, inp.X, inp.dY, saved, dX, dA, dB, False, ws)
        torch.cuda.synchronize()
        assert torch.equal(Y, ref["Y"]) and torch.equal(dX, ref["dX"])
        for k in range(len(ranks)):
            assert torch.equal(dA[k], ref["dA"][k]) and torch.equal(dB[k], ref["dB"][k])


# aligned kernels; 16 x 64 tiles and a shared launch; small tiles in ranges; the general kernel's tiles, in fp32 and ranges
@pytest.mark.parametrize("T,h,d,tokens,ranks,f32", [
    (900, 2048, 5632, [256, 515], [8, 16], False),
    (128, 256, 256, [60, 60], [8, 64], False),
    (60, 584, 4040, [37, 20], [12, 40], False),
    (300, 704, 70, [150, 100], [5, 16], False),
    (300, 2001, 501, [150, 140], [16, 3], True),
    (6, 4096, 4096, [2, 3], [16, 100], False),
])
def test_timed_launches(T, h, d, tokens, ranks, f32):
    """Every launch of a call is timed, and its work counted once."""
    inp = _inputs(T, h, d, tokens, ranks, torch.float32 if f32 else torch.bfloat16, lead=1, seed=97)
    prob = mb.Problem(T, h, d, inp.W, inp.seg_offsets, inp.ranks, inp.scalings, inp.A, inp.B)
    shared = prob.kernel_plan()["shared"]
    run_hip(inp)
    mb.profile_kernels_read()
    mb.profile_kernels(True)
    try:
        run_hip(inp)
    finally:
        mb.profile_kernels(False)
    got = mb.profile_kernels_read()
    el, rows, r = (4 if f32 else 2), sum(tokens), sum(ranks)
    lora = sum(t * k for t, k in zip(tokens, ranks))
    assert got["gemm"][1] == 4 * T * h * d + 2 * lora * (h + d) * (2 if shared else 1)
    assert (got["grad"][1] > 0) == (not shared) and got["gemm"][2] == 2 and got["rows"][2] >= 2
    low = el * ((rows + r) * (h + d))
    assert low < got["rows"][1] <= low + 2 * el * rows * 128
    if not shared:
        low = el * rows * (h + d) + 4 * r * (h + d)
        assert low < got["grad"][1] <= low + 2 * el * rows * 128
    assert all(got[k][0] > 0 for k in got if got[k][2])
