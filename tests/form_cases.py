"""Sizes at which the launches of a call take a certain form: (T, h, d, tokens, ranks, lead) and the form,
as mlora_kernel_plan names it ({"f32": .., "bf16": ..} where the two differ).  The GPU tests run them, the
CPU test holds them to their forms, so that a changed threshold cannot move them elsewhere unnoticed."""

# General kernels, fp32 and bf16
GENERAL = [
    # one element around the contraction tiles (32 fp32, 64 bf16) of the 64 x 64 form
    ((2000, 31, 1000, [900, 1050], [16, 5], 30), {"Y": "64", "Y_parts": 1}),
    ((2000, 33, 1000, [1990], [17], 3), {"Y": "64"}),
    ((2000, 63, 1000, [900, 1050], [3, 40], 30), {"Y": "64"}),
    ((2000, 65, 1000, [900, 1050], [33, 8], 0), {"Y": "64"}),
    ((2000, 1000, 33, [900, 1050], [33, 8], 7), {"dX": "64"}),
    ((2000, 1000, 63, [900, 1050], [16, 20], 7), {"dX": "64"}),
    # one column around its column tiles
    ((1500, 2300, 127, [700, 0, 755], [9, 4, 32], 5), {"Y": "64", "dX": "64"}),
    ((1500, 2300, 129, [700, 755], [9, 32], 5), {"Y": "64", "dX": "64"}),
    # 128 x 128 tiles (fp32: a round of them, the rest as quarters, see QUARTERS): ragged contraction, odd strides,
    # several contraction tiles
    ((2200, 139, 2101, [1000, 0, 1150], [7, 64, 32], 25), {"Y": "128"}),
    ((2200, 2101, 139, [1000, 0, 1150], [7, 64, 32], 25), {"dX": "128", "dX_parts": 1}),
    ((2200, 2101, 320, [1000, 1150], [128, 3], 25), {"dX": "128"}),
    # 32 rows per block of the low-rank rows
    ((17000, 41, 24, [9000, 7500], [4, 40], 300), {"Z_rows": 32, "G_rows": 32}),
    # 64 tasks: the tasks of a block are searched by all lanes
    ((1500, 41, 600, [k % 40 for k in range(64)], [1 + k % 20 for k in range(64)], 11), {"Y": "64"}),
    ((700, 60, 70, [k % 15 for k in range(64)], [1 + k % 20 for k in range(64)], 40), {"Y": "skinny", "dX": "skinny"}),
]

# General kernels, 128 x 128 tiles: all of them, or whole rounds and the rest as quarters of 64 x 64, in one
# contraction range or several; quarters beyond the last row and column
QUARTERS = [
    # dtype, (T, h, d, tokens, ranks, lead), form
    ("f32", (2150, 1700, 2101, [1000, 0, 1100], [7, 64, 32], 25), {"Y": "128", "Y_parts": 5, "Y_whole": 256, "Y_tiles": 306}),
    ("f32", (2150, 2101, 1700, [1000, 0, 1100], [7, 64, 32], 25), {"dX": "128", "dX_parts": 5, "dX_whole": 256, "dX_tiles": 306}),
    ("f32", (2200, 139, 2101, [1000, 0, 1150], [7, 64, 32], 25), {"Y": "128", "Y_parts": 1, "Y_whole": 256, "Y_tiles": 306}),
    ("f32", (2200, 2101, 139, [1000, 0, 1150], [7, 64, 32], 25), {"dX": "128", "dX_parts": 1, "dX_whole": 256, "dX_tiles": 306}),
    ("bf16", (8330, 1500, 1000, [4100, 4150], [9, 100], 70), {"Y": "128", "Y_parts": 4, "Y_whole": 512, "Y_tiles": 528}),
    ("bf16", (8330, 1000, 1500, [4100, 4150], [9, 100], 70), {"dX": "128", "dX_parts": 4, "dX_whole": 512, "dX_tiles": 528}),
    ("bf16", (1308, 2050, 6500, [1248, 40], [9, 24], 7), {"Y": "128", "Y_parts": 1, "Y_whole": 512, "Y_tiles": 561}),
    ("bf16", (1308, 6500, 2050, [1248, 40], [9, 24], 7), {"dX": "128", "dX_parts": 1, "dX_whole": 512, "dX_tiles": 561}),
    ("bf16", (2200, 139, 2101, [1000, 0, 1150], [7, 64, 32], 25), {"Y": "128", "Y_parts": 1, "Y_whole": 306, "Y_tiles": 306}),
    ("bf16", (2200, 2101, 139, [1000, 0, 1150], [7, 64, 32], 25), {"dX": "128", "dX_parts": 1, "dX_whole": 306, "dX_tiles": 306}),
]

# ... forward, the last column tile alone in quarters and ranges, 1 .. V - 1 columns wide (V = columns of a
# 16-byte piece): the piece of columns at the right edge begins in the tile before it
EDGE_QUARTERS = [
    ("f32", (1436, 600, 5377, [1376, 40], [9, 24], 7), {"Y": "128", "Y_parts": 4, "Y_whole": 512, "Y_tiles": 516}),
    ("f32", (1436, 600, 5379, [1376, 40], [9, 24], 7), {"Y": "128", "Y_parts": 4, "Y_whole": 512, "Y_tiles": 516}),
    ("bf16", (2460, 2050, 1537, [2400, 40], [9, 24], 7), {"Y": "128", "Y_parts": 7, "Y_whole": 256, "Y_tiles": 260}),
    ("bf16", (2460, 2050, 1543, [2400, 40], [9, 24], 7), {"Y": "128", "Y_parts": 7, "Y_whole": 256, "Y_tiles": 260}),
]

# bf16, h and d multiples of 64: half tiles (128 x 256) of both layouts, in one contraction range, several and several
# of unequal length; tiles whose lower half is empty, tasks across half tiles, rows of no task, ranks above 32 and 64
HALVES = [
    ((1100, 2048, 5632, [337, 320, 440], [16, 7, 128], 3), {"Y": "halves", "Y_parts": 1, "dX": "halves", "dX_parts": 3}),
    ((1100, 1024, 4096, [337, 0, 441], [64, 33, 8], 20), {"Y": "halves", "Y_parts": 1, "dX": "halves", "dX_parts": 6}),
    ((1100, 5696, 2048, [337, 20, 640], [16, 7, 30], 3), {"Y": "halves", "Y_parts": 3, "dX": "halves", "dX_parts": 1}),
    ((4200, 1024, 4096, [2100, 2050], [16, 24], 50), {"Y": "mixed"}),
]


def _group_ranks(P, K):
    return [[1 + (7 * k + 5 * p) % 64 for k in range(K)] for p in range(P)]


_PACKED = [(5 * k) % 17 for k in range(60)]

# Summed input gradients of two, three and four operand pairs, bf16: (T, h, d per projection, tokens, ranks per
# projection, lead) and the form as mlora_kernel_plan_group names it
GROUPS = [(T, h, ds, tokens, _group_ranks(len(ds), len(tokens)), lead, want) for T, h, ds, tokens, lead, want in [
    # half tiles in contraction ranges, which cross operand pairs
    (1500, 2048, [2048, 512], [700, 750], 3, {"dX": "halves", "dX_parts": 2}),
    (700, 2048, [2048, 2048, 2048], [300, 333], 60, {"dX": "halves", "dX_parts": 5}),
    (700, 2048, [2048, 1024, 1024, 2048], [300, 0, 333], 60, {"dX": "halves", "dX_parts": 5}),
    # ... that end in partial contraction tiles
    (326, 2816, [1280, 3320], [123, 108], 3, {"dX": "halves", "dX_parts": 5}),
    (172, 3072, [3664, 3592, 768], [46, 57], 3, {"dX": "halves", "dX_parts": 10}),
    (223, 2224, [3664, 3272, 440, 3304], [71, 74], 3, {"dX": "halves", "dX_parts": 13}),
    # ... one range
    (2000, 2056, [2056, 520], [900, 1055], 3, {"dX": "halves", "dX_parts": 1}),
    # whole tiles that end in partial contraction tiles, one of them alone among them
    (9268, 1032, [56, 136], [4000, 33, 5000], 3, {"dX": "whole"}),
    (9268, 1032, [632, 72, 200], [4000, 33, 5000], 3, {"dX": "whole"}),
    (9268, 1032, [136, 64, 72, 8], [4000, 33, 5000], 3, {"dX": "whole"}),
    # half tiles of packed rows (60 tasks of up to 16 rows): the tiles are those of the 494 rows alone
    (494, 4104, [4104, 2056], _PACKED, 9, {"dX": "halves", "dX_parts": 3, "dX_tiles": 34}),
    (494, 4480, [2104, 2240, 704], _PACKED, 9, {"dX": "halves", "dX_parts": 3, "dX_tiles": 36}),
    (494, 4224, [384, 336, 3992, 3864], _PACKED, 9, {"dX": "halves", "dX_parts": 3, "dX_tiles": 34}),
    # small tiles
    (500, 520, [712, 264, 1000, 72], [100, 197, 170], 3, {"dX": "ring"}),
]]

# bf16, h and d multiples of 64: contraction ranges of the low-rank rows
SPLIT_ROWS = [
    ((4300, 4160, 64, [2000, 2140], [16, 33], 60), {"Z_rows": 128, "Z_parts": 4, "G_parts": 1}),
    ((4300, 64, 4160, [2000, 2140], [12, 40], 60), {"G_rows": 128, "G_parts": 4, "Z_parts": 1}),
    ((4300, 8256, 64, [2000, 2140], [16, 5], 0), {"Z_rows": 128, "Z_parts": 8}),   # ranges of unequal length
    ((4300, 64, 8256, [2000, 2140], [16, 33], 0), {"G_rows": 128, "G_parts": 8}),
]

# bf16, h and d multiples of 64: whole tiles that hold several tasks of mixed ranks (forward, backward).
# (Fewer than 256 tiles of several tasks run as halves.)
_SHARED = [1, 255, 257, 31, 33, 95, 97, 160, 161, 500, 12, 700] * 4
WHOLE_TILES = [
    ((9268, 128, 1024, _SHARED, [8, 64, 128, 16] * 12, 20), {"Y": "whole"}),
    ((9268, 1024, 128, _SHARED, [8, 64, 128, 16] * 12, 20), {"dX": "whole"}),
    ((9268, 128, 1024, _SHARED, [5, 33, 127, 12] * 12, 20), {"Y": "whole"}),
    ((9268, 1024, 128, _SHARED, [5, 33, 127, 12] * 12, 20), {"dX": "whole"}),
] + [
    # one, three and five base tiles in front of the LoRA tiles: the short forms of prologue and tail
    c for k in (64, 192, 320) for c in (
        ((9268, k, 1024, _SHARED, [128, 8, 33, 64] * 12, 20), {"Y": "whole"}),
        ((9268, 1024, k, _SHARED, [128, 8, 33, 64] * 12, 20), {"dX": "whole"}))
]

# bf16, h and d multiples of 64: around the number of tasks from which a wave's lanes search for a row's task
# (eight), in blocks of 32 rows with four waves each, 128 with ranges, 64 and 128


def _lanes_case(T, h, d, rank, K):
    """Empty tasks at either end and in between, tasks of one row; the second task takes what is left."""
    left, tokens = T - 60, []
    for k in range(K):
        t = 0 if k in (0, 4, K - 1) else 1 if k % 7 == 5 else min(left, 2 * (T - 60) // K * (1 + k % 3) // 4)
        tokens.append(t)
        left -= t
    tokens[1] += left
    return T, h, d, tokens, [max(1, rank - 5 * (k % 4)) for k in range(K)], 31


LANES = [(_lanes_case(*size, K), dict(want, **({"Z_parts": 2 if K == 64 else 4} if size[0] == 4300 else {})))
         for K in (8, 9, 33, 64) for size, want in [
             ((1700, 4096, 128, 24), {"Y": "ring", "Z_rows": 32, "G_rows": 32, "Z_parts": 1}),
             ((4300, 2048, 192, 128), {"Y": "ring", "dX": "whole", "Z_rows": 128}),
             ((17000, 128, 1088, 16), {"Y": "whole", "Z_rows": 64, "G_rows": 64}),
             ((33600, 128, 64, 16), {"Y": "whole", "dX": "whole", "Z_rows": 128, "G_rows": 128, "Z_parts": 1, "G_parts": 1})]]

# Isolation of a diverged task (the last entry of a case) from its neighbours
ISOLATION = [
    # dtype, (T, h, d, tokens, ranks, lead), form, task
    # ragged ranks, whole tiles: A_k's tile put together in registers, 64-row blocks of the low-rank rows
    ("bf16", (17000, 1024, 64, [9000, 7900], [5, 12], 3), {"dX": "whole", "Z_rows": 64}, 0),
    ("bf16", (9268, 1024, 128, _SHARED, [5, 33, 127, 12] * 12, 20), {"dX": "whole"}, 14),
    ("bf16", (9268, 128, 1024, _SHARED, [8, 64, 128, 16] * 12, 20), {"Y": "whole"}, 14),
    ("bf16", (1100, 64, 64, [300, 90, 700], [9, 127, 33], 7), {"Y": "skinny", "dX": "skinny", "Z_rows": 32}, 1),
    ("bf16", (300, 64, 64, [60, 90, 33, 100], [9, 127, 33, 2], 7), {"Y": "skinny", "dX": "skinny"}, 1),
    # half tiles, in one contraction range and in several, the diverged task across two of them and inside one
    ("bf16", (900, 1088, 4160, [300, 90, 500], [9, 27, 33], 7), {"Y": "halves", "dX": "halves", "dX_parts": 6}, 0),
    ("bf16", (1100, 5696, 2048, [337, 20, 640], [16, 7, 30], 3), {"Y": "halves", "Y_parts": 3, "dX": "halves"}, 1),
    ("bf16", (700, 1088, 64, [300, 33, 360], [3, 20, 30], 2), {"Z_rows": 32, "Z_parts": 1}, 1),
    ("bf16", (4300, 4160, 64, [2000, 2140], [16, 33], 60), {"Z_rows": 128, "Z_parts": 4}, 0),
    ("bf16", (33100, 64, 64, [16500, 16500], [1, 44], 60), {"Z_rows": 128, "Z_parts": 1}, 1),
    # a round of whole tiles with halves behind it; contraction ranges
    ("bf16", (4300, 1024, 4096, [2100, 100, 2050], [16, 24, 30], 50), {"Y": "mixed", "dX": "halves"}, 1),
    # general tiles
    ("bf16", (2200, 139, 2101, [1000, 33, 1100], [7, 64, 32], 25), {"Y": "128"}, 1),
    ("f32", (2200, 139, 2101, [1000, 33, 1100], [7, 64, 32], 25), {"Y": "128"}, 1),
    ("bf16", (2200, 2101, 139, [1000, 33, 1100], [7, 64, 32], 25), {"dX": "128"}, 1),
    ("f32", (2200, 2101, 139, [1000, 33, 1100], [7, 64, 32], 25), {"dX": "128"}, 1),
    ("f32", (1500, 40, 600, [k % 40 for k in range(64)], [1 + k % 20 for k in range(64)], 11), {"Y": "64"}, 38),
]
