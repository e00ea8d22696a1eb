"""Sizes at which the bf16 base products run in small tiles, or in any tile with a last, partial contraction tile
(features that are multiples of 8 but not of 64): (T, h, d, tokens, ranks, lead) and parts of mlora_kernel_plan's
answer.  The GPU tests run them, the CPU test holds them to their forms."""

CASES = [
    # 64 x 64 tiles, one group of waves: rows and columns around the tile, two tasks in a tile, ranks around a slot of 32
    ((2900, 192, 704, [63, 65, 1, 2700], [8, 32, 33, 64], 3), {"Y_rows": 64}),
    ((2900, 704, 192, [31, 33, 95, 97, 160, 2461], [8, 16, 33, 127, 5, 128], 17), {"dX_rows": 64}),
    ((1100, 1024, 1024, [1000], [16], 20), {"Y_rows": 64, "dX_rows": 64, "Y_parts": 1}),
    # ... two groups: an odd and an even number of contraction tiles behind their LoRA tiles
    ((220, 1920, 2688, [22] * 9 + [21], [64] * 10, 0), {"Y_rows": 64, "dX_rows": 64}),
    ((300, 1984, 1216, [100, 190], [5, 100], 10), {"Y_rows": 64, "dX_rows": 64}),
    # ... contraction ranges
    ((60, 4096, 576, [37, 20], [16, 64], 1), {"Y_rows": 64, "Y_parts": 8}),
    ((60, 576, 4096, [37, 20], [12, 40], 1), {"dX_rows": 64, "dX_parts": 8}),
    # ... tiles that would leave one block to some CUs: no ranges, or half tiles in ranges
    ((3230, 4104, 384, [1600, 1600], [64, 33], 3), {"Y_rows": 64, "Y_parts": 1}),
    ((3230, 7248, 368, [1615, 1600], [64, 33], 3), {"Y": "halves", "Y_rows": 128, "Y_parts": 4}),
    ((3230, 368, 7248, [1615, 1600], [64, 33], 3), {"dX": "halves", "dX_rows": 128, "dX_parts": 4}),
    # ... weights of more than 32 MiB, features that are multiples of 64 and of 8, several tasks in a tile
    ((50, 4896, 4072, [7, 11, 20], [14, 33, 8], 2), {"Y_rows": 64, "dX_rows": 64}),
    ((90, 4096, 4608, [30, 0, 55], [16, 64, 5], 3), {"Y_rows": 64, "dX_rows": 64}),
    ((25, 1824, 10296, [12, 13], [16, 100], 0), {"Y_rows": 64, "dX_rows": 64}),
    # ... more than 64 tiles of 256 x 256
    ((2740, 368, 1600, [230] * 11 + [201], [64, 9, 16] * 4, 4), {"Y_rows": 64}),
    ((3191, 1232, 312, [1600, 1560], [32, 17], 4), {"dX_rows": 64}),
    # ... between three and four of them per CU: the general kernel's
    ((641, 200, 4504, [200, 203, 231], [64, 9, 16], 3), {"Y_rows": 64, "Y": "64"}),
    # ... no more than two tiles of 128 x 128 per CU, or a second round of whole tiles half full at most: its larger tiles, to rank 16
    ((2400, 152, 2128, [900, 33, 1450], [8, 16, 3], 3), {"Y": "128"}),
    ((2400, 152, 2128, [900, 33, 1450], [8, 17, 3], 3), {"Y": "halves"}),
    ((9268, 200, 1608, [4000, 33, 5000], [16, 8, 3], 20), {"Y": "128"}),
    ((9268, 200, 1608, [4000, 33, 5000], [16, 8, 17], 20), {"Y": "whole"}),
    # 16 x 64 tiles
    ((128, 256, 256, [60, 60], [8, 64], 4), {"Y_rows": 16, "dX_rows": 16}),
    # partial contraction tiles, one chunk more or less than a whole one; 64 x 64 tiles
    ((2900, 200, 712, [63, 65, 1, 2700], [8, 32, 33, 64], 3), {"Y_rows": 64}),
    ((600, 1016, 520, [63, 65, 1, 300], [8, 32, 33, 64], 3), {"Y_rows": 64, "dX_rows": 64}),
    ((600, 520, 1032, [63, 500], [9, 127], 3), {"Y_rows": 64, "dX_rows": 64}),
    ((60, 4040, 584, [37, 20], [16, 64], 1), {"Y_rows": 64}),
    ((60, 584, 4040, [37, 20], [12, 40], 1), {"dX_rows": 64}),
    ((3000, 8, 712, [2000, 900], [3, 17], 1), {"Y_rows": 64}),                 # a single, partial tile
    ((3000, 712, 8, [2000, 900], [3, 24], 1), {"dX_rows": 64}),
    # ... halves, in ranges and not, and whole tiles
    ((900, 2056, 5640, [256, 515], [8, 17], 30), {"Y": "halves", "Y_rows": 128}),
    ((900, 5640, 2056, [256, 515], [8, 16], 30), {"dX": "halves", "dX_rows": 128}),
    ((200, 5128, 4104, [80, 90], [16, 30], 3), {"Y": "halves", "dX": "halves", "Y_rows": 128, "dX_rows": 128}),
    ((9268, 136, 1032, [4000, 33, 5000], [128, 8, 33], 20), {"Y": "whole"}),
    ((9268, 1032, 136, [4000, 33, 5000], [128, 8, 33], 20), {"dX": "whole"}),
    ((9268, 56, 1032, [4000, 33, 5000], [64, 8, 16], 20), {"Y": "whole"}),      # ... of one partial tile
    ((9268, 1032, 56, [4000, 33, 5000], [64, 8, 16], 20), {"dX": "whole"}),
    ((9268, 120, 1032, [4000, 33, 5000], [64, 8, 16], 20), {"Y": "whole"}),
    ((9268, 1032, 184, [4000, 33, 5000], [64, 8, 16], 20), {"dX": "whole"}),
    ((9268, 632, 1032, [4000, 33, 5000], [64, 8, 16], 20), {"Y": "whole"}),
    ((9268, 1032, 632, [4000, 33, 5000], [64, 8, 20], 20), {"dX": "whole"}),
    # ... a single base tile before the LoRA tiles of ranks that are no multiple of 8, waves without a weight row in the last column
    ((17000, 264, 64, [9000, 33, 7900], [12, 5, 20], 20), {"dX": "whole"}),
    ((17000, 264, 40, [9000, 33, 7900], [12, 5, 100], 20), {"dX": "whole"}),
]

# Many tasks of few rows, whose rows are packed in pieces of 32 (half tiles, and 64 x 64 tiles of the general kernel): the
# tiles are those of the rows alone.  Empty tasks, tasks of one row, rows of no task before, between and after.
_MANY = [(5 * k) % 17 for k in range(60)]
_FEW = [(3 * k) % 16 for k in range(47)]
PACKED = [
    ("bf16", (494, 4096, 4096, _MANY, [1 + k % 30 for k in range(60)], 9), {"Y": "halves", "Y_tiles": 32, "dX_tiles": 32}),
    ("bf16", (494, 4104, 4104, _MANY, [8 * (1 + k % 4) for k in range(60)], 9), {"Y": "halves", "Y_tiles": 34, "dX_tiles": 34}),
    ("f32", (367, 2896, 388, _FEW, [1 + 3 * k % 20 for k in range(47)], 9), {"Y": "64", "Y_tiles": 42}),
    ("f32", (367, 388, 2896, _FEW, [1 + 3 * k % 20 for k in range(47)], 9), {"dX": "64", "dX_tiles": 42}),
    ("bf16", (367, 2501, 1003, _FEW, [1 + 3 * k % 20 for k in range(47)], 9), {"Y": "64", "Y_tiles": 96}),
    ("bf16", (367, 1003, 2501, _FEW, [1 + 3 * k % 20 for k in range(47)], 9), {"dX": "64", "dX_tiles": 96}),
]

# Low-rank products: few rows of deep contractions in ranges, in the general kernel (fp32, and features that are no
# multiple of 64) and in blocks of one wave; ranks above 64 that are no multiple of 4 in the general kernel
ROWS = [
    ("f32", (91, 3840, 388, [10, 0, 44, 30], [64, 3, 17, 40], 2), {"Z_rows": 16, "Z_parts": 16, "G_parts": 1}),
    ("f32", (90, 130, 4999, [50, 33], [64, 33], 2), {"G_rows": 16, "G_parts": 16}),
    ("f32", (700, 2480, 132, [600, 33], [9, 58], 2), {"Z_rows": 16, "Z_parts": 6}),
    ("bf16", (112, 4967, 132, [50, 33], [87, 16], 2), {"Z_rows": 16, "Z_parts": 16}),
    ("bf16", (112, 132, 4960, [50, 33], [128, 16], 2), {"G_rows": 16, "G_parts": 16}),
    ("bf16", (68, 9536, 64, [20, 1, 40], [15, 8, 3], 2), {"Z_rows": 32, "Z_parts": 16}),
    ("bf16", (68, 64, 4160, [20, 1, 40], [15, 64, 3], 2), {"G_rows": 32, "G_parts": 8}),
    ("bf16", (219, 1920, 128, [22] * 9, [114, 5, 70, 128, 1, 99, 66, 8, 33], 2), {"Z_rows": 16, "Z_parts": 8}),
    ("bf16", (4458, 640, 128, [100] * 43, [123, 64, 7] * 14 + [97], 2), {"Z_rows": 16, "Z_parts": 1}),
]


# Small backward calls, whose dX and gradients share a launch: every form of the product, with one range and several of
# either (grads_alone: the gradients' ranges where they have a launch to themselves)
SMALL_BACK = [(t, c, dict(w, shared=1)) for t, c, w in [
    ("f32", (128, 256, 256, [60, 60], [8, 5], 4), {"dX": "skinny", "grads": 1}),
    ("bf16", (400, 64, 64, [100, 0, 290], [16, 3, 8], 4), {"dX": "skinny", "grads": 1}),
    ("bf16", (1001, 70, 514, [980], [40], 13), {"dX": "skinny", "grads": 7, "grads_alone": 11}),
    ("f32", (714, 256, 64, [200, 300, 214], [8, 8, 8], 0), {"dX": "skinny", "grads": 4}),
    ("f32", (571, 1088, 256, [100, 371, 100], [46, 4, 2], 0), {"dX": "64"}),
    ("f32", (500, 700, 1001, [100, 390], [17, 4], 3), {"dX": "64", "dX_parts": 2, "grads": 5}),
    ("f32", (900, 300, 1500, [880], [64], 3), {"dX": "64", "dX_parts": 6, "grads": 10}),
    ("f32", (300, 2001, 501, [150, 140], [16, 3], 0), {"dX": "64", "grads": 1}),
    ("f32", (500, 701, 701, [500], [16], 0), {"dX": "64", "dX_parts": 5, "grads": 6}),
    ("bf16", (913, 1000, 1500, [300, 77, 513], [8, 10, 16], 5), {"dX": "64", "dX_parts": 1, "grads": 1}),
    ("bf16", (1500, 999, 1500, [1400], [50], 5), {"dX": "64", "dX_parts": 1, "grads": 9}),
    ("bf16", (913, 1024, 1536, [300, 77, 513], [8, 10, 16], 5), {"dX": "ring", "dX_parts": 1, "grads": 1, "grads_alone": 2}),
    ("bf16", (300, 1216, 1984, [100, 190], [32, 5], 10), {"dX": "ring", "dX_parts": 1, "grads": 1}),
    ("bf16", (60, 584, 4040, [37, 20], [12, 40], 1), {"dX": "ring", "dX_parts": 8, "grads": 1}),
    # two blocks of gradients in one of the two-group ring, an odd number of them
    ("bf16", (908, 768, 2624, [16, 8, 87, 48, 200, 15, 5, 100, 373, 28, 23, 5], [16, 3, 8] * 4, 0), {"dX": "ring", "dX_parts": 1, "grads": 1}),
    ("bf16", (908, 768, 2496, [16, 8, 87, 48, 90, 15, 5, 90, 90, 28, 23], [16] * 11, 4), {"dX": "ring", "dX_parts": 1, "grads": 1}),
    ("bf16", (1400, 2048, 192, [700, 691], [20, 8], 4), {"dX": "ring", "dX_parts": 1, "grads": 5, "grads_alone": 2}),
]]
# ... and calls of no more activation elements whose product runs in larger tiles: the gradients have their own launch, in
# its ranges, as without dX
APART = [(t, c, dict(w, shared=0)) for t, c, w in [
    ("bf16", (512, 4096, 4096, [512], [16], 0), {"dX": "halves", "grads": 2, "grads_alone": 2}),
    ("bf16", (256, 4096, 11008, [256], [16], 0), {"dX": "halves", "grads": 1, "grads_alone": 1}),
    ("bf16", (300, 5120, 5120, [300], [8], 0), {"dX": "halves"}),
    ("bf16", (150, 13824, 5120, [150], [8], 0), {"dX": "halves"}),
    ("bf16", (4000, 901, 99, [1000] * 4, [40] * 4, 0), {"dX": "128", "grads": 11, "grads_alone": 11}),
    ("bf16", (1000, 512, 512, [1000], [40], 0), {"grads": 3, "grads_alone": 3}),       # ranks above 32 in the aligned kernel
]]
