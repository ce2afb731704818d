"""Layers that the kernels for larger work take (tables streamed through LDS, samples sorted by cell), small
enough for the oracle, with the kernels that their calls reach.  test_gpu_streamed.py runs them;
test_routes_host.py checks, without a GPU, that they reach what they are listed for: the rules that choose a
kernel follow measured times and move."""
import random

SLAB, SLAB16, LANE = "forward_slab_kernel", "forward_slab_f16_kernel", "backward_input_lane_kernel"
LANE32, LANE32F = "forward_lane32_kernel", "forward_lane32_f32_kernel"
NARROW, GATHER = "forward_slab_narrow_kernel", "forward_gather_kernel"
IN_SLAB, IN_SLAB16, IN_NARROW = "backward_input_slab_kernel", "backward_input_slab_f16_kernel", "backward_input_slab_narrow_kernel"
IN_LANE32, IN_LANE32F = "backward_input_lane32_kernel", "backward_input_lane32_f32_kernel"
WALK, STREAM, COEF_GATHER = "backward_fused_kernel", "backward_coef_stream_kernel", "backward_coef_gather_kernel"

PAPER, PACKED = 0, 1

# B, n_in, n_out, G, storage, layout, kernel of the forward pass, kernels of both gradients
SHAPES = [
    # 64-output tiles: fewer rows than a tile's, ragged last tiles, every table type and layout
    (119, 428, 662, 13, "f32", PACKED, SLAB, (LANE, COEF_GATHER)),
    (130, 600, 818, 16, "f32", PACKED, SLAB, (LANE, COEF_GATHER)),
    (1300, 364, 132, 16, "f32", PAPER, SLAB, (LANE, COEF_GATHER)),
    (1025, 500, 260, 3, "f32", PAPER, SLAB, (LANE, STREAM)),
    (20000, 480, 9, 16, "f32", PACKED, SLAB, ("backward_input_gather_kernel", STREAM)),
    (228, 502, 1033, 10, "f16", PACKED, SLAB16, (IN_SLAB16, COEF_GATHER)),
    (169, 408, 1180, 16, "f16", PACKED, SLAB16, (IN_SLAB16, COEF_GATHER)),
    (228, 502, 1033, 10, "bf16", PACKED, SLAB, (IN_SLAB, COEF_GATHER)),
    (169, 408, 1180, 16, "bf16", PACKED, SLAB, (IN_SLAB, COEF_GATHER)),
    # tables that cannot be gathered (16-bit rows of 8 bytes, Alg. 1's layout): down to a single row
    (1, 128, 132, 16, "f16", PAPER, SLAB, (IN_SLAB, COEF_GATHER)),
    (300, 10, 220, 6, "f16", PAPER, SLAB, (IN_SLAB, COEF_GATHER)),
    (3, 64, 260, 8, "bf16", PAPER, SLAB, (IN_SLAB, COEF_GATHER)),
    (1, 234, 100, 30, "bf16", PAPER, NARROW, (IN_NARROW, COEF_GATHER)),
    (2, 300, 76, 34, "f16", PAPER, NARROW, (IN_NARROW, COEF_GATHER)),
    (1, 108, 180, 44, "bf16", PAPER, NARROW, ("backward_generic_kernel", COEF_GATHER)),
    (110, 160, 132, 40, "f16", PAPER, NARROW, (WALK, COEF_GATHER)),
    # 32-output tiles (packed, two slabs fit as stored) at both ends of their grids, tiles of 2048 rows
    (2049, 300, 100, 17, "f32", PACKED, LANE32F, (IN_LANE32F, STREAM)),
    (4100, 480, 37, 24, "f32", PACKED, LANE32F, (IN_LANE32F, STREAM)),
    (2047, 450, 200, 17, "bf16", PACKED, LANE32, (IN_LANE32, STREAM)),
    (3000, 460, 67, 34, "f16", PACKED, LANE32, (IN_LANE32, COEF_GATHER)),
    # 16-output tiles: the grids left to them, and the one slab at a time from 35 to 48
    (4097, 392, 21, 25, "f32", PACKED, NARROW, (IN_NARROW, STREAM)),
    (4100, 392, 20, 34, "f32", PAPER, NARROW, (IN_NARROW, STREAM)),
    (2000, 600, 72, 20, "f32", PAPER, NARROW, (IN_NARROW, COEF_GATHER)),
    (3400, 386, 36, 35, "f32", PACKED, NARROW, (WALK, COEF_GATHER)),
    (4300, 300, 40, 48, "f32", PAPER, NARROW, (WALK, COEF_GATHER)),
    (4300, 300, 140, 48, "bf16", PACKED, NARROW, (WALK,)),
    # both gradients from one walk: the 16-output range with dense cells, no slab at all, several blocks
    # of the batch (even and ragged outputs, one tile and several)
    (7000, 240, 72, 20, "f32", PAPER, NARROW, (WALK,)),
    (8914, 190, 18, 54, "f32", PACKED, GATHER, (WALK,)),
    (2330, 40, 12, 36, "f16", PAPER, NARROW, (WALK,)),
    (4619, 20, 12, 55, "bf16", PAPER, "forward_generic_kernel", (WALK,)),
    (1336, 98, 600, 63, "f16", PACKED, GATHER, (WALK, COEF_GATHER)),
    (958, 478, 135, 39, "bf16", PACKED, GATHER, (WALK, COEF_GATHER)),
    (1100, 160, 132, 41, "bf16", PAPER, NARROW, (WALK, COEF_GATHER)),
    (16384, 128, 128, 40, "f32", PACKED, NARROW, (WALK,)),
    (13000, 160, 67, 36, "f32", PACKED, NARROW, (WALK,)),
    (12289, 160, 132, 36, "f16", PACKED, NARROW, (WALK,)),
    # the sorted stream: one block at its longest and the first of two, wide rows of gy copied tile by tile
    (12288, 96, 132, 6, "f32", PACKED, SLAB, (LANE, STREAM)),
    (12289, 96, 132, 6, "f32", PACKED, SLAB, (LANE, STREAM)),
    (1500, 40, 2116, 9, "f32", PACKED, SLAB, (LANE, STREAM)),
]

# grad_x of 16-bit packed or 8-aligned tables where it streams them: B, n_in, n_out, G, storage, layout, kernel.  Edges of
# the tiles of rows and outputs, every pitch of a grid line, the smallest batch
INPUT_16BIT = [
    (1023, 2000, 65, 16, "f16", PACKED, IN_SLAB16), (1025, 1000, 260, 11, "f16", PACKED, IN_SLAB16),
    (2049, 600, 191, 16, "f16", PACKED, IN_SLAB16), (1023, 2000, 129, 3, "f16", PACKED, IN_SLAB16),
    (1025, 600, 200, 16, "f16", PAPER, IN_SLAB16), (3000, 600, 200, 6, "f16", PAPER, IN_SLAB16),
    (256, 2000, 129, 16, "bf16", PACKED, IN_LANE32), (1023, 2000, 97, 12, "bf16", PACKED, IN_LANE32),
    (1025, 2000, 67, 15, "bf16", PACKED, IN_LANE32), (1023, 2000, 260, 3, "bf16", PACKED, IN_LANE32),
    (1024, 1000, 100, 17, "bf16", PACKED, IN_LANE32), (2049, 1000, 65, 20, "bf16", PACKED, IN_LANE32),
    (1100, 1000, 100, 30, "bf16", PACKED, IN_LANE32), (1030, 1000, 130, 33, "bf16", PACKED, IN_LANE32),
    (1030, 1000, 130, 34, "bf16", PACKED, IN_LANE32), (3000, 1000, 33, 32, "bf16", PACKED, IN_LANE32),
]
# the same with unusual values in gy and tables, and with smooth tables
UNUSUAL_16BIT = [(600, 1000, 260, G, storage, PACKED, IN_SLAB16 if storage == "f16" and G <= 16 else IN_LANE32)
                 for storage in ("f16", "bf16") for G in (8, 16, 20, 24)]
SMOOTH_16BIT = [(2048, 400, 256, 16, "f16", PACKED, IN_SLAB16), (2048, 400, 256, 11, "f16", PACKED, IN_SLAB16),
                (2048, 400, 256, 16, "f16", PAPER, IN_SLAB16), (2048, 400, 256, 16, "bf16", PACKED, IN_LANE32),
                (2048, 400, 256, 11, "bf16", PACKED, IN_LANE32), (2048, 400, 256, 24, "bf16", PACKED, IN_LANE32)]

# tables in the layout of Alg. 1 whose rows lie so far apart that the rows of one load to LDS are 4 GiB apart: n_in, n_out,
# G, storage (batch 512; 23, 12 and 93 GB)
FAR_ROWS = [(32768, 22016, 3, "f32"), (32768, 22016, 3, "f16"), (16384, 8768, 17, "f32")]

# Forward pass of packed float32 tables from one slab at a time with the next one brought near (B, n_in, n_out, G).  One to six tiles
# of 4096 rows, the last one ragged, the fifth and sixth with the share of the first and second; one to sixteen tiles of 16 outputs and
# a count of 21 (the last one alone with its lines where there is one tile of rows); both ends of the range of grids
NEAR = [(9000, 512, 72, 41), (17000, 400, 100, 45), (20500, 150, 96, 48), (20000, 672, 12, 43), (4800, 564, 80, 41), (5000, 200, 256, 44),
        (2500, 300, 330, 48), (980, 260, 336, 35), (12400, 180, 100, 36), (7000, 300, 144, 38), (8192, 512, 16, 40), (4133, 564, 80, 41)]
# ... and as it was, on the other side of the rule: rows too few for the grid, nobody to share the lines with, runs of few pairs
NOT_NEAR = [(970, 260, 336, 35), (4096, 512, 16, 40), (4096, 1024, 13, 36), (4096, 500, 100, 48)]

# Tiles of 16 outputs (float32) that share lines of the table in groups of four and a rest, forward and grad_x: B, n_in, n_out, G, layout.
# One to seven tiles of 4096 rows, pairs split or not; grad_x has them side by side up to 16384 rows and in the last layer
SIDE_BY_SIDE = [(9000, 128, 100, 33, PACKED), (1500, 300, 130, 28, PACKED), (20000, 300, 72, 30, PACKED), (16384, 160, 48, 34, PACKED),
                (16385, 160, 48, 34, PACKED), (5000, 300, 100, 25, PACKED), (2000, 600, 72, 20, PAPER), (26000, 100, 200, 27, PACKED),
                (21000, 360, 130, 25, PACKED)]
# ... and of 32 outputs, grad_x of bfloat16 tables, in pairs and a rest (side by side from G = 17 on): B, n_in, n_out, G
SIDE_BY_SIDE_BF16 = [(2600, 900, 161, 30), (1100, 1000, 160, 17), (3000, 600, 416, 28), (1030, 1000, 130, 16), (3000, 300, 260, 12),
                     (16400, 300, 100, 20)]

# Coefficient gradient alone by the walk of sparse cells: B, n_in, n_out, G.  Streams uncut and in 2, 4, ... 64 runs, the largest batch of
# several of them, two and three blocks, ragged and even outputs, wide rows of gy copied tile by tile, the finest grid
SPARSE = [(2001, 256, 2050, 20), (1371, 1000, 448, 14), (447, 800, 1000, 8), (1878, 700, 333, 17), (2600, 700, 260, 28), (3311, 300, 256, 24),
          (4499, 200, 128, 30), (3001, 130, 261, 64), (5779, 100, 131, 37), (8379, 36, 85, 62), (12289, 130, 66, 46), (20000, 260, 40, 48)]
# ... and by the one of whole chunks: one more row, a small gradient, blocks of more samples or in more runs
NOT_SPARSE = [(1372, 1000, 448, 14), (448, 800, 1000, 8), (3312, 300, 256, 24), (4500, 200, 128, 30), (3000, 64, 64, 30), (12290, 128, 130, 45),
              (12289, 40, 66, 50), (1791, 400, 192, 16), (1792, 400, 192, 16), (1100, 600, 333, 13), (4031, 300, 65, 24), (12290, 64, 130, 44)]

# walks that are not cut into runs: a gradient that one wave writes repeats bit for bit
WHOLE_STREAMS = (2000, 512, 1024, 8)
# grad_x of the walk over the sorted samples repeats bit for bit, with the coefficient gradient and without
WALKS = [(16384, 128, 128, 40), (3400, 386, 36, 35)]

# as SHAPES, for a convolution: images, H, W, C, window, stride, n_out, G, storage, layout, kernels: the walk over
# the sorted samples writes the transposed gradient of a layer on windows
CONV = [
    (9, 23, 24, 30, 2, 1, 130, 40, "f32", PACKED, NARROW, (WALK, "conv_input_gradient_kernel")),
    (300, 9, 9, 15, 2, 2, 260, 37, "f32", PAPER, NARROW, (WALK, "conv_input_gradient_scatter_kernel")),
    # 64-output tiles: windows side by side, over odd channel counts (pairs straddle pixels), overlapping, with
    # pixels that no window holds, single pixels
    (20, 32, 32, 60, 2, 2, 126, 8, "f32", PACKED, SLAB, (LANE, STREAM)),
    (40, 22, 23, 51, 2, 2, 128, 12, "f32", PAPER, SLAB, (LANE, STREAM)),
    (8, 24, 24, 20, 3, 1, 100, 16, "f32", PACKED, SLAB, (LANE, STREAM)),
    (60, 28, 29, 40, 3, 3, 184, 16, "f16", PACKED, SLAB16, (IN_SLAB16, STREAM)),
    (24, 16, 16, 200, 1, 1, 128, 10, "f32", PACKED, SLAB, (LANE, STREAM)),
    (7, 20, 20, 24, 3, 1, 140, 12, "f16", PAPER, SLAB, (IN_SLAB, STREAM)),
    # 32-output and 16-output tiles
    (20, 18, 18, 40, 3, 1, 62, 20, "f32", PACKED, LANE32F, (IN_LANE32F, STREAM)),
    (20, 18, 18, 40, 3, 1, 94, 28, "bf16", PACKED, LANE32, (IN_LANE32, STREAM)),
    (20, 18, 19, 40, 3, 1, 62, 26, "f32", PACKED, NARROW, (IN_NARROW, STREAM)),
]


# Forward pass and both gradients at every grid that some slab fits: a layer per grid, storage type, layout and
# output count rotating with G
def every_grid(G):
    storage, layout = ("f32", "f16", "bf16")[G % 3], (PACKED, PAPER)[(G // 3) % 2]
    B, n_in, n_out = (1300, 600, 124) if G <= 16 else (2100, 400, 100) if G <= 34 else (3400, 386, 60)
    if storage != "f32":
        n_out += 64 if G <= 16 else 100
        layout = PAPER if G <= 12 else layout     # (smaller 16-bit tables are gathered; 188 outputs cannot be)
    return B, n_in, n_out + ((0, 1, 2, 3)[G % 4] if layout == PACKED else 0), G, storage, layout


# Layers drawn at random from those that are more work than the gathers take: batch, sizes, grid, storage, layout, which
# gradients ("both", "x", "coef"), whether the coefficient gradient is added to one that is there
def drawn(n, seed):
    rng, out = random.Random(seed), []
    while len(out) < n:
        B, n_in = round(100 * 150 ** rng.random()), 2 * rng.randint(60, 300)
        n_out, G = rng.choice([rng.randint(9, 64), rng.randint(100, 128), rng.randint(30, 700)]), rng.choice([rng.randint(3, 16), rng.randint(17, 34), rng.randint(35, 48)])
        storage, layout = rng.choice(["f32", "f32", "f16", "bf16"]), rng.choice([PAPER, PACKED, PACKED])
        if layout == PAPER:
            n_out = (n_out + 3) // 4 * 4
        if not 2e7 < B * n_in // 2 * n_out < 8e7 or (G + 1) ** 2 * n_in // 2 * n_out > 4e7:
            continue
        grads = rng.choice(["both", "both", "x", "coef"])
        out.append((B, n_in, n_out, G, storage, layout, grads, grads != "x" and rng.random() < 0.5))
    return out


DRAWN = drawn(60, 20260101)

# layers recorded into a graph: partial outputs, tiles of every kind, runs that meet through atomics, blocks
REPLAYED = [(1025, 500, 260, 3, "f32", PAPER), (169, 408, 1180, 16, "f16", PACKED), (2049, 300, 100, 17, "f32", PACKED),
            (4097, 392, 21, 25, "f32", PACKED), (3400, 386, 36, 35, "f32", PACKED), (13000, 160, 67, 36, "f32", PACKED),
            (12289, 96, 132, 6, "f32", PACKED)]
