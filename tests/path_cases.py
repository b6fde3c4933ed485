"""Shapes that take the bf16 products along named paths: the GPU tests run them against the oracle, test_launches.py checks on
the CPU that today's choice of kernels takes each of them there.  A case is (T, d, f, E, k, options of run_layer_and_check);
the paths are {product: (rows of a tile, form of the last k tile, K slices of the last round)}, the slices for rows spread evenly
over the experts (and cut off by the capacity limit)."""
from paper_2403_07816_amd import binding as B

UP, DOWN, BWD_ACT, BWD_DX, DW13, DW2 = range(6)
SWITCH = dict(mode=B.BTX_ROUTE_SWITCH_TOP1)
WHOLE, HALF, ANY = 0, 1, 2          # K a multiple of 64; 32 more; any other multiple of 8

LAST_ROUND_CUT = [
    # DOWN and both K passes of BWD_DX
    ((2050, 1032, 8192, 2, 1, SWITCH), {DOWN: (256, WHOLE, 5), BWD_DX: (256, WHOLE, 5)}),
    ((2050, 1032, 8224, 2, 1, SWITCH), {DOWN: (256, HALF, 5), BWD_DX: (256, HALF, 5)}),
    ((2050, 1032, 8232, 2, 1, dict(SWITCH, cf=0.9, bias=[0.5, 0.0])), {DOWN: (256, ANY, 6), BWD_DX: (256, ANY, 6)}),
    ((1200, 2056, 4104, 12, 2, dict(cf=1.0)), {DOWN: (256, ANY, 2), BWD_DX: (256, ANY, 2)}),
    # UP, whose finishing kernel applies the SwiGLU
    ((2050, 4096, 1160, 2, 1, SWITCH), {UP: (256, WHOLE, 2)}),
    ((2050, 4128, 1160, 2, 1, SWITCH), {UP: (256, HALF, 2)}),
    ((2050, 4104, 1160, 2, 1, dict(SWITCH, cf=0.9, bias=[0.5, 0.0])), {UP: (256, ANY, 3)}),
    # 192 rows, the third LDS stage on the weights
    ((260, 4096, 768, 16, 8, {}), {UP: (192, WHOLE, 2)}),
    ((260, 4104, 768, 16, 8, {}), {UP: (192, ANY, 2)}),
    ((260, 1536, 4096, 16, 8, dict(cf=0.9)), {DOWN: (192, WHOLE, 2), BWD_DX: (192, WHOLE, 2)}),
    ((260, 1544, 4104, 16, 8, {}), {DOWN: (192, ANY, 2), BWD_DX: (192, ANY, 2)}),
    ((280, 4104, 1160, 16, 8, {}), {BWD_DX: (192, ANY, 2)}),
]


def whole_tile_case(i):
    """Seeded random shapes whose row-grouped products all run 256-row tiles; BWD_DX cuts its last round."""
    import numpy as np
    rng = np.random.default_rng(2000 + i)
    E, k = [(2, 1), (3, 2), (3, 1)][i % 3]
    T = int(rng.integers(10300, 13000)) // k
    d, f = (8 * int(rng.integers(130, 160)) for _ in range(2))
    return T, d, f, E, k


WHOLE_TILE_CASES = 6

# contractions of 1 to 6 k tiles in 256-row tiles, where the main loop gives way to its last k tiles: UP and BWD_ACT (few columns of x),
# DOWN and both passes of BWD_DX (narrow experts)
FEW_K_TILES = [((12300, d, 1032, 2, 1, SWITCH), (UP, BWD_ACT)) for d in (64, 72, 128, 160, 192, 248, 256, 384)] + \
              [((12300, 1032, f, 2, 1, SWITCH), (DOWN, BWD_DX)) for f in (64, 72, 128, 160, 192, 248, 256, 320)]

# weight gradients from transposed rows: more than 8 experts, experts without rows, dropped pairs; dW2 streamed and not
TRANSPOSED_ROWS = [
    (2200, 264, 2056, 12, 2, dict(cf=0.8, poison=True)), (2200, 320, 2056, 12, 2, dict(cf=0.8, poison=True)),
    (1100, 136, 2056, 3, 1, dict(bias=[0.0, -60.0, 0.0], poison=True)), (6100, 64, 2056, 33, 2, dict(bias=[0.0] * 32 + [-60.0], poison=True)),
    (1500, 520, 3608, 4, 1, dict(bias=[3.0, 0.0, 0.0, 0.0], poison=True)),
]

# small fp32 layers, both products of the forward pass in one launch: 1 to 17 rows of a tile of 16; widths below, at and past one and
# several pieces of 64, contractions that end inside 16; dropped pairs, experts without rows; as many slices as the combine takes
JOINT_FORWARD = [
    (1, 8, 8, 1, 1, {}), (15, 64, 64, 1, 1, {}), (16, 72, 72, 1, 1, {}), (17, 56, 120, 1, 1, {}), (33, 192, 136, 2, 1, {}),
    (64, 128, 56, 4, 2, dict(poison=True)), (512, 64, 176, 4, 2, dict(cf=0.8, poison=True)), (90, 136, 320, 64, 4, dict(poison=True)),
    (40, 184, 776, 2, 2, dict(poison=True)), (100, 24, 1376, 3, 2, dict(bias=[4.0, 0.0, -60.0])), (1270, 192, 192, 3, 1, {}), (50, 40, 512, 8, 8, {}),
]

# fp32 forward products in two launches just past what takes one: contractions of one short k tile and widths below a tile's, experts of
# uneven numbers of rows, dropped pairs -> is DOWN cut along K; its slices added by the combine, and by a kernel of their own (12 slots)
TILED_FORWARD = [
    ((5700, 136, 8, 3, 2, dict(poison=True)), False), ((300, 264, 8, 3, 2, dict(cf=0.8, poison=True)), False), ((16100, 8, 8, 1, 1, {}), False),
    ((2700, 8, 136, 2, 2, dict(bias=[1.0, 0.0])), True), ((2700, 24, 136, 3, 2, dict(cf=0.8, poison=True)), True), ((1800, 72, 184, 4, 3, {}), False),
    ((330, 72, 1032, 4, 2, dict(poison=True)), True), ((300, 136, 1032, 2, 2, dict(cf=0.8, poison=True)), True), ((130, 200, 776, 4, 2, dict(cf=0.8, poison=True)), True),
    ((30, 264, 1384, 12, 12, dict(poison=True)), True), ((620, 8, 3000, 3, 2, dict(bias=[0.0, 0.0, -60.0])), True),
]

# weight gradients of tiles whose dW2 reads dY's token rows (d E from 4096 on, up to 4096 columns): experts of 0, 1 and a few k tiles beside
# long ones, remainders of a k tile, one and several column tiles, tokens of several slots, dropped pairs; and those that read them transposed
DY_ROWS = [
    (1001, 4104, 1304, 1, 1, {}), (8100, 256, 1400, 16, 1, dict(bias=[2.0, 0.0, -60.0, -3.0] + [0.0] * 12, poison=True)),
    (1700, 1032, 3208, 4, 1, dict(bias=[5.0, 0.0, 0.0, -60.0], poison=True)), (1000, 1376, 2056, 3, 2, dict(cf=0.8, poison=True)),
    (1700, 520, 1496, 9, 5, dict(bias=[0.0] * 8 + [-3.0], poison=True)),
]
DY_TRANSPOSED = [
    (500, 264, 6152, 1, 1, {}), (420, 72, 6400, 2, 2, dict(bias=[3.0, 0.0], poison=True)),
    (1001, 64, 1400, 1, 1, {}), (1088, 264, 1400, 1, 1, {}), (1500, 520, 3608, 4, 1, dict(bias=[5.0, 0.0, 0.0, -60.0], poison=True)),
    (1000, 1032, 2056, 3, 2, dict(cf=0.8, poison=True)), (1300, 248, 1496, 9, 5, dict(bias=[0.0] * 8 + [-3.0], poison=True)),
]

# fp32 DOWN whose last round of tiles is cut along K: last k tiles of 8, 16 and 32, column tiles of 24 to 64; experts of uneven numbers of
# rows (other numbers of tiles than expected: more slices, fewer, none), dropped pairs
F32_LAST_ROUND = [
    (592, 864, 552, 2, 2, {}), (634, 544, 528, 4, 3, dict(cf=0.9)), (808, 640, 552, 3, 2, dict(bias=[1.0, 0.0, 0.0])), (2176, 496, 576, 5, 1, {}),
    (649, 728, 648, 8, 2, dict(bias=[2.0, 1.0] + [0.0] * 6)), (933, 568, 528, 4, 2, dict(bias=[0.0, 0.0, 0.0, -60.0])),
]

# bf16 experts on both sides of the widths whose rows of act, dh1, dh3 and ga start on whole lines; ga in row order longer than transposed
ROW_PITCH = [
    (70, 72, 128, 2, 1, {}), (70, 72, 136, 2, 1, {}), (300, 264, 136, 4, 2, dict(cf=0.8)), (2300, 1032, 136, 2, 1, {}), (5000, 264, 136, 1, 1, {}),
    (40, 64, 65536, 2, 1, {}), (40, 64, 65544, 2, 1, {}), (600, 64, 65536, 1, 1, {}), (600, 72, 65544, 1, 1, {}),
]

# few tokens' routing with the normalisation, two pieces of wide rows requested ahead: (T, d, E, k, dtype).  Rows that end inside the
# second piece, at its end and behind it; passes over 2, 4 and 8 experts, whole or not, one and two of them
ROUTE_AHEAD = [
    (30, 4096, 1, 1, B.BTX_F32), (30, 2064, 2, 1, B.BTX_BF16), (512, 4088, 3, 2, B.BTX_F32), (16, 2056, 4, 2, B.BTX_BF16), (256, 6144, 4, 2, B.BTX_BF16),
    (70, 2056, 5, 2, B.BTX_BF16), (16, 4104, 6, 2, B.BTX_BF16), (70, 3080, 7, 3, B.BTX_F32), (512, 4096, 8, 2, B.BTX_F32), (512, 8192, 8, 2, B.BTX_BF16),
    (300, 6152, 8, 2, B.BTX_BF16), (33, 8192, 16, 4, B.BTX_BF16), (70, 2056, 16, 9, B.BTX_BF16),
]

# many tokens' routing: (T, d, E, k, dtype, with the normalisation) -> experts of a pass over the columns, wavefronts that share 16
# tokens.  Ragged last blocks; one workgroup on a compute unit, two, more.
ROUTE_MANY = [
    ((1030, 136, 1, 1, B.BTX_BF16, True), (1, 16)), ((1030, 136, 2, 2, B.BTX_BF16, True), (2, 16)), ((1030, 4104, 3, 2, B.BTX_BF16, True), (4, 16)),
    ((1035, 4096, 4, 2, B.BTX_BF16, True), (4, 16)), ((1030, 1032, 5, 2, B.BTX_BF16, True), (8, 8)), ((1030, 520, 40, 3, B.BTX_BF16, True), (8, 16)),
    ((4203, 136, 3, 2, B.BTX_BF16, True), (4, 8)), ((8190, 72, 2, 1, B.BTX_BF16, True), (2, 4)),
    ((1030, 136, 1, 1, B.BTX_F32, True), (1, 16)), ((1030, 520, 2, 1, B.BTX_F32, True), (2, 8)), ((1030, 136, 3, 2, B.BTX_F32, True), (4, 16)),
    ((1030, 1032, 5, 2, B.BTX_F32, True), (8, 8)), ((1030, 8200, 2, 1, B.BTX_F32, True), (2, 4)), ((1030, 8200, 3, 2, B.BTX_F32, True), (4, 4)),
    ((1030, 8200, 7, 2, B.BTX_F32, True), (8, 4)), ((4203, 4104, 8, 2, B.BTX_F32, True), (8, 4)),
    ((1030, 136, 1, 1, B.BTX_BF16, False), (1, 8)), ((1030, 1032, 2, 1, B.BTX_BF16, False), (2, 8)), ((1030, 136, 3, 2, B.BTX_BF16, False), (4, 8)),
    ((4203, 72, 2, 2, B.BTX_BF16, False), (2, 4)), ((1030, 136, 1, 1, B.BTX_F32, False), (1, 8)), ((1030, 520, 2, 1, B.BTX_F32, False), (2, 8)),
    ((1030, 8200, 2, 1, B.BTX_F32, False), (2, 4)), ((1030, 8200, 3, 2, B.BTX_F32, False), (4, 4)), ((1030, 8200, 7, 2, B.BTX_F32, False), (8, 4)),
    ((520, 4096, 5, 2, B.BTX_BF16, False), (8, 8)), ((520, 4096, 5, 2, B.BTX_BF16, True), (8, 8)), ((1024, 4096, 1, 1, B.BTX_F32, False), (1, 8)),
]
