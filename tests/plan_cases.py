"""Shapes of the GPU tests of the tiled matrix products and the tiles they are there for (rows, weight rows, in several parts):
test_rows_plan.py checks that the plan still takes them, test_gpu_parity.py runs them."""

# d_model, vocabulary, rows: the output head's tile
HEAD_TILES = [
    (256, 2111, 5, (16, 128, False)),
    (2048, 2111, 12, (16, 128, True)),
    (256, 16000, 17, (32, 128, False)),
    (2048, 2111, 17, (32, 128, True)),
    (256, 8000, 130, (64, 128, False)),
    (2048, 4000, 40, (64, 128, True)),
    (256, 33000, 5, (64, 256, False)),    # few rows, more than a round of narrow blocks
    (256, 66000, 17, (128, 384, False)),
    (2048, 33000, 100, (128, 384, True)),
    (256, 131072, 17, (128, 512, False)),
    (256, 131072, 130, (256, 256, False)),
    # reductions of an odd number of 32s, the half step in the last of several parts
    (2016, 2111, 12, (16, 128, True)),
    (2080, 2111, 17, (32, 128, True)),
    (2080, 4000, 40, (64, 128, True)),
]

# d_model, d_ffn, rows: the tiles of the 2d -> d projection, gate/up and the down projection (query heads of 128, d / 128 of them)
BODY_TILES = [
    (2048, 6144, 12, ((16, 128, True), (16, 128, False), (16, 128, True))),
    (1824, 6112, 9, ((16, 128, True), (16, 128, False), (16, 128, True))),  # half steps
    (2048, 6144, 17, ((32, 128, True), (32, 128, False), (32, 128, True))),
    (2048, 6144, 33, ((64, 128, True), (32, 128, False), (64, 128, True))),
    (2048, 6144, 400, ((64, 256, True), (128, 384, False), (128, 384, True))),
    (2080, 6176, 17, ((32, 128, True), (32, 128, True), (32, 128, True))),  # half steps, but for the projection
    (2048, 16384, 400, ((64, 256, True), (256, 256, False), (256, 256, True))),
]

# d_model, ((rows, rows of the list), ...): lists of a larger batch that few_rows.h serves with row-major activations
LIST_GROUPS = [
    (2304, ((7, 8195), (8, 7000), (9, 17000), (16, 8300))),
]
