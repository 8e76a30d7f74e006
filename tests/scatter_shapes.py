"""Layers (tokens, columns, blocks, units, blocks per token) by what the K = Bs contraction's planner chooses for them: tiles of 16 rows
per record, whether the block list is in parts, and the pieces of a run that holds every token of its range.  Four wavefronts share a
workgroup's records, so that with five pieces or more a wavefront meets a later piece of the run it has had one of; a part of the block list
can begin in the middle of a run.  tests/test_scatter_layout.py pins the choice, tests/test_gpu_scatter.py runs them with two blocks that every
token takes: every number of tiles, each block size, with and without parts."""

# (tiles, parts > 1, pieces of a full run, layer)
LAYERS = [
    (2, False, 1, (101, 64, 16, 32, 2)), (2, True, 1, (104, 64, 40, 32, 2)),
    (2, False, 1, (101, 64, 12, 64, 2)), (2, True, 1, (118, 64, 44, 64, 2)),
    (2, False, 1, (100, 64, 19, 96, 2)), (2, True, 1, (106, 64, 32, 96, 2)),
    (2, False, 1, (102, 64, 14, 128, 2)), (2, True, 1, (135, 64, 36, 128, 2)),
    (4, False, 6, (2243, 2112, 26, 32, 2)), (4, True, 6, (3375, 768, 57, 32, 3)),
    (4, False, 5, (5741, 768, 30, 64, 2)), (4, True, 8, (3362, 384, 123, 64, 4)),
    (4, False, 5, (1589, 2432, 17, 96, 2)), (4, True, 6, (1306, 640, 102, 96, 3)),
    (4, False, 5, (1301, 3008, 18, 128, 2)), (4, True, 5, (2151, 256, 143, 128, 5)),
    (6, False, 7, (6335, 1600, 26, 32, 3)), (6, True, 3, (814, 1792, 138, 32, 42)),
    (6, False, 6, (2580, 3008, 25, 64, 3)), (6, True, 6, (1465, 1728, 91, 64, 11)),
    (6, False, 6, (4871, 1536, 13, 96, 2)), (6, True, 6, (1561, 704, 154, 96, 18)),
    (6, False, 6, (5322, 1408, 12, 128, 2)), (6, True, 6, (4170, 512, 64, 128, 9)),
    (8, False, 5, (4438, 2304, 20, 32, 3)), (8, True, 3, (5332, 640, 139, 32, 40)),
    (8, False, 5, (5683, 1728, 12, 64, 2)), (8, True, 2, (967, 1792, 49, 64, 29)),
    (8, False, 4, (4280, 1472, 18, 96, 5)), (8, True, 5, (2070, 1344, 106, 96, 22)),
    (8, False, 5, (5061, 1984, 13, 128, 2)), (8, True, 4, (2711, 384, 131, 128, 32)),
    (10, False, 4, (8867, 1152, 27, 32, 6)), (10, True, 2, (2707, 1792, 140, 32, 66)),
    (10, False, 4, (8866, 1152, 26, 64, 6)), (10, True, 2, (10011, 128, 111, 64, 64)),
    (10, False, 4, (11381, 896, 24, 96, 5)), (10, True, 2, (10570, 192, 90, 96, 48)),
    (10, False, 4, (3797, 2624, 19, 128, 4)), (10, True, 4, (10559, 128, 154, 128, 41)),
]

# ... of the low-rank pass, whose token rows are added when a slab is written out (or with the parts' sums): one slab for all wavefronts.
LORA_LAYERS = [
    (4, True, 6, (1306, 640, 102, 96, 3)), (6, False, 3, (974, 2944, 12, 64, 4)),
]

# (dX and both weight gradients in one launch, tokens, columns, blocks, units, blocks per token, uneven routing): every block size, one and
# several column tiles, ragged ones, few and many pieces; slabs of 80 KB and the next larger ones, more than two workgroups a CU and up to
# 20000 rows, and more of either, which are launches of their own.
JOINED = [
    (True, 33, 192, 17, 128, 5, False), (True, 512, 256, 16, 64, 4, True), (True, 300, 320, 24, 32, 5, True),
    (True, 777, 192, 9, 96, 3, False), (True, 1900, 448, 12, 128, 3, True), (True, 1300, 512, 12, 96, 6, True),
    (True, 1024, 1024, 32, 128, 8, False), (True, 5000, 64, 7, 32, 2, False), (True, 1250, 1024, 20, 64, 5, False),
    (False, 1270, 1024, 20, 64, 5, False),
    (True, 1024, 1856, 7, 32, 3, False), (False, 1892, 1024, 57, 32, 29, False), (False, 10472, 512, 99, 32, 1, False),
]
