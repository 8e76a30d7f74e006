"""Layers (tokens, columns, blocks, units, blocks per token) by what the K = Bs contraction's planner chooses for them: tiles of 16 rows
per record, whether the block list is in parts, and the pieces of a run that holds every token of its range.  Four wavefronts share a
workgroup's records, so that with five pieces or more a wavefront meets a later piece of the run it has had one of.  tests/test_scatter_layout.py
pins the choice, tests/test_gpu_scatter.py runs them with blocks that every token takes."""

# (tiles, parts > 1, pieces of a full run, layer)
LAYERS = [
    (4, False, 6, (2243, 2112, 26, 32, 2)), (4, True, 6, (3375, 768, 57, 32, 3)),
    (4, False, 5, (5741, 768, 30, 64, 2)), (4, True, 8, (3362, 384, 123, 64, 4)),
    (4, False, 5, (1589, 2432, 17, 96, 2)), (4, True, 6, (1306, 640, 102, 96, 3)),
    (4, False, 5, (1301, 3008, 18, 128, 2)), (4, True, 5, (2151, 256, 143, 128, 5)),
]
