"""Shapes (p, q, k, batch) that reach every form of the short-block FC kernel in fp32 and in 16-bit storage, forward and
backward-data: tests/test_dispatch_host.py checks on the CPU that they do, tests/test_gpu_parity.py the results.
Block rows, input blocks and batch rows leave remainders of the kernel's tiles (16 or 32 block rows, 16 batch rows) and
steps (4 input blocks per wave)."""

# (tiles of 16 block rows per workgroup, reduction cut into slices) -> shapes
ONE_TILE, TWO_TILES, SLICED = (1, False), (2, False), (1, True)
CASES = [
    ((17, 130, 4, 17), ONE_TILE), ((65, 33, 4, 2731), TWO_TILES), ((4, 700, 4, 18), SLICED),
    ((33, 31, 8, 33), ONE_TILE), ((66, 33, 8, 2731), TWO_TILES), ((5, 520, 8, 19), SLICED),
    ((33, 34, 16, 450), ONE_TILE), ((31, 5, 16, 700), ONE_TILE), ((47, 19, 16, 4451), TWO_TILES), ((70, 9, 16, 3000), TWO_TILES),
    ((7, 260, 16, 20), SLICED),
    ((33, 9, 32, 790), ONE_TILE), ((3, 1, 32, 1307), ONE_TILE), ((40, 66, 32, 700), ONE_TILE), ((5, 721, 32, 19), SLICED),
    ((3, 811, 32, 35), SLICED),
]
