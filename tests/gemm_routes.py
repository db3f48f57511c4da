"""Shapes (M, N, K, block) of the dequantise-on-load GEMM by the kernel that runs
them on 256 compute units, as tests/c/gemm_plan.cpp names it: every variant of
every kernel, with rows and columns that no tile divides.  The CPU test asserts
the names; the GPU tests run the shapes."""

ROUTES = [
    # k_dqrows: weight-row tiles, waves, x staged in LDS, sets of accumulators
    ("rows:1x1,waves8,staged,sets2", 1, 305, 448, 128), ("rows:1x1,waves8,staged,sets2", 5, 2049, 2112, 64),
    ("rows:1x2,waves16,sets2", 15, 434, 1728, 512), ("rows:1x2,waves16,sets2", 16, 6145, 2048, 256),
    ("rows:1x3,waves8", 15, 8193, 1728, 256), ("rows:1x3,waves8,staged,sets2", 1, 16396, 448, 1024),
    ("rows:1x4,waves8", 15, 12461, 1728, 1024), ("rows:1x5,waves8", 15, 16585, 1728, 64),
    ("rows:1x6,waves8", 15, 20697, 1728, 256), ("rows:1x6,waves8", 16, 24560, 1664, 512),
    ("rows:2x2,waves8", 17, 65, 704, 32), ("rows:2x2,waves8,sets2", 20, 677, 3264, 512),
    ("rows:2x3,waves8,sets2", 17, 8344, 448, 32), ("rows:2x4,waves8,sets2", 31, 12503, 448, 128),
    ("rows:2x5,waves8,sets2", 17, 16481, 448, 256), ("rows:2x6,waves8,sets2", 17, 20577, 448, 256),
    ("rows:2x6,waves8,sets2", 32, 24550, 704, 128),
    ("rows:4x2,waves4", 129, 8172, 448, 32), ("rows:4x2,waves4,sets2", 523, 1430, 4288, 32),
    ("rows:4x2,waves8", 48, 301, 448, 512), ("rows:4x2,waves8,sets2", 35, 129, 2240, 1024),
    ("rows:4x3,waves4", 67, 4097, 448, 64), ("rows:4x3,waves4,sets2", 67, 4098, 960, 1024),
    ("rows:4x4,waves4", 65, 6241, 448, 512), ("rows:4x4,waves4,sets2", 66, 6252, 1600, 512),
    ("rows:4x5,waves4,sets2", 67, 8204, 448, 64), ("rows:4x6,waves4,sets2", 65, 10296, 448, 32),
    ("rows:4x6,waves4,sets2", 63, 24561, 576, 256),
    # the same with K in ranges, added into y
    ("ranges:1x6,waves8,sets2", 15, 3071, 9280, 512), ("ranges:2x6,waves8,sets2", 23, 1000, 8640, 1024),
    # k_dqgemv: longest range of K
    ("stream:256", 7, 4, 64, 64), ("stream:256,split", 16, 64, 4160, 256), ("stream:512,split", 1, 839, 37568, 32),
    ("stream:1024,split", 3, 1987, 31808, 128),
    # k_dqgemm_pp: tiles of y, whole K and split
    ("tiles:128x256", 17, 49222, 448, 64), ("tiles:128x256,split", 50, 300, 2752, 1024),
    ("tiles:256x256", 263, 24683, 448, 32), ("tiles:256x256", 513, 16390, 64, 256),
    ("tiles:256x256,split", 131, 10962, 3520, 1024), ("tiles:256x192", 130, 13924, 448, 256),
    ("tiles:256x192,split", 142, 261, 4160, 64), ("tiles:256x128", 976, 2572, 448, 64),
    ("tiles:256x128,split", 700, 257, 6144, 128),
    # k_dqgemm
    ("plain", 17, 3, (1 << 21) + 256, 256),
]
