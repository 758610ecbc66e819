"""K-major bf16 products for every kernel and tile that the launcher chooses from, once with whole k-steps and once ending in
half a step, ragged in both directions where a tile allows it.  The route is asserted on the CPU (test_dispatch_host.py)
for the epilogues that the values are checked with on the GPU (test_gpu_ops.py), so the list cannot go stale unseen.
Entries: (M, N, K, kernel, its leading template arguments)."""
SPLIT, RING, RING16, PP = ("gemm_bf16_split_kernel", "gemm_bf16_w48s_kernel", "gemm_bf16_w48_kernel",
                           "gemm_bf16_pingpong_kernel")
SHAPES = [
    # split kernel: blocks of 16 rows and columns of the tile
    (32, 64, 192, SPLIT, (1, 1)), (64, 32, 352, SPLIT, (1, 1)),
    (416, 160, 192, SPLIT, (1, 2)), (416, 160, 352, SPLIT, (1, 2)),
    (160, 832, 192, SPLIT, (2, 2)), (96, 1376, 352, SPLIT, (2, 2)),
    (224, 1184, 192, SPLIT, (2, 3)), (416, 640, 352, SPLIT, (2, 3)),
    (2080, 160, 192, SPLIT, (2, 4)), (2080, 160, 352, SPLIT, (2, 4)),
    (4192, 96, 192, SPLIT, (4, 2)), (1184, 416, 352, SPLIT, (4, 2)),
    (864, 608, 192, SPLIT, (4, 3)), (1184, 448, 352, SPLIT, (4, 3)),
    (288, 2528, 192, SPLIT, (4, 4)), (224, 3168, 352, SPLIT, (4, 4)),
    (864, 1184, 1088, SPLIT, (4, 6)), (928, 1120, 1056, SPLIT, (4, 6)),
    # producer/consumer rings: 128x96, 128x128, 128x144, 128x192, 256x144
    (544, 1824, 192, RING, (2, 2, 3)), (352, 2976, 352, RING, (2, 2, 3)),
    (1056, 992, 192, RING, (2, 2, 4)), (1120, 928, 352, RING, (2, 2, 4)),
    (1984, 2304, 64, RING, (2, 3, 3)), (1984, 2304, 96, RING, (2, 3, 3)),
    (1632, 2496, 192, RING, (2, 4, 3)), (3552, 1344, 352, RING, (2, 4, 3)),
    (2976, 2880, 192, RING, (4, 3, 3)), (3520, 2592, 352, RING, (4, 3, 3)),
    # 256x192 tiles of single k-steps
    (3968, 3072, 64, RING16, (4, 4)), (3968, 3072, 32, RING16, (4, 4)),
    # ping-pong kernel: 256x128, 256x192, 256x256
    (1184, 3392, 192, PP, (4, 2, 2, 2)), (1440, 2752, 352, PP, (4, 2, 2, 2)),
    (2464, 3360, 192, PP, (4, 2, 2, 3)), (3200, 2624, 352, PP, (4, 2, 2, 3)),
    (3392, 3520, 192, PP, (2, 4, 4, 2)), (3360, 3616, 352, PP, (2, 4, 4, 2)),
]
# float32 layers of 32 tokens whose weight-gradient group takes each tile: (heads, ffn, rows and columns of the tile)
F32_GROUPS = [(2, 96, (32, 32)), (5, 352, (64, 48)), (5, 608, (64, 64)), (6, 608, (64, 96)), (4, 3616, (64, 144)),
              (8, 1504, (64, 192))]
