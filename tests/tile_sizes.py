"""Sizes (M, K, N) of the tiled GEMMs' tests, and the tile shape and split that
each takes on 256 compute units with a workspace of the queried size
(csrc/gemm_plan.h): "whole" tiles, all "split" along K, or whole tiles with a
split "tail".  test_tile_choice.py holds the choice to them, so that every kernel
instance stays covered by the GPU tests that run on these lists."""

# 8-bit activations: (128-wide weight groups, one step per channel)
EIGHT = {
    (129, 256, 64): ("64x64 whole", "64x64 whole"),
    (131, 1536, 64): ("64x64 split", "64x64 split"),
    (257, 3072, 6592): ("64x64 tail", "64x64 tail"),
    (513, 256, 7296): ("64x128 whole", "64x128 whole"),
    (129, 5120, 4160): ("64x128 split", "64x64 whole"),
    (129, 5120, 5568): ("64x128 split", "64x128 split"),
    (131, 5120, 5760): ("64x128 split", "64x128 split"),
    (385, 5120, 5568): ("64x128 tail", "64x128 whole"),
    (1537, 1536, 8128): ("256x128 whole", "256x128 whole"),
    (2100, 1536, 5952): ("256x128 whole", "256x128 whole"),
    (1001, 256, 6208): ("128x128 whole", "128x128 whole"),
    (1001, 2048, 8320): ("128x128 tail", "128x128 tail"),
    (385, 5120, 5376): ("128x128 split", "64x128 whole"),
    (206, 5120, 2944): ("64x64 split", "128x128 split"),
    (2731, 3072, 6016): ("128x128 tail", "256x128 tail"),
    (2948, 3456, 5568): ("256x128 tail", "256x128 tail"),
}

# 4-bit activations on the fp8 matrix cores
FOUR = {
    (129, 128, 64): "64x64 whole",
    (131, 1536, 64): "64x64 split",
    (129, 5120, 4160): "64x128 split",
    (513, 256, 5568): "64x128 whole",
    (193, 3072, 8256): "128x128 split",
    (1537, 256, 4160): "128x128 whole",
    (1001, 2048, 8256): "128x128 tail",
    (513, 5120, 4160): "128x128 split",
    (1000, 256, 4224): "64x64 whole",  # more tiles than workgroups
}

# the GELU epilogue (N a multiple of 128: it is the next layer's K)
GELU_EIGHT = {
    (129, 256, 128): ("64x64 whole", "64x64 whole"),
    (131, 1536, 128): ("64x64 split", "64x64 split"),
    (513, 256, 7296): ("64x128 whole", "64x128 whole"),
    (129, 5120, 5632): ("64x128 split", "64x128 split"),
    (1537, 1536, 8192): ("256x128 whole", "256x128 whole"),
    (1001, 2048, 8320): ("128x128 tail", "128x128 tail"),
    (2731, 3072, 6016): ("128x128 tail", "256x128 tail"),
    (3047, 1536, 8320): ("256x128 tail", "256x128 tail"),
}
GELU_FOUR = {
    (131, 1536, 128): "64x64 split",
    (513, 256, 5632): "64x128 whole",
    (129, 5120, 5632): "128x128 split",
    (129, 5120, 4224): "64x128 split",
    (1537, 256, 4224): "128x128 whole",
    (193, 3072, 8320): "128x128 split",
    (1001, 2048, 8320): "128x128 tail",
    (1000, 256, 4224): "64x64 whole",
}

# the calibration's error epilogue
ERR_EIGHT = {
    (129, 256, 64): ("64x64 whole", "64x64 whole"),
    (200, 1024, 192): ("64x64 whole", "64x64 whole"),
    (257, 512, 128): ("64x64 whole", "64x64 whole"),
    (1000, 256, 4160): ("64x128 whole", "64x128 whole"),
    (1001, 256, 6208): ("128x128 whole", "128x128 whole"),
    (131, 1536, 64): ("64x64 split", "64x64 split"),
    (257, 3072, 6592): ("64x64 tail", "64x64 tail"),
    (129, 5120, 5568): ("64x128 split", "64x128 split"),
    (385, 5120, 5568): ("64x128 tail", "64x128 whole"),
    (385, 5120, 5376): ("128x128 split", "64x128 whole"),
    (206, 5120, 2944): ("64x64 split", "128x128 split"),
    (1001, 2048, 8320): ("128x128 tail", "128x128 tail"),
    (1537, 1536, 8128): ("256x128 whole", "256x128 whole"),
    (2731, 3072, 6016): ("128x128 tail", "256x128 tail"),
    (2948, 3456, 5568): ("256x128 tail", "256x128 tail"),
}
ERR_FOUR = {
    (129, 256, 64): "64x64 whole",
    (200, 1024, 192): "64x64 split",
    (257, 512, 128): "64x64 whole",
    (1000, 256, 4160): "64x64 whole",
    (513, 256, 5568): "64x128 whole",
    (129, 5120, 4160): "64x128 split",
    (193, 3072, 8256): "128x128 split",
    (1537, 256, 4160): "128x128 whole",
    (1001, 2048, 8256): "128x128 tail",
}
