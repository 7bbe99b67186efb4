"""Which kernel a call takes: host arithmetic only, nothing is launched."""
import pytest

import kernels as k
from paper_1706_06873_amd import workloads as wl


# the layers and the edges of the rules whose figures stand in the sources
@pytest.mark.parametrize("dims,dtype,algo,want", [
    (wl.LAYERS["tiny"].dims, "f32", "lowered", (k.FIXED, False)),
    (wl.LAYERS["resnet_mid"].dims, "f32", "fused", (k.TILE, True)),
    (wl.LAYERS["vgg_first"].dims, "f32", "fused", (k.FIXED, True)),
    (wl.LAYERS["alexnet_conv1"].dims, "f32", "lowered", (k.TILE, True)),
    (wl.LAYERS["deep_bf16"].dims, "bf16", "lowered", (k.FIXED, False)),
    ((32, 227, 227, 3, 11, 11, 96, 4, 4), "bf16", "lowered", (k.FIRST, True)),
    ((1, 227, 227, 3, 11, 11, 96, 4, 4), "bf16", "lowered", (k.FIXED, False)),
    ((32, 224, 224, 64, 7, 7, 64, 2, 2), "bf16", "lowered", (k.PATCH, True)),
    ((1, 14, 14, 256, 3, 3, 256, 1, 1), "f32", "lowered", (k.SMALL, False)),
    ((128, 227, 227, 3, 11, 11, 32, 4, 4), "f32", "lowered", (k.FIXED, False)),
    ((32, 227, 227, 3, 11, 11, 96, 4, 4), "f32", "lowered", (k.FIXED, False)),
])
def test_product_routes(dims, dtype, algo, want):
    assert k.route(dims, dtype, algo) == want


# fp32 shapes that the fixed kernels' 2-row tiles do faster, and their neighbours
@pytest.mark.parametrize("dims,algo,want", [
    ((8, 67, 67, 288, 7, 7, 32, 2, 2), "fused", k.FIXED),     # 128 tiles, split in two
    ((9, 67, 67, 288, 7, 7, 32, 2, 2), "fused", k.TILE),      # 144
    ((1, 32, 32, 320, 5, 5, 528, 1, 1), "lowered", k.FIXED),  # 126 tiles
    ((109, 7, 7, 420, 3, 3, 84, 1, 1), "fused", k.FIXED),     # rows of 1260, 108 tiles
    ((109, 7, 7, 420, 3, 3, 84, 1, 1), "lowered", k.FIXED),
    ((109, 7, 7, 418, 3, 3, 84, 1, 1), "fused", k.TILE),      # rows of 1254, no vectors of 4
    ((109, 7, 7, 140, 3, 3, 84, 1, 1), "fused", k.TILE),      # reduction of 1260
    ((109, 7, 7, 420, 3, 3, 96, 1, 1), "lowered", k.FIXED),
    ((140, 7, 7, 420, 3, 3, 84, 1, 1), "fused", k.TILE),      # 132 tiles
    ((2, 40, 240, 2, 3, 200, 128, 1, 1), "lowered", k.FIXED),  # vectors of 4 in L
    ((2, 40, 240, 2, 3, 200, 128, 1, 1), "fused", k.TILE),    # but not in I
    ((1, 93, 93, 496, 5, 5, 32, 1, 1), "fused", k.FIXED),     # 5x5 half chunks, 135 tiles
    ((1, 93, 93, 496, 5, 5, 32, 1, 1), "lowered", k.TILE),
    ((1, 93, 93, 480, 5, 5, 32, 1, 1), "fused", k.TILE),      # whole chunks
    ((19, 18, 18, 368, 3, 3, 192, 1, 1), "lowered", k.FIXED),  # half chunks, 240 tiles
    ((19, 18, 18, 384, 3, 3, 192, 1, 1), "lowered", k.TILE),   # whole chunks
    ((21, 18, 18, 368, 3, 3, 192, 1, 1), "fused", k.TILE),     # half chunks, 264 tiles
    ((29, 79, 79, 80, 1, 1, 496, 1, 1), "fused", k.FIXED),     # 1x1, two and a half chunks
    ((2, 79, 79, 80, 1, 1, 496, 1, 1), "fused", k.TILE),       # 1568 tiles
    ((29, 79, 79, 96, 1, 1, 496, 1, 1), "fused", k.TILE),
    ((29, 79, 79, 112, 1, 1, 496, 1, 1), "fused", k.TILE),
])
def test_fixed_tiles_kept(dims, algo, want):
    assert k.route(dims, "f32", algo)[0] == want


# bf16 7x7 at stride 2, where the fixed tiles of few input or output channels win
@pytest.mark.parametrize("dims,want", [
    ((90, 78, 78, 16, 7, 7, 112, 2, 2), k.FIXED),
    ((24, 168, 164, 48, 7, 7, 72, 2, 2), k.FIXED),
    ((90, 78, 78, 32, 7, 7, 112, 2, 2), k.PATCH),
    ((90, 78, 78, 18, 7, 7, 112, 2, 2), k.PATCH),  # no fixed tile for it
    ((4, 224, 224, 64, 7, 7, 64, 2, 2), k.PATCH),
    ((1, 224, 224, 64, 7, 7, 64, 2, 2), k.FIXED),
])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_strided_bf16_routes(dims, algo, want):
    assert k.route(dims, "bf16", algo)[0] == want


def test_unaligned_routes():
    dims = (32, 224, 224, 64, 7, 7, 64, 2, 2)
    assert k.route(dims, "bf16", "fused", I=k.ALIGNED + 2)[0] == k.FIXED
    assert k.route((32, 227, 227, 3, 11, 11, 96, 4, 4), "bf16", "fused", I=k.ALIGNED + 2)[0] != k.FIRST
    # the fixed kernels' fast forms need 16-byte vectors
    assert k.route((19, 18, 18, 368, 3, 3, 192, 1, 1), "f32", "fused", I=k.ALIGNED + 4)[0] == k.TILE


# (L of more than 2 GiB: from L and from I alike; one image's L of more: neither)
@pytest.mark.parametrize("dims,want", [
    ((32, 58, 58, 64, 3, 3, 64, 1, 1), k.WGRAD_TILE),
    ((20, 200, 200, 256, 3, 3, 16, 1, 1), k.WGRAD_TILE),
    ((1, 900, 900, 256, 3, 3, 16, 1, 1), k.WGRAD_GENERAL),
    ((8, 40, 40, 2, 3, 3, 16, 1, 1), k.WGRAD_GENERAL),
    ((50, 92, 92, 164, 1, 1, 280, 2, 2), k.WGRAD_SLAB),        # rows of L no whole groups of 8
    ((50, 92, 92, 168, 1, 1, 280, 2, 2), k.WGRAD_TILE),
    ((21, 100, 100, 20, 3, 3, 128, 1, 1), k.WGRAD_SLAB),       # rows of 60: 180 of 256, 60 of 64
    ((21, 100, 100, 28, 3, 3, 128, 1, 1), k.WGRAD_TILE),       # rows of 84: 252 of 256, 84 of 128
    ((1, 100, 100, 20, 3, 3, 128, 1, 1), k.WGRAD_TILE),        # short
    ((21, 100, 100, 20, 5, 5, 128, 1, 1), k.WGRAD_TILE),
    ((6, 10, 7, 466, 7, 7, 160, 2, 2), k.WGRAD_GENERAL),       # 12 pixels
    ((20, 10, 7, 466, 7, 7, 160, 2, 2), k.WGRAD_TILE),         # 40
])
def test_wgrad_routes(dims, want):
    assert k.wgrad_route(dims) == want


# what bench.py calls the kernel that it times, and the peak that it holds it against
@pytest.mark.parametrize("name,algo,kernel,six", [
    ("resnet_mid", "lowered", "tile_gemm_f32_kernel", True),
    ("resnet_mid", "fused", "tile_gemm_f32_kernel", True),
    ("alexnet_conv1", "lowered", "slab_gemm_f32_*kernel", False),  # mec_gemm from L: the ring
    ("alexnet_conv1", "fused", "tile_gemm_f32_kernel", True),
    ("vgg_first", "fused", "slab_gemm_f32_*kernel", False),
    ("deep_bf16", "lowered", "slab_gemm_bf16_*kernel", False),
    ("resnet_mid", "im2col", "tile_gemm_f32_kernel", True),
])
def test_bench_names_the_kernel(name, algo, kernel, six):
    import bench
    import paper_1706_06873_amd as mec
    layer = wl.LAYERS[name]
    got, peak = bench.products_kernel(mec, layer.dims, layer.dtype, algo)
    assert got == kernel
    assert peak == (bench.PEAK_TFLOPS["bf16"] / 6 if six else bench.PEAK_TFLOPS[layer.dtype])
