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


def test_unaligned_routes():
    dims = (32, 224, 224, 64, 7, 7, 64, 2, 2)
    assert k.route(dims, "bf16", "fused", I=k.ALIGNED + 2)[0] == k.FIXED
    assert k.route((32, 227, 227, 3, 11, 11, 96, 4, 4), "bf16", "fused", I=k.ALIGNED + 2)[0] != k.FIRST


# (L of more than 2 GiB: from L and from I alike; one image's L of more: neither)
@pytest.mark.parametrize("dims,want", [
    ((32, 58, 58, 64, 3, 3, 64, 1, 1), k.WGRAD_TILE),
    ((20, 200, 200, 256, 3, 3, 16, 1, 1), k.WGRAD_TILE),
    ((1, 900, 900, 256, 3, 3, 16, 1, 1), k.WGRAD_GENERAL),
    ((8, 40, 40, 2, 3, 3, 16, 1, 1), k.WGRAD_GENERAL),
])
def test_wgrad_routes(dims, want):
    assert k.wgrad_route(dims) == want
