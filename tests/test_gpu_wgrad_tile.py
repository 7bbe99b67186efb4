"""The weight gradient's products on the bf16 matrix cores (fp32 as six bf16
products): exact on small integers; on floats within the fp32 sums' own error."""
import numpy as np
import pytest
import torch

import paper_1706_06873_amd as mec
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w; rows of dK k_h*k_w*i_c in tiles of
# 128, columns k_c in tiles of 64, pixels in chunks of 32
CASES = [
    (1, 10, 10, 16, 2, 4, 64, 1, 1),     # one row tile, two chunks, the last 31 pixels short
    (2, 9, 8, 43, 1, 3, 65, 1, 1),       # 129 rows, one column past a tile
    (3, 20, 19, 5, 3, 3, 63, 2, 1),      # runs of 15: groups of 8 span two runs
    (5, 12, 13, 9, 5, 1, 70, 1, 2),      # runs of 9
    (1, 5, 5, 64, 5, 5, 40, 1, 1),       # one pixel
    (7, 30, 31, 48, 3, 3, 96, 1, 1),     # many shares
    (40, 8, 8, 256, 3, 3, 130, 1, 1),    # many tiles, pixels of several images a chunk
]


def inputs(dims, dist, seed):
    I, K = wl.random_case(seed, *dims, dist=dist)
    o_h, o_w = mec.output_dims(dims[1], dims[2], dims[4], dims[5], dims[7], dims[8])
    g = torch.Generator().manual_seed(seed)
    shape = (dims[0], o_h, o_w, dims[6])
    G = torch.randint(-3, 4, shape, generator=g).float() if dist == "int" else torch.rand(shape, generator=g) - 0.5
    return I, G


def both(I, G, dims):
    k_h, k_w, k_c, s_h, s_w = dims[4:]
    Id, Gd = I.to(DEV), G.to(DEV)
    dK = mec.conv2d_wgrad(Id, Gd, k_h, k_w, s_h, s_w)
    L = mec.lower(Id, k_h, k_w, k_c, s_h, s_w)
    dK2 = mec.wgrad_gemm(L, Gd, k_h, dims[2], s_h, s_w)
    torch.cuda.synchronize()
    dK, dK2 = dK.cpu().numpy(), dK2.cpu().numpy()
    assert np.array_equal(dK, dK2, equal_nan=True)
    return dK


@pytest.mark.parametrize("dims", CASES)
def test_wgrad_tile(orc, dims):
    print("[case] wgrad tile", dims, flush=True)
    for dist, tol in (("int", 0.0), ("u11", 2e-6)):
        I, G = inputs(dims, dist, 51)
        ref = orc.conv2d_wgrad(I.numpy(), G.numpy(), dims[4], dims[5], dims[7], dims[8]).astype(np.float64)
        got = both(I, G, dims).astype(np.float64)
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("what", ["inf", "nan", "overflow", "tiny", "huge"])
def test_wgrad_values_the_split_does_not_hold(orc, what):
    dims = (3, 14, 13, 20, 3, 3, 70, 1, 1)
    print("[case] wgrad values", what, flush=True)
    I, G = inputs(dims, "u11", 52)
    G = G + 0.75
    I = I.abs()
    if what == "inf":
        I[1, 7, 9, 3] = float("inf")
    elif what == "nan":
        G[2, 11, 10, 69] = float("nan")
    elif what == "overflow":
        G = G * 2e38
    elif what == "tiny":
        G = G * 1e-36
    elif what == "huge":
        G, I = G * 1e38, I * 1e-37
    ref = orc.conv2d_wgrad(I.numpy(), G.numpy(), 3, 3, 1, 1).astype(np.float64)
    with np.errstate(over="ignore"):
        ref32 = ref.astype(np.float32)
    got = both(I, G, dims)
    fine = np.isfinite(ref32)
    assert np.array_equal(np.isnan(got), np.isnan(ref32))
    assert np.array_equal(got[~fine & ~np.isnan(ref32)], ref32[~fine & ~np.isnan(ref32)])
    ref, got = ref[fine], got[fine].astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# operands below 2^-133, where no bf16 part holds anything, against ordinary ones
@pytest.mark.parametrize("which", ["input", "gradient"])
def test_wgrad_values_below_every_part(orc, which):
    dims = (3, 14, 13, 20, 3, 3, 70, 1, 1)
    print("[case] wgrad values below every part", which, flush=True)
    I, G = inputs(dims, "u11", 53)
    I, G = (I * 4e-41, G * 1e6) if which == "input" else (I * 1e6, G * 4e-41)
    ref = orc.conv2d_wgrad(I.numpy(), G.numpy(), 3, 3, 1, 1).astype(np.float64)
    assert np.abs(ref).max() > 1e-36
    got = both(I, G, dims).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# Every value the same x, 63 terms: as in test_gpu_tile.py's test_tile_products_left_out,
# and the shares' own sum is rounded once more
@pytest.mark.parametrize("bits", [0x3f80ffff, 0x3f807f40, 0x3f808040])
def test_wgrad_products_left_out(bits):
    dims = (1, 10, 10, 16, 2, 4, 64, 1, 1)
    print("[case] wgrad left out", hex(bits), flush=True)
    x = float(np.array([bits], np.uint32).view(np.float32)[0])
    got = both(torch.full(dims[:4], x), torch.full((1, 9, 7, 64), x), dims).astype(np.float64)
    ref = 63 * x ** 2
    assert np.abs(got - ref).max() <= 3 * 2.0 ** -24 * ref


def test_wgrad_tile_of_a_large_l():
    """L of more than 2 GiB, I of less: both ways take this kernel, and dK is the same
    bit for bit; one image's L stays below the limit."""
    dims = (20, 200, 200, 256, 3, 3, 16, 1, 1)
    print("[case] wgrad large L", dims, flush=True)
    g = torch.Generator(device=DEV).manual_seed(54)
    I = torch.rand(dims[:4], generator=g, device=DEV) - 0.5
    G = torch.rand((20, 198, 198, 16), generator=g, device=DEV) - 0.5
    dK = mec.conv2d_wgrad(I, G, 3, 3, 1, 1)
    L = mec.lower(I, 3, 3, 16, 1, 1)
    assert L.numel() * 4 > 2 ** 31 > I.numel() * 4
    dK2 = mec.wgrad_gemm(L, G, 3, dims[2], 1, 1)
    del L
    assert torch.equal(dK, dK2)
    for a, b in ((0, 0), (2, 1)):
        ref = I[:, a:a + 198, b:b + 198].reshape(-1, 256).double().t().contiguous() @ G.reshape(-1, 16).double()
        assert (dK[a, b].double() - ref).norm() <= 2e-6 * ref.norm()
