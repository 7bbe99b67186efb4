"""The slab products on the bf16 matrix cores (fp32 as six bf16 products).

Small integers split and sum exactly, so O must match the oracle bit for bit.
On floats the bar is the split's own: the six products leave out at most
2^-24 of each product, and the sums are the fp32 accumulators', so O stays
within a few fp32 roundings per sum of the 64-bit result, well inside 2e-6.

The entry points give some of these shapes to other kernels; test_gpu_kernels.py calls
this one itself on all of them.
"""
import numpy as np
import pytest
import torch

import paper_1706_06873_amd as mec
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def say(*a):
    print("[case]", *a, flush=True)


def run(I, K, s_h, s_w, algo):
    O = mec.conv2d(I.to(DEV), K.to(DEV), s_h, s_w, algo=algo)
    torch.cuda.synchronize()
    return O.cpu().numpy()


# i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w; rows = i_n*o_h*o_w
CASES = [
    (1, 66, 66, 32, 3, 3, 128, 1, 1),    # whole rows, whole channels, an odd number of chunks
    (5, 30, 31, 32, 3, 3, 65, 1, 1),     # one channel past a tile; rows past whole tiles
    (2, 61, 60, 11, 3, 3, 63, 1, 1),     # runs of 33, one short of a channel tile
    (3, 64, 65, 11, 1, 3, 200, 1, 1),    # one run: two chunks, the second one element
    (9, 40, 40, 5, 2, 3, 40, 2, 1),      # runs of 15: a group of 8 spans two runs
    (9, 40, 40, 2, 11, 3, 40, 2, 1),     # runs of 6: a group may span three
    (2, 300, 33, 4, 5, 3, 96, 3, 2),     # strides apart, tall image
    (40, 9, 9, 64, 3, 3, 256, 1, 1),     # a tile touches several images
    (130, 5, 4, 33, 5, 4, 64, 1, 1),     # one output pixel per image
    (16, 58, 58, 64, 3, 3, 256, 1, 1),   # the largest tile
]


@pytest.mark.parametrize("dims", CASES)
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_tile_products(orc, dims, algo):
    say("tile", dims, algo)
    s_h, s_w = dims[7], dims[8]
    I, K = wl.random_case(31, *dims, dist="int")
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), s_h, s_w)
    assert np.array_equal(run(I, K, s_h, s_w, algo), ref.astype(np.float32))
    I, K = wl.random_case(32, *dims)
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), s_h, s_w).astype(np.float64)
    got = run(I, K, s_h, s_w, algo).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# tall kernels over 3 channels, which both read I: channel counts at the rule's
# edges, a batch of less than a tile and one of many
@pytest.mark.parametrize("k_c", [32, 33, 64, 65, 96, 97, 128, 129])
@pytest.mark.parametrize("size", [(2, 31, 33, 3, 11, 11), (5, 90, 91, 3, 9, 9)])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_tall_products_from_the_input(orc, size, k_c, algo):
    dims = size + (k_c, 4, 4)
    say("tall", dims, algo)
    I, K = wl.random_case(35, *dims, dist="int")
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 4, 4)
    assert np.array_equal(run(I, K, 4, 4, algo), ref.astype(np.float32))
    I, K = wl.random_case(36, *dims)
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 4, 4).astype(np.float64)
    got = run(I, K, 4, 4, algo).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_tile_unaligned_and_guarded(orc, shift):
    dims = (4, 40, 41, 32, 3, 3, 66, 1, 1)
    say("tile unaligned", shift)
    I, K = wl.random_case(33, *dims, dist="int")
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 1, 1).astype(np.float32)

    def off(t, n):
        buf = torch.full((t.numel() + 8,), 7.0, device=DEV)
        buf[n:n + t.numel()] = t.reshape(-1).to(DEV)
        return buf, buf[n:n + t.numel()].view(t.shape)

    _, Id = off(I, shift)
    _, Kd = off(K, shift)
    obuf, Od = off(torch.zeros(ref.shape), shift)
    mec.conv2d(Id, Kd, 1, 1, algo="fused", O=Od)
    torch.cuda.synchronize()
    assert np.array_equal(Od.cpu().numpy(), ref)
    guard = obuf.cpu().numpy()
    assert (guard[:shift] == 7).all() and (guard[shift + ref.size:] == 7).all()


@pytest.mark.parametrize("algo", ["lowered", "fused"])
@pytest.mark.parametrize("what", ["inf", "nan", "inf weight", "overflow", "tiny", "huge", "subnormal"])
def test_tile_values_the_split_does_not_hold(orc, what, algo):
    """Infinities, NaNs, sums past fp32's range and values whose last bits a
    bf16 part cannot hold come out as the plain fp32 products give them."""
    dims = (3, 40, 40, 20, 3, 3, 70, 1, 1)
    say("tile values", what, algo)
    I, K = wl.random_case(34, *dims)
    I = I.abs()
    tol = 2e-6
    if what == "inf":
        I[1, 7, 9, 3] = float("inf")
    elif what == "nan":
        I[2, 39, 39, 19] = float("nan")
    elif what == "inf weight":
        K[1, 2, 5, 69] = -float("inf")
    elif what == "overflow":
        K = K.abs() * 1e38
    elif what == "tiny":
        I = I * 1e-35
    elif what == "huge":
        I, K = I * 1.5e38, K * 1e-37
    elif what == "subnormal":
        I, K = I * 1e-39, K * 1e6
        tol = 1e-4  # the inputs themselves hold about 17 bits: their sums are exact to that or better
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 1, 1).astype(np.float64)
    with np.errstate(over="ignore"):
        ref32 = ref.astype(np.float32)
    got = run(I, K, 1, 1, algo)
    fine = np.isfinite(ref32)
    assert np.array_equal(np.isnan(got), np.isnan(ref32))
    assert np.array_equal(got[~fine & ~np.isnan(ref32)], ref32[~fine & ~np.isnan(ref32)])
    if what == "overflow":
        assert not fine.all()
    ref, got = ref[fine], got[fine].astype(np.float64)
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


# operands below 2^-133, where no bf16 part holds anything, against ordinary ones:
# their products are ordinary fp32 numbers
@pytest.mark.parametrize("which", ["input", "kernel"])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_tile_values_below_every_part(orc, which, algo):
    dims = (3, 40, 40, 20, 3, 3, 70, 1, 1)
    say("tile values below every part", which, algo)
    I, K = wl.random_case(37, *dims)
    I, K = (I * 4e-41, K * 1e6) if which == "input" else (I * 1e6, K * 4e-41)
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 1, 1).astype(np.float64)
    assert np.abs(ref).max() > 1e-36
    got = run(I, K, 1, 1, algo).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


def test_tile_plain_products_of_the_largest_tile(orc):
    """Values below 2^-110 throughout: every block of every wave is computed again,
    runs of whole chunks, tiles of 256 x 128."""
    dims = (16, 58, 58, 64, 3, 3, 256, 1, 1)
    say("tile plain products", dims)
    I, K = wl.random_case(38, *dims)
    I = I * 1e-35
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 1, 1).astype(np.float64)
    got = run(I, K, 1, 1, "fused").astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# small values that the parts hold whole: bf16 subnormals, and values whose middle part
# is one
@pytest.mark.parametrize("what", ["subnormal", "subnormal middle part"])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_tile_small_values_held(orc, what, algo):
    dims = (3, 40, 40, 20, 3, 3, 70, 1, 1)
    say("tile small values", what, algo)
    I, K = wl.random_case(39, *dims)
    if what == "subnormal":
        I = torch.round(I * 127) * 2.0 ** -133
    else:
        I = (1 + torch.round(I.abs() * 8191) / 8192) * 2.0 ** -120
    K = K * 2.0 ** 40
    ref = orc.conv2d_direct(I.numpy(), K.numpy(), 1, 1).astype(np.float64)
    got = run(I, K, 1, 1, algo).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# Every value the same x. The parts' own products and their sums are exact here (288
# terms of at most 15 bits), so what differs from the 64-bit result is what the six
# products leave out, below 2^-24 of it, and the rounding of the stored value, 2^-24.
# x: its last 16 bits set, and the largest middle and last parts there are.
@pytest.mark.parametrize("bits", [0x3f80ffff, 0x3f807f40, 0x3f808040])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_tile_products_left_out(bits, algo):
    dims = (5, 30, 31, 32, 3, 3, 65, 1, 1)
    say("tile left out", hex(bits), algo)
    x = np.array([bits], np.uint32).view(np.float32)[0]
    I, K = torch.full(dims[:4], float(x)), torch.full((3, 3, 32, 65), float(x))
    got = run(I, K, 1, 1, algo).astype(np.float64)
    ref = 288 * float(x) ** 2
    assert np.abs(got - ref).max() <= 2.0 ** -23 * ref
