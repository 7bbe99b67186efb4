"""The bf16 products over at most 4 input channels: bit for bit on integers.

The entry points give some of these shapes to other kernels; test_gpu_kernels.py calls
this one itself on all of them."""
import numpy as np
import pytest
import torch

import paper_1706_06873_amd as mec
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w
CASES = [
    (1, 30, 33, 3, 3, 3, 64, 1, 1),     # odd kernel rows, images of an even number of bytes not whole words
    (3, 17, 19, 3, 7, 7, 61, 2, 2),     # a tile touches two images, ragged channels
    (5, 9, 8, 1, 5, 4, 97, 1, 2),       # one channel, even kernel rows, two channel tiles
    (2, 40, 21, 2, 2, 1, 33, 2, 1),     # two channels, one tap a row: half of each pair is padding
    (7, 3, 260, 4, 3, 3, 40, 3, 2),     # one output row per image, several column ranges
    (66, 57, 57, 3, 11, 11, 96, 4, 4),  # K of 101 KB
    (300, 20, 20, 3, 5, 5, 32, 2, 2),   # many tiles, K of 20 KB
]


@pytest.mark.parametrize("dims", CASES)
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_first_products(orc, dims, algo):
    print("[case] first", dims, algo, flush=True)
    s_h, s_w = dims[7], dims[8]
    for dist, tol in (("int", 0.0), ("u11", 2e-6)):
        I, K = wl.random_case(71, *dims, dtype="bf16", dist=dist)
        ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), s_h, s_w).astype(np.float64)
        n = 64
        buf = torch.full((ref.size + 2 * n,), 7.0, device=DEV)
        O = buf[n:n + ref.size].view(ref.shape)
        mec.conv2d(I.to(DEV), K.to(DEV), s_h, s_w, algo=algo, O=O)
        torch.cuda.synchronize()
        guard = buf.cpu().numpy()
        assert (guard[:n] == 7).all() and (guard[-n:] == 7).all()
        assert np.linalg.norm(O.cpu().numpy().astype(np.float64) - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_first_unaligned(orc, shift):
    dims = (3, 17, 19, 3, 3, 3, 61, 1, 1)
    print("[case] first unaligned", shift, flush=True)
    I, K = wl.random_case(72, *dims, dtype="bf16", dist="int")
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), 1, 1).astype(np.float32)

    def off(t):
        buf = torch.zeros(t.numel() + 8, dtype=t.dtype, device=DEV)
        buf[shift:shift + t.numel()] = t.reshape(-1).to(DEV)
        return buf[shift:shift + t.numel()].view(t.shape)

    O = mec.conv2d(off(I), off(K), 1, 1, algo="fused")
    torch.cuda.synchronize()
    assert np.array_equal(O.cpu().numpy(), ref)


def test_first_non_finite(orc):
    """Infinities reach the outputs whose windows hold them, and no other."""
    dims = (2, 20, 21, 3, 3, 3, 62, 1, 1)
    I, K = wl.random_case(73, *dims, dtype="bf16")
    I[:, 9, 10, 1] = float("inf")
    I[1, 19, 20, 2] = float("nan")
    K[0, 0, 0, 61] = float("inf")
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), 1, 1)
    got = mec.conv2d(I.to(DEV), K.to(DEV), 1, 1, algo="fused").cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))


# an odd number of steps of two pairs of taps (3x3: 3, 11x11: 33), whose last step
# stands alone, and an even one (5x5: 8, the last half empty)
@pytest.mark.parametrize("dims", [(2, 20, 21, 3, 3, 3, 62, 1, 1), (12000, 11, 15, 3, 11, 11, 96, 4, 4),
                                  (3, 17, 19, 3, 5, 5, 61, 2, 2)])
@pytest.mark.parametrize("algo", ["lowered", "fused"])
def test_first_infinite_weight_in_the_last_tap(orc, dims, algo):
    print("[case] first infinite weight", dims, algo, flush=True)
    I, K = wl.random_case(74, *dims, dtype="bf16")
    I = (I.abs() + 0.25).to(I.dtype)  # no zero meets the infinities
    K[-1, -1, -1, 0] = float("inf")
    K[-1, -1, 0, dims[6] - 1] = -float("inf")
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), dims[7], dims[8])
    assert np.isinf(ref).any() and not np.isnan(ref).any()
    got = mec.conv2d(I.to(DEV), K.to(DEV), dims[7], dims[8], algo=algo).cpu().numpy()
    assert not np.isnan(got).any()
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
