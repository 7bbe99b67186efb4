"""The slab products of few outputs, whose reduction a workgroup's waves share.

Small integers sum exactly in any order, so O must match the oracle bit for bit;
on floats the products are exact or rounded to 32 bits and the sums are 32-bit
sums of at most a few thousand terms, well inside 2e-6 of the 64-bit result.
"""
import numpy as np
import pytest
import torch

import paper_1706_06873_amd as mec
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w
CASES = [
    (1, 1, 1, 64, 1, 1, 1, 1, 1),        # one output: two bf16 steps, two waves
    (1, 4, 4, 128, 1, 1, 16, 1, 1),      # one whole tile
    (1, 1, 17, 70, 1, 1, 17, 1, 1),      # one row and one channel past a tile, part of a step
    (3, 7, 7, 482, 1, 1, 76, 1, 1),      # runs that are no whole groups of 8
    (4, 7, 7, 130, 7, 7, 27, 2, 2),      # one pixel per image, a long reduction
    (2, 9, 8, 33, 3, 3, 40, 2, 1),       # odd channels: bf16 windows at odd elements
    (2, 9, 8, 24, 3, 3, 40, 1, 2),       # a group of 8 ends where a run ends
    (1, 14, 14, 256, 3, 3, 48, 1, 1),    # 16 waves, several rounds each
    (2, 12, 11, 7, 9, 5, 33, 3, 4),      # tall kernel, strides apart
]


@pytest.mark.parametrize("dims", CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("algo", ["lowered", "fused", "im2col"])
def test_small_products(orc, dims, dtype, algo):
    print("[case] small", dims, dtype, algo, flush=True)
    s_h, s_w = dims[7], dims[8]
    for dist in ("int", None):
        I, K = wl.random_case(51, *dims, dtype=dtype, **({"dist": dist} if dist else {}))
        ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), s_h, s_w)
        O = mec.conv2d(I.to(DEV), K.to(DEV), s_h, s_w, algo=algo)
        torch.cuda.synchronize()
        got = O.cpu().numpy()
        if dist:
            assert np.array_equal(got, ref.astype(np.float32))
        else:
            ref = ref.astype(np.float64)
            assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [1, 3])
def test_small_unaligned_and_guarded(orc, dtype, shift):
    """Operands at odd elements; nothing is written beside O, and values outside
    the operands, infinities here, reach no output."""
    dims = (2, 9, 9, 24, 3, 3, 21, 1, 1)
    print("[case] small unaligned", dtype, shift, flush=True)
    I, K = wl.random_case(52, *dims, dist="int", dtype=dtype)
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), 1, 1).astype(np.float32)

    def off(t, fill):
        buf = torch.full((t.numel() + 16,), fill, device=DEV, dtype=t.dtype)
        buf[shift:shift + t.numel()] = t.reshape(-1).to(DEV)
        return buf, buf[shift:shift + t.numel()].view(t.shape)

    _, Id = off(I, float("inf"))
    _, Kd = off(K, float("inf"))
    obuf, Od = off(torch.zeros(ref.shape), 7.0)
    mec.conv2d(Id, Kd, 1, 1, algo="fused", O=Od)
    torch.cuda.synchronize()
    assert np.array_equal(Od.cpu().numpy(), ref)
    guard = obuf.cpu().numpy()
    assert (guard[:shift] == 7).all() and (guard[shift + ref.size:] == 7).all()
