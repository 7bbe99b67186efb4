"""Kernels called past the choice that the entry points make: the fixed and generic slab
kernels and the fp32 gradient kernels on the shapes that the parity tests list for them,
most of which the entry points give to other kernels now. Bit for bit on small integers."""
import numpy as np
import pytest
import torch

import kernels
import paper_1706_06873_amd as mec
import test_gpu_grad as grad
import test_gpu_parity as parity
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

ROW_TILES = [(8, 66, 66, 16, 3, 3, 192, 1, 1), (8, 58, 58, 16, 3, 3, 256, 1, 1)]  # 4 and 14 rows
F32 = list(dict.fromkeys(parity.SWEEP + ROW_TILES + parity.STREAM_CASES + parity.SPLIT_CASES + parity.DMA_CASES_F32 +
                         parity.K7S2_CASES + parity.K5S1_CASES + parity.K3S2_CASES + parity.FLAT_CASES))
BF16 = list(dict.fromkeys(parity.SWEEP_BF16 + parity.FLAT_CASES_BF16 + parity.DMA_CASES_BF16 + parity.SPLIT_CASES_BF16))


def check(orc, dims, dtype):
    s_h, s_w = dims[7], dims[8]
    I, K = wl.random_case(17 + sum(dims), *dims, dtype=dtype, dist="int")
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), s_h, s_w).astype(np.float32)
    assert np.abs(ref).max() < 2 ** 24
    Id, Kd = I.to(DEV), K.to(DEV)
    L = mec.lower(Id, dims[4], dims[5], dims[6], s_h, s_w)
    for A, fused in ((L, False), (Id, True)):
        print("[case] fixed", dtype, dims, "fused" if fused else "lowered", flush=True)
        O = kernels.gemm(kernels.FIXED, A, Kd, dims, fused)
        torch.cuda.synchronize()
        assert O is not None and np.array_equal(O.cpu().numpy(), ref), fused


@pytest.mark.parametrize("dims", F32)
def test_fixed_products_f32(orc, dims):
    check(orc, dims, "f32")


@pytest.mark.parametrize("dims", BF16)
def test_fixed_products_bf16(orc, dims):
    check(orc, dims, "bf16")


@pytest.mark.parametrize("dims", grad.SHAPES)
def test_fp32_gradient_kernels(orc, dims):
    print("[case] fp32 gradient kernels", dims, flush=True)
    I, K, G = grad.problem(19 + sum(dims), dims, "int")
    k_h, k_w, s_h, s_w = dims[4], dims[5], dims[7], dims[8]
    Id, Gd = I.to(DEV), G.to(DEV)
    L = mec.lower(Id, k_h, k_w, dims[6], s_h, s_w)
    ref = orc.conv2d_wgrad(I.numpy(), G.numpy(), k_h, k_w, s_h, s_w).astype(np.float32)
    ran = 0
    for kernel in (kernels.WGRAD_SLAB, kernels.WGRAD_GENERAL):
        for A, fused in ((L, False), (Id, True)):
            dK = kernels.wgrad(kernel, A, Gd, dims, fused)
            torch.cuda.synchronize()
            if dK is not None:
                assert np.array_equal(dK.cpu().numpy(), ref), (kernel, fused)
                ran += 1
    assert ran == 2  # the shape's own kernel, from L and from I
    dL = kernels.dgrad_gemm(False, Gd, K.to(DEV), dims)
    torch.cuda.synchronize()
    ref = orc.mec_dgrad_lowered(G.numpy(), K.numpy(), dims[1], dims[2], s_h, s_w).astype(np.float32)
    assert np.array_equal(dL.cpu().numpy(), ref)
