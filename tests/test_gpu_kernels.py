"""Kernels called past the choice that the entry points make, on the shapes that the
tests list for them, of which the entry points give many to other kernels. Bit for bit
on small integers, within 2e-6 on floats, nothing written beside O."""
import numpy as np
import pytest
import torch

import kernels
import paper_1706_06873_amd as mec
import test_gpu_first as first
import test_gpu_grad as grad
import test_gpu_parity as parity
import test_gpu_patch as patch
import test_gpu_small as small
import test_gpu_tile as tile
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


# each on its own shapes, from L and from I where it reads both; the first-layer kernel's
# workgroups take several tiles on the last two (of 64 and of 96 channels)
OWN = ([(kernels.TILE, d, "f32") for d in tile.CASES] +
       [(kernels.SMALL, d, t) for d in small.CASES for t in ("f32", "bf16")] +
       [(kernels.PATCH, d, "bf16") for d in patch.CASES] +
       [(kernels.FIRST, d, "bf16") for d in first.CASES + [(2300, 20, 20, 3, 5, 5, 32, 2, 2),
                                                           (12000, 11, 15, 3, 11, 11, 96, 4, 4)]])


@pytest.mark.parametrize("kernel,dims,dtype", OWN)
def test_kernel_on_its_own_shapes(orc, kernel, dims, dtype):
    k_h, s_h, s_w = dims[4], dims[7], dims[8]
    runs = 0
    for dist, tol in (("int", 0.0), ("u11", 2e-6)):
        I, K = wl.random_case(23, *dims, dtype=dtype, dist=dist)
        ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), s_h, s_w).astype(np.float64)
        Id, Kd = I.to(DEV), K.to(DEV)
        for fused in (False, True):
            if not fused and kernel in (kernels.PATCH, kernels.FIRST):
                continue
            print("[case] own", kernel, dims, dtype, dist, "fused" if fused else "lowered", flush=True)
            A = Id if fused else mec.lower(Id, k_h, dims[5], dims[6], s_h, s_w)
            buf = torch.full((ref.size + 128,), 7.0, device=DEV)
            O = kernels.gemm(kernel, A, Kd, dims, fused, buf[64:64 + ref.size].view(ref.shape))
            torch.cuda.synchronize()
            if O is None:  # the tile kernel reads runs of at least 8 from I
                assert kernel == kernels.TILE and fused and dims[5] * dims[3] < 8
                continue
            runs += 1
            guard = buf.cpu().numpy()
            assert (guard[:64] == 7).all() and (guard[-64:] == 7).all()
            assert np.linalg.norm(O.cpu().numpy().astype(np.float64) - ref) <= tol * np.linalg.norm(ref)
    assert runs >= 2


# the lowered calls whose products read I leave the whole of L in the workspace all the same
@pytest.mark.parametrize("dims,dtype,want", [
    ((1, 30, 33, 3, 3, 3, 64, 1, 1), "bf16", kernels.FIRST),
    ((1, 40, 41, 34, 3, 3, 64, 1, 1), "bf16", kernels.PATCH),
    ((5, 90, 91, 3, 9, 9, 96, 4, 4), "f32", kernels.TILE),
])
def test_l_is_left_where_the_products_read_the_input(orc, dims, dtype, want):
    print("[case] L left", dims, dtype, flush=True)
    assert kernels.route(dims, dtype, "lowered") == (want, True)
    k_h, k_w, k_c, s_h, s_w = dims[4:]
    I, K = wl.random_case(29, *dims, dtype=dtype, dist="int")
    refL = orc.mec_lower(wl.to_oracle_array(I), k_h, k_w, k_c, s_h, s_w)
    L = torch.full(refL.shape, 9.0, device=DEV, dtype=I.dtype)
    O = mec.conv2d(I.to(DEV), K.to(DEV), s_h, s_w, workspace=L)
    torch.cuda.synchronize()
    assert np.array_equal(wl.to_oracle_array(L.cpu()), refL)
    ref = orc.conv2d_direct(wl.to_oracle_array(I), wl.to_oracle_array(K), s_h, s_w)
    assert np.array_equal(O.cpu().numpy(), ref.astype(np.float32))
