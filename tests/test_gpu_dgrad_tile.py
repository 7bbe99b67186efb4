"""dL on the bf16 matrix cores (fp32 as six bf16 products): exact on small
integers; on floats within the fp32 sums' own error."""
import numpy as np
import pytest
import torch

import paper_1706_06873_amd as mec
from paper_1706_06873_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w; rows of dL i_n*o_w*i_h by classes of
# s_h in tiles of 128, columns k_w*i_c in tiles of 64, chunks of 32 of k_c per tap
CASES = [
    (1, 64, 10, 8, 3, 3, 16, 1, 1),      # whole tiles, half a chunk of channels
    (2, 33, 18, 22, 5, 3, 33, 1, 2),     # one channel past a chunk, one column tile and two columns
    (3, 30, 20, 13, 3, 5, 47, 2, 1),     # two classes, channels not a multiple of 8
    (2, 41, 17, 32, 2, 2, 40, 3, 3),     # s_h > k_h: a class that no tap reaches
    (5, 40, 9, 16, 11, 4, 64, 4, 2),     # four classes, two or three taps
    (40, 7, 9, 40, 7, 3, 24, 1, 1),      # one output row: every row of dL meets one tap
    (3, 70, 12, 24, 3, 3, 96, 8, 3),     # eight classes, five of them without taps
]


def inputs(dims, dist, seed):
    I, K = wl.random_case(seed, *dims, dist=dist)
    o_h, o_w = mec.output_dims(dims[1], dims[2], dims[4], dims[5], dims[7], dims[8])
    g = torch.Generator().manual_seed(seed)
    shape = (dims[0], o_h, o_w, dims[6])
    G = torch.randint(-3, 4, shape, generator=g).float() if dist == "int" else torch.rand(shape, generator=g) - 0.5
    return K, G


def run(G, K, dims):
    dL = mec.dgrad_gemm(G.to(DEV), K.to(DEV), dims[1], dims[2], dims[7], dims[8])
    torch.cuda.synchronize()
    return dL.cpu().numpy()


@pytest.mark.parametrize("dims", CASES)
def test_dgrad_tile(orc, dims):
    print("[case] dgrad tile", dims, flush=True)
    for dist, tol in (("int", 0.0), ("u11", 2e-6)):
        K, G = inputs(dims, dist, 61)
        ref = orc.mec_dgrad_lowered(G.numpy(), K.numpy(), dims[1], dims[2], dims[7], dims[8]).astype(np.float64)
        got = run(G, K, dims).astype(np.float64)
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("what", ["inf", "nan", "overflow", "tiny", "huge"])
def test_dgrad_values_the_split_does_not_hold(orc, what):
    dims = (3, 30, 20, 13, 3, 5, 47, 2, 1)
    print("[case] dgrad values", what, flush=True)
    K, G = inputs(dims, "u11", 62)
    G, K = G + 0.75, K.abs()
    if what == "inf":
        G[1, 7, 9, 46] = float("inf")
    elif what == "nan":
        K[2, 4, 12, 3] = float("nan")
    elif what == "overflow":
        G = G * 2e38
    elif what == "tiny":
        G = G * 1e-36
    elif what == "huge":
        G, K = G * 1e38, K * 1e-37
    ref = orc.mec_dgrad_lowered(G.numpy(), K.numpy(), dims[1], dims[2], dims[7], dims[8]).astype(np.float64)
    with np.errstate(over="ignore"):
        ref32 = ref.astype(np.float32)
    got = run(G, K, dims)
    fine = np.isfinite(ref32)
    assert np.array_equal(np.isnan(got), np.isnan(ref32))
    assert np.array_equal(got[~fine & ~np.isnan(ref32)], ref32[~fine & ~np.isnan(ref32)])
    ref, got = ref[fine], got[fine].astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# operands below 2^-133, where no bf16 part holds anything, against ordinary ones
@pytest.mark.parametrize("which", ["kernel", "gradient"])
def test_dgrad_values_below_every_part(orc, which):
    dims = (3, 30, 20, 13, 3, 5, 47, 2, 1)
    print("[case] dgrad values below every part", which, flush=True)
    K, G = inputs(dims, "u11", 63)
    K, G = (K * 4e-41, G * 1e6) if which == "kernel" else (K * 1e6, G * 4e-41)
    ref = orc.mec_dgrad_lowered(G.numpy(), K.numpy(), dims[1], dims[2], dims[7], dims[8]).astype(np.float64)
    assert np.abs(ref).max() > 1e-36
    got = run(G, K, dims).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


# as test_tile_products_left_out: every value the same, up to 48 terms, exact sums of
# the parts' products
@pytest.mark.parametrize("bits", [0x3f80ffff, 0x3f807f40, 0x3f808040])
def test_dgrad_products_left_out(orc, bits):
    dims = (1, 64, 10, 8, 3, 3, 16, 1, 1)
    print("[case] dgrad left out", hex(bits), flush=True)
    x = float(np.array([bits], np.uint32).view(np.float32)[0])
    G, K = torch.full((1, 62, 8, 16), x), torch.full((3, 3, 8, 16), x)
    ref = orc.mec_dgrad_lowered(G.numpy(), K.numpy(), 64, 10, 1, 1).astype(np.float64)
    got = run(G, K, dims).astype(np.float64)
    assert (np.abs(got - ref) <= 2.0 ** -23 * np.abs(ref)).all()
