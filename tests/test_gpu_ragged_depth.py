"""Reduction lengths that are no multiple of the 128-element K stage: every
count of blocks in the last stage, on the wave-K kernel (32 x 32
tiles, K shares of one to three stages), the lane kernel's 128 x 128 and
256 x 256 tiles and the workgroup-shared kernel, and on MXFP4's wave-K kernel.  Block scales are powers of
two that differ from block to block, so a misplaced scale shows, and all
FP32 sums are exact: the output is the oracle's bit for bit.  The bytes
behind the operands are large codes and scales that must not be read."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_from_dev, device, f32_to_dev

pytestmark = pytest.mark.gpu

WAVEK = ([(33, 40, K) for K in range(144, 272, 16) if K != 256] + [(1, 9, 656), (65, 100, 528)]
         + [(100, 1000, 208), (70, 650, 1104), (128, 1152, 1120), (256, 128, 160)])
LANE = ([(40, 48, K) for K in (16, 48, 64, 80, 96, 112)] + [(2, 5, 112), (129, 260, 96)]
        + [(8, 9, 16), (131, 259, 16), (131, 300, 48), (2930, 2235, 144), (1024, 2432, 1120)])
LANE256 = ([(2564, 3087, K) for K in (160, 176, 208, 240, 272)] + [(3601, 4083, K) for K in (80, 112, 144)]
           + [(4353, 4363, 16), (4353, 4363, 48), (3601, 4083, 1088)])
SHARED = [(7, 40, 16), (3601, 4083, 16), (3601, 4083, 48), (3601, 4083, 192), (1, 3, 32)]


def kernel_of(M, N, K):
    p = sol.gemm_plan(M, N, K)
    return p["kernel"], p["tile"]


def test_plans():
    lane = "nvfp4_gemm_lane_kernel"
    assert {kernel_of(*s) for s in WAVEK} == {("nvfp4_gemm_wavek_kernel", 32)}
    assert {kernel_of(*s) for s in LANE} == {(lane, 128)}
    assert {kernel_of(*s) for s in LANE256} == {(lane, 256)}
    assert {kernel_of(*s) for s in SHARED} == {("nvfp4_gemm_kernel", 256)}


def guarded(a, fill):
    """`a` on the GPU with 256 bytes of `fill` behind it."""
    flat = torch.full((a.size + 256,), fill, dtype=torch.uint8, device=device())
    t = flat[: a.size].view(*a.shape)
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("M,N,K", WAVEK + LANE + LANE256 + SHARED)
def test_ragged_depth_is_exact(M, N, K):
    g = np.random.Generator(np.random.PCG64(M * 1000 + N + K))

    def operand(rows):
        codes = g.integers(0, 256, size=(rows, K // 2), dtype=np.uint8)
        scales = g.choice(np.array([0x30, 0x38, 0x40], np.uint8), size=(rows, K // 16))
        return codes, scales
    (ac, as_), (bc, bs) = operand(M), operand(N)
    one = f32_to_dev(1.0)
    out = sol.nvfp4_gemm(guarded(ac, 0x77), guarded(as_, 0x7E), one, guarded(bc, 0x77),
                         guarded(bs, 0x7E), one)
    torch.cuda.synchronize()
    ref = O.nvfp4_gemm_ref(ac, as_, np.float32(1), bc, bs, np.float32(1))
    assert np.array_equal(bf16_from_dev(out), O.bf16_output(ref))


MX_WAVEK = [(33, 40, K) for K in (160, 192, 224, 288)] + [(1, 9, 672), (65, 100, 544),
                                                          (250, 1900, 160), (70, 650, 1120),
                                                          (128, 1152, 1120), (256, 1920, 160)]


@pytest.mark.parametrize("M,N,K", MX_WAVEK)
def test_mx_ragged_depth_is_exact(M, N, K):
    assert sol.gemm_plan(M, N, K, sol.FORMAT_MXFP4)["kernel"] == "mxfp4_gemm_wavek_kernel"
    g = np.random.Generator(np.random.PCG64(M * 1000 + N + K))

    def operand(rows):
        codes = g.integers(0, 256, size=(rows, K // 2), dtype=np.uint8)
        scales = g.integers(126, 129, size=(rows, K // 32), dtype=np.uint8)
        return codes, scales
    (ac, as_), (bc, bs) = operand(M), operand(N)
    out = sol.mxfp4_gemm(guarded(ac, 0x77), guarded(as_, 0xFF), guarded(bc, 0x77), guarded(bs, 0xFF))
    torch.cuda.synchronize()
    ref = O.mxfp4_gemm_ref(ac, as_, bc, bs)
    assert np.array_equal(bf16_from_dev(out), O.bf16_output(ref))
