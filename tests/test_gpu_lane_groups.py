"""128 x 128 tiles of the NVFP4 GEMM in two wave groups that share the K
stages (long K): whole pairs of stages, an odd stage count, a last stage of 5
blocks and one of 1, K halves with an even and an odd stage count, 128 x 128
quadrants of a last round, more tiles than CUs; ragged M and N.  Codes are
uniform and block scales 0.5, 1 or 2, so the FP32 sums are exact and the
output is the oracle's bit for bit: a stage left out, counted twice or under
another stage's scales shows."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_from_dev, f32_to_dev, poison_bf16
from test_gpu_ragged_depth import guarded

pytestmark = pytest.mark.gpu

CASES = [  # M, N, K, K halves over two workgroups
    (600, 2000, 2048, False), (513, 2057, 3456, False), (1130, 3050, 3408, False),
    (1130, 3049, 3344, False), (600, 2000, 4096, True), (600, 2000, 6912, True),
    (4352, 4352, 2048, False), (2600, 2600, 6160, False)]


@pytest.mark.parametrize("M,N,K,split", CASES)
def test_exact_sums_in_two_groups(M, N, K, split):
    plan = sol.gemm_plan(M, N, K, with_workspace=split)
    assert plan["kernel"] == "nvfp4_gemm_lane_kernel" and plan["tile"] >= 128 and plan["splits"] == (2 if split else 1)
    g = np.random.Generator(np.random.PCG64(M + N + K))
    scale = np.array([0x30, 0x38, 0x40], np.uint8)
    ac, bc = (g.integers(0, 256, size=(r, K // 2), dtype=np.uint8) for r in (M, N))
    as_, bs = (scale[g.integers(0, 3, size=(r, K // 16))] for r in (M, N))
    aa, ba = np.float32(2.0 ** -3), np.float32(2.0 ** 5)
    out = poison_bf16((M, N))
    sol.nvfp4_gemm(guarded(ac, 0x77), guarded(as_, 0x7E), f32_to_dev(aa), guarded(bc, 0x77), guarded(bs, 0x7E),
                   f32_to_dev(ba), None, out, split=split)
    torch.cuda.synchronize()
    ref = O.nvfp4_gemm_ref(ac, as_, aa, bc, bs, ba)
    assert np.array_equal(bf16_from_dev(out), O.bf16_output(ref))
