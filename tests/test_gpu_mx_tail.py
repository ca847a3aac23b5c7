"""MXFP4 GEMMs whose last round of 256 x 256 tiles is small enough to run as
64 x 64 sixteenths in a second launch (at most 16 tiles): the plan,
and exact sums against the oracle on ragged shapes whose last tiles have
parts outside the output."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_from_dev, poison_bf16, u8_to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,rem", [(4224, 4001, 1152, 16), (4097, 4096, 1056, 16),
                                       (2290, 7400, 1152, 5), (4224, 4001, 96, 16),
                                       (4097, 4096, 1024, 16)])
def test_sixteenths_are_exact(M, N, K, rem):
    tiles = ((M + 255) // 256) * ((N + 255) // 256)
    assert tiles % 256 == rem
    p = sol.gemm_plan(M, N, K, sol.FORMAT_MXFP4)
    assert p["tile"] == 256 and p["workgroups"] == tiles + 15 * rem
    g = np.random.Generator(np.random.PCG64(M + N + K))
    ac = g.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    bc = g.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    as_ = np.full((M, K // 32), 127, np.uint8)
    bs = np.full((N, K // 32), 125, np.uint8)
    out = poison_bf16((M, N))
    sol.mxfp4_gemm(u8_to_dev(ac), u8_to_dev(as_), u8_to_dev(bc), u8_to_dev(bs), None, out)
    torch.cuda.synchronize()
    assert np.array_equal(bf16_from_dev(out), O.bf16_output(O.mxfp4_gemm_ref(ac, as_, bc, bs)))
