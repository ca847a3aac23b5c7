"""MXFP4 GEMMs whose last round of 256 x 256 tiles is small enough to run as
64 x 64 sixteenths in a second launch (at most 16 tiles): the plan, and exact
sums against the oracle on ragged shapes whose last tiles have parts outside
the output.  Block scales are powers of two that differ from block to block,
so a part that took scales from another row, tile or K group shows (products
are multiples of 2^-4 and sums stay under 36 * 4 * K < 2^18: exact in FP32).
Bytes behind the operands are large codes and NaN scales, elements behind the
output must keep their value."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_from_dev, poison_bf16
from test_gpu_ragged_depth import guarded

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

    def operand(rows):
        codes = g.integers(0, 256, size=(rows, K // 2), dtype=np.uint8)
        return codes, g.integers(126, 129, size=(rows, K // 32), dtype=np.uint8)
    (ac, as_), (bc, bs) = operand(M), operand(N)
    flat = poison_bf16((M * N + 64,))
    sol.mxfp4_gemm(guarded(ac, 0x77), guarded(as_, 0xFF), guarded(bc, 0x77), guarded(bs, 0xFF), None,
                   flat[: M * N].view(M, N))
    torch.cuda.synchronize()
    got = bf16_from_dev(flat)
    assert np.array_equal(got[: M * N].reshape(M, N), O.bf16_output(O.mxfp4_gemm_ref(ac, as_, bc, bs)))
    assert np.all(got[M * N:] == 0x7FC1)
