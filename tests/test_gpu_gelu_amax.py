"""nvfp4_gelu_amax: GELU (tanh form) in place with the amax pass of its
result.  Every finite BF16 value against float64 (within half a BF16 step and
the FP32 evaluation's 2^-15), infinities and NaN as the definition gives them,
and the quantization that it starts equal, bit for bit, to nvfp4_quantize of
the same result.  Sizes: one block, a partial small-unroll iteration, partial
second rounds of both unrolls."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_from_dev, bf16_to_dev, device
from workloads import draw_activations

pytestmark = pytest.mark.gpu


def run(x):
    rows, K = x.shape
    ws = torch.empty(max(sol.nvfp4_quantize_workspace_bytes(rows, K), 256), dtype=torch.uint8, device=device())
    assert sol.nvfp4_gelu_amax(x, ws) is x
    u8 = dict(dtype=torch.uint8, device=device())
    q = sol.nvfp4_quantize_encode(x, torch.empty(rows, K // 2, **u8), torch.empty(rows, K // 16, **u8),
                                  torch.empty(1, device=device()), ws)
    torch.cuda.synchronize()
    return q


def test_every_value():
    bits = np.arange(1 << 16, dtype=np.uint16).reshape(256, 256)
    x = bf16_to_dev(bits)
    run(x)
    got = O.bf16_bits_to_f32(bf16_from_dev(x)).astype(np.float64)
    with np.errstate(all="ignore"):
        v = O.bf16_bits_to_f32(bits).astype(np.float64)
        z = np.sqrt(2 / np.pi) * (v + 0.044715 * v ** 3)
        want = v / (1 + np.exp(-2 * z))
    fin = np.isfinite(v)
    # 2^-8: half a BF16 step (8 significant bits); 2^-15: the exponent, at most
    # 128 in base 2, after three FP32 roundings; absolute: the sigmoid is
    # flushed to zero below 2^-126, where |x| is under 16
    err = np.abs(got[fin] - want[fin])
    assert np.all(err <= np.abs(want[fin]) * (2.0 ** -8 + 2.0 ** -15) + 2.0 ** -122)
    assert np.isnan(got[np.isnan(v)]).all() and got[v == np.inf] == np.inf and np.isnan(got[v == -np.inf]).all()
    # and no element further from float64 than torch's kernel for the same form
    t = torch.nn.functional.gelu(bf16_to_dev(bits), approximate="tanh")
    t = O.bf16_bits_to_f32(bf16_from_dev(t)).astype(np.float64)
    assert np.all(err <= np.abs(t[fin] - want[fin]))


@pytest.mark.parametrize("rows,K", [(1, 16), (3, 1040), (777, 1232), (2000, 3008), (3001, 4096)])
def test_equals_quantize_of_the_result(rows, K):
    x = bf16_to_dev(draw_activations("t3_1pct", rows, K, seed=rows + K))
    ref = torch.nn.functional.gelu(x.double(), approximate="tanh")
    got = run(x)
    assert (x.double() - ref).norm() <= 2.0 ** -8 * ref.norm()
    want = sol.nvfp4_quantize(x)
    torch.cuda.synchronize()
    assert all(torch.equal(g.view(torch.uint8), w.view(torch.uint8)) for g, w in zip(got, want))
