"""Small NVFP4 tensors are quantized in one launch (up to 18 workgroups of
1024 pieces of 8 elements), larger ones in two passes: codes, scales and
alpha equal the oracle's on both sides of every boundary of that choice, and
the two separate passes give the same."""
import numpy as np
import pytest
import torch

import oracle.nvfp4 as O
import paper_2604_06916_amd as sol
from gpu_util import bf16_to_dev, device, f32_bits, poison_u8, u8_from_dev
from workloads import draw_activations

pytestmark = pytest.mark.gpu

WG = 1024 * 8          # elements of one workgroup
SIZES = [16, 48, WG - 16, WG, WG + 16, 4 * WG, 4 * WG + 16, 8 * WG - 32, 8 * WG + 16, 17 * WG + 496,
         18 * WG, 18 * WG + 16, 19 * WG]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("where", ["first", "last", "zeros"])
def test_matches_the_oracle_and_the_two_passes(n, where):
    K = 16
    rows = n // K
    xb = draw_activations("normal", rows, K, seed=n)
    if where == "zeros":
        xb[:] = 0
        xb[::3, ::5] = 0x8000
    else:
        # the tensor's largest element in the first or last piece: every
        # workgroup has to see it
        xb.reshape(-1)[0 if where == "first" else -1] = 0xC2F7     # -123.5
    x = bf16_to_dev(xb)
    rc, rs, ra = O.nvfp4_quantize_ref(xb)
    flat_c, flat_s = poison_u8((n // 2 + 64,)), poison_u8((n // 16 + 64,))
    codes, scales = flat_c[: n // 2].view(rows, K // 2), flat_s[: n // 16].view(rows, 1)
    _, _, alpha = sol.nvfp4_quantize(x, codes, scales)
    ws = torch.empty(sol.nvfp4_quantize_workspace_bytes(rows, K), dtype=torch.uint8, device=device())
    c2, s2, a2 = torch.empty_like(codes), torch.empty_like(scales), torch.empty_like(alpha)
    sol.nvfp4_quantize_amax(x, ws)
    sol.nvfp4_quantize_encode(x, c2, s2, a2, ws)
    torch.cuda.synchronize()
    assert np.array_equal(u8_from_dev(codes), rc) and np.array_equal(u8_from_dev(scales), rs)
    assert f32_bits(alpha.item()) == f32_bits(ra)
    assert torch.equal(codes, c2) and torch.equal(scales, s2) and torch.equal(alpha, a2)
    assert bool((flat_c[n // 2:] == 0xAB).all()) and bool((flat_s[n // 16:] == 0xAB).all())
