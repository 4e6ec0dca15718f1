"""Plain products whose plan is an LDS tile or a few-column split: short K, long K
of few columns, very wide outputs too narrow for the lm_head's widest tile.  The
plan's own choice, on operands whose sums are exact in binary32 whatever the
order, so every result is checked bit for bit."""

import pytest
import torch

from paper_2608_28003_amd import w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def ints(g, rows, k, top):
    return torch.randint(-top, top + 1, (rows, k), generator=g, device=DEV).float()


@pytest.mark.parametrize("m,n,k", [(64, 2304, 144), (129, 16384, 256), (256, 16400, 1152), (100, 20480, 640),
                                   (128, 32000, 208), (1000, 1536, 256), (2048, 1160, 128), (17, 65536, 640),
                                   (31, 65552, 208)])
def test_int8(m, n, k):
    """Codes of integers: |x| <= 63 with a maximum of 127 / 2, so the codes are 2 x
    (sums below 2^24 for K <= 1152)."""
    print("int8 plan", m, n, k, flush=True)
    g = torch.Generator(device=DEV).manual_seed(m + n)
    x, w = ints(g, m, k, 50), ints(g, n, k, 50)
    x[:, 0], w[:, 0] = 63.5, 63.5
    layer = w8a8.LinearW8A8.from_weight(w)
    codes = lambda t: t * 2
    y = ((codes(x) @ codes(w).t()) * 0.5) * 0.5
    assert torch.equal(w8a8.linear(layer, x.bfloat16(), torch.float32), y)
    assert torch.equal(w8a8.linear(layer, x.bfloat16(), torch.bfloat16), y.bfloat16())


@pytest.mark.parametrize("m,n,k", [(256, 12288, 128), (70, 16384, 256), (120, 32000, 384), (512, 2304, 256),
                                   (1000, 1160, 512), (24, 65536, 640), (129, 20480, 128)])
def test_fp8(m, n, k):
    """Powers of two up to 448 = 1.75 x 2^8 are their own E4M3 codes at scale 1."""
    print("fp8 plan", m, n, k, flush=True)
    g = torch.Generator(device=DEV).manual_seed(m + n)
    x, w = (torch.exp2(torch.randint(3, 8, (r, k), generator=g, device=DEV).float()) *
            torch.randint(-1, 2, (r, k), generator=g, device=DEV) for r in (m, n))
    x[:, 0], w[:, 0] = 448.0, 448.0
    y = x @ w.t()
    layer = w8a8.fp8_linear_layer(w)
    assert torch.equal(w8a8.fp8_linear(layer, x.bfloat16(), torch.float32), y)
    assert torch.equal(w8a8.fp8_linear(layer, x.bfloat16(), torch.bfloat16), y.bfloat16())


@pytest.mark.parametrize("m,n,k", [(64, 12288, 128), (200, 16384, 640), (96, 20480, 256), (512, 8192, 1024),
                                   (4096, 640, 4096), (1000, 650, 4224), (2048, 2304, 4096), (20, 16400, 4128)])
def test_bf16(m, n, k):
    print("bf16 plan", m, n, k, flush=True)
    g = torch.Generator(device=DEV).manual_seed(m + n)
    x, w = ints(g, m, k, 8), ints(g, n, k, 8)
    y = w8a8.bf16_linear(x.bfloat16(), w8a8.pack_bf16(w.bfloat16()), n, k)
    assert torch.equal(y, (x @ w.t()).bfloat16())
