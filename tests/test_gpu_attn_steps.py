"""Decode attention at the edges of a wave's 32 rows, a workgroup's 128 and a
merge's partials, with windows that begin at any row, for every head count and
both caches: against binary64 on the cache's own values."""

import numpy as np
import pytest
import torch

from paper_2608_28003_amd import w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HD = 256


@pytest.mark.parametrize("int8", [True, False])
@pytest.mark.parametrize("heads", [1, 2, 4, 8])
@pytest.mark.parametrize("pos,rows", [(0, 1), (1, 2), (40, 31), (32, 33), (200, 127), (128, 129), (300, 97),
                                      (8500, 8193), (40000, 33003), (70000, 65665)])
def test_rows(int8, heads, pos, rows):
    print("attn", int8, heads, pos, rows, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(pos + heads)
    k, v = ((torch.randn((pos + 3, HD), generator=g, device=DEV) * 2).to(torch.bfloat16) for _ in range(2))
    qkv = (torch.randn((heads + 2) * HD, generator=g, device=DEV) * 2).to(torch.bfloat16)
    c = w8a8.KVCache(pos + 3, int8=int8, device=DEV)
    c.fill(0, k, v)  # rows past pos are there and must not count
    out = w8a8.attn_decode(qkv, c, pos, rows, n_heads=heads).double().view(heads, HD)
    t0 = pos + 1 - rows
    if int8:
        kd, vd = (x[t0:pos + 1].double() * s[t0:pos + 1].double()[:, None] for x, s in ((c.k, c.sk), (c.v, c.sv)))
    else:
        kd, vd = c.k[t0:pos + 1].view(torch.bfloat16).double(), c.v[t0:pos + 1].view(torch.bfloat16).double()
        assert torch.equal(c.k[pos].view(torch.bfloat16), qkv[heads * HD:(heads + 1) * HD])
    q = qkv[:heads * HD].double().view(heads, HD)
    ref = torch.softmax(q @ kd.t() / 16.0, 1) @ vd
    # one bf16 rounding (2^-9 of the value), and binary32 scores: 256 products of
    # |q . k| <= 2^10 or so, over 16, each rounded to 2^-24, move a weight by 2^-12 at most
    scale = vd.abs().amax()
    err = (out - ref).abs()
    assert (err <= ref.abs() * 2.0 ** -8 + scale * 2.0 ** -12).all(), err.max().item()
    rel = float(torch.linalg.norm(out - ref) / torch.linalg.norm(ref))
    assert rel <= 2.5e-3, rel  # bf16 rounding alone: 1.7e-3
