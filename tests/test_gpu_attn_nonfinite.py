"""Decode attention over caches that hold infinities and NaN: an infinite value
under a positive weight stays infinite with its sign, both signs or a NaN give
NaN, other dimensions are untouched; rows whose score is -inf have no weight,
also where they are all the rows that a wave takes at a time."""

import pytest
import torch

from paper_2608_28003_amd import w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HD = 256
INF = float("inf")


def setup(int8, heads, rows):
    g = torch.Generator(device=DEV).manual_seed(rows + heads)
    k, v = ((torch.randn((rows, HD), generator=g, device=DEV)).to(torch.bfloat16) for _ in range(2))
    qkv = (torch.randn((heads + 2) * HD, generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    qkv[:heads * HD:HD] = 2.0  # dimension 0 of every head
    c = w8a8.KVCache(rows, int8=int8, device=DEV)
    c.fill(0, k, v)
    return c, qkv


def check(c, qkv, heads, rows):
    out = w8a8.attn_decode(qkv, c, rows - 1, rows, n_heads=heads).double().view(heads, HD)
    if c.int8:
        kd, vd = (x.double() * s.double()[:, None] for x, s in ((c.k, c.sk), (c.v, c.sv)))
        score = (qkv[:heads * HD].double().view(heads, HD) @ c.k.double().t()) * c.sk.double() / 16.0
    else:
        kd, vd = c.k.view(torch.bfloat16).double(), c.v.view(torch.bfloat16).double()
        score = (qkv[:heads * HD].double().view(heads, 1, HD) * kd).sum(-1) / 16.0
    wt = torch.softmax(score, 1)
    ref = (wt[:, :, None] * vd).sum(1)
    fin = torch.isfinite(ref)
    for kind in (torch.isposinf, torch.isneginf, torch.isnan):
        assert torch.equal(kind(out), kind(ref)), kind.__name__
    # one bf16 rounding, and binary32 scores and sums
    scale = vd[torch.isfinite(vd)].abs().amax()
    assert ((out - ref).abs()[fin] <= ref.abs()[fin] * 2.0 ** -8 + scale * 2.0 ** -12).all()
    return ref


@pytest.mark.parametrize("heads", [1, 2, 4, 8])
@pytest.mark.parametrize("rows", [1, 40, 300, 5000])
def test_values_bf16(heads, rows):
    print("attn bf16 inf", heads, rows, flush=True)
    c, qkv = setup(False, heads, rows)
    v = c.v.view(torch.bfloat16)
    for d, marks in ((3, {0: INF}), (77, {rows // 2: -INF}), (130, {0: INF, rows // 2: -INF}),
                     (200, {rows // 3: float("nan")}), (255, {rows // 2: INF, rows // 3: INF})):
        for r, x in marks.items():
            if r < rows - 1:
                v[r, d] = x
    qkv[(heads + 1) * HD + 9] = -INF  # the new row's own value
    ref = check(c, qkv, heads, rows)
    assert torch.isneginf(ref[:, 9]).all() and int(torch.isfinite(ref[0]).sum()) >= HD - 6


@pytest.mark.parametrize("heads", [1, 4, 8])
@pytest.mark.parametrize("rows", [40, 300])
def test_value_scale_int8(heads, rows):
    """An infinite value scale: infinite where the code is not 0, else NaN."""
    print("attn int8 inf scale", heads, rows, flush=True)
    c, qkv = setup(True, heads, rows)
    c.sv[rows // 2] = INF
    ref = check(c, qkv, heads, rows)
    assert not torch.isfinite(ref).any() and torch.isinf(ref).any()


@pytest.mark.parametrize("int8", [True, False])
@pytest.mark.parametrize("heads", [1, 4, 8])
@pytest.mark.parametrize("lo,hi,rows", [(0, 32, 64), (32, 64, 300), (0, 128, 300), (128, 256, 1000)])
def test_scores_of_minus_infinity(int8, heads, lo, hi, rows):
    print("attn -inf scores", int8, heads, lo, hi, rows, flush=True)
    c, qkv = setup(int8, heads, rows)
    if int8:
        c.k[lo:hi] = 0
        c.k[lo:hi, 0] = 127
        c.sk[lo:hi] = -INF
    else:
        kb = c.k.view(torch.bfloat16)
        kb[lo:hi] = 0
        kb[lo:hi, 0] = -INF
    ref = check(c, qkv, heads, rows)
    assert torch.isfinite(ref).all()
