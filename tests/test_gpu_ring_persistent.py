"""The ring GEMM kernel where a workgroup takes several tiles: the operand ring
and the scales run on across tiles, with K shorter than, as long as and longer
than the ring (4 or 5 steps of 64; E4M3 3 of 128), an odd step count, and a last
row and column of tiles that are masked.  Every tile shape is forced on at least
three tiles a workgroup (256 CUs); the last tests leave the choice to the plan."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_28003_amd import synth, w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

RING = (64, 65, 66, 67, 68)  # 256 rows x 256, 224, 192, 160, 128 weight rows
M, N = 1100, 45000           # 5 x 176 tiles of the widest, 5 x 352 of the narrowest
F = 22512                    # gated: 5 x 176 and 5 x 352


def codes(g, rows, k):
    return torch.randint(-127, 128, (rows, k), generator=g, device=DEV, dtype=torch.int8)


def packed(q):
    """Codes in the packed layout, on the GPU (16 x 64 fragments, lane l holding
    row l % 16, columns 16 (l / 16) .. + 15)."""
    n, k = q.shape
    rp, kp = -(-n // 16) * 16, -(-k // 64) * 64
    full = torch.zeros((rp, kp), dtype=torch.int8, device=DEV)
    full[:n, :k] = q
    return full.view(rp // 16, 16, kp // 64, 4, 16).permute(0, 2, 3, 1, 4).contiguous().view(torch.uint8).flatten()


def force(name, tile):
    w8a8.clear_plan_overrides()
    w8a8.set_plan_override("NO_STREAM", 1)
    w8a8.set_plan_override(name, tile)


def test_packed_helper():
    q = codes(torch.Generator(device=DEV).manual_seed(1), 33, 144)
    ref = torch.from_numpy(w8a8.rowmajor_to_frag(q.cpu().numpy())).view(torch.uint8)
    assert torch.equal(packed(q).cpu(), ref.flatten())


@pytest.mark.parametrize("k", [16, 64, 128, 256, 320, 384, 448])
def test_int8_many_tiles_exact(k):
    """Sums below 127^2 * 448 < 2^24: binary32 products of the codes are exact, and
    so is the whole reference, two scalings included."""
    g = torch.Generator(device=DEV).manual_seed(k)
    x = torch.randn((M, k), generator=g, device=DEV).bfloat16()
    qw = codes(g, N, k)
    sw = torch.rand(N, generator=g, device=DEV) * 0.01 + 0.001
    qp, sx = w8a8.quantize_act(x)
    qx = torch.from_numpy(w8a8.frag_to_rowmajor(qp.cpu().numpy(), M, k)).to(DEV)
    acc = qx.float() @ qw.float().t()
    y = (acc * sx[:, None]) * sw
    layer = w8a8.LinearW8A8(N, k, packed(qw), sw, None)
    for tile in RING:
        print("ring int8", tile, M, N, k, flush=True)
        force("GEMM_TILE", tile)
        assert torch.equal(w8a8.gemm_i8_i32(qp, M, layer.wq, N, k), acc.int()), tile
        assert torch.equal(w8a8.linear(layer, x, torch.float32), y), tile
        assert torch.equal(w8a8.linear(layer, x, torch.bfloat16), y.bfloat16()), tile


@pytest.mark.parametrize("k", [64, 256, 320, 448])
def test_int8_gated_many_tiles_bit_identical(k):
    """Gate and up on the ring give the h of the LDS tile (exact sums, one epilogue)."""
    g = torch.Generator(device=DEV).manual_seed(k + 1)
    x = torch.randn((M, k), generator=g, device=DEV).bfloat16()
    part = [w8a8.LinearW8A8(F, k, packed(codes(g, F, k)), torch.rand(F, generator=g, device=DEV) * 0.01, None)
            for _ in range(2)]
    layer = w8a8.FfnW8A8(k, F, part[0], part[1], w8a8.LinearW8A8(k, F, part[0].wq, part[0].s_w, None))
    qp, sx = w8a8.quantize_act(x)
    force("GLU_TILE", 5)
    ref = w8a8.ffn_gate_up(layer, qp, sx, M).view(torch.int16)
    for tile in RING:
        print("ring gated int8", tile, M, F, k, flush=True)
        force("GLU_TILE", tile)
        assert torch.equal(w8a8.ffn_gate_up(layer, qp, sx, M).view(torch.int16), ref), tile


@pytest.mark.parametrize("k", [64, 160, 448])
def test_bf16_many_tiles(k):
    """Integers up to 8 in bf16: every sum is exact in binary32, in any order."""
    g = torch.Generator(device=DEV).manual_seed(k + 2)
    x, w = (torch.randint(-8, 9, (r, k), generator=g, device=DEV).bfloat16() for r in (M, N))
    ref = (x.float() @ w.float().t()).bfloat16()
    wp = w8a8.pack_bf16(w)
    for tile in RING:
        print("ring bf16", tile, M, N, k, flush=True)
        force("GEMM_TILE", tile)
        assert torch.equal(w8a8.bf16_linear(x, wp, N, k), ref), tile


@pytest.mark.parametrize("k", [128, 256, 384, 512, 640])
def test_fp8_many_tiles(k):
    """Codes of small integers: products and sums are exact, the scalings too."""
    g = torch.Generator(device=DEV).manual_seed(k + 3)
    x, w = (torch.randint(-8, 9, (r, k), generator=g, device=DEV).float() for r in (M, N))
    x[:, 0], w[:, 0] = 8.0, 8.0  # row maximum 8: the codes of even values are multiples of 16 up to 448
    x, w = (torch.where(t.abs() % 2 == 1, t.sign() * 4, t) for t in (x, w))
    (qx, sx), (qw, sw) = w8a8.fp8_quantize_act(x), w8a8.fp8_quantize_weights(w)
    dec = lambda q, r: torch.from_numpy(w8a8.frag_to_rowmajor(q.cpu().numpy(), r, k).view(np.uint8).copy()) \
        .view(torch.float8_e4m3fn).float().to(DEV)
    layer = w8a8.LinearW8A8(N, k, qw, sw * (1 + torch.arange(N, device=DEV) % 7), None)
    y = ((dec(qx, M) @ dec(qw, N).t()) * sx[:, None]) * layer.s_w
    force("GEMM_TILE", RING[-1])
    print("ring fp8", M, N, k, flush=True)
    for dt in (torch.float32, torch.bfloat16):
        assert torch.equal(w8a8.fp8_linear(layer, x, dt), y.to(dt)), dt


@pytest.mark.parametrize("dt,m,n,k", [("int8", 256, 262144, 256), ("int8", 129, 262144, 64), ("fp8", 100, 262144, 384),
                                      ("int8", 4096, 12288, 256)])
def test_planned_short_k(dt, m, n, k):
    """The plan's own choice on short K, against the oracle on sampled columns."""
    print("planned", dt, m, n, k, flush=True)
    rng = np.random.default_rng(n + k)
    x = synth.to_bf16_bits(rng.standard_normal((m, k)).astype(np.float32))
    w = synth.to_bf16_bits((rng.standard_normal((n, k)) * np.exp(rng.uniform(-2, 2, (n, 1)))).astype(np.float32))
    dev = lambda u: torch.from_numpy(u.view(np.int16)).view(torch.bfloat16).to(DEV)
    cols = np.sort(rng.choice(n, 512, replace=False))
    if dt == "int8":
        layer = w8a8.LinearW8A8.from_weight(dev(w))
        wq, sw = oracle.quantize_weights(w[cols], None)
        ref = oracle.w8a8_linear(x, wq, sw, None, "bf16")
        y = w8a8.lm_head(layer, dev(x))[:, torch.from_numpy(cols).to(DEV)].contiguous().cpu()
        np.testing.assert_array_equal(y.view(torch.int16).numpy().view(np.uint16), ref)
    else:
        layer = w8a8.fp8_linear_layer(dev(w))
        y = w8a8.fp8_lm_head(layer, dev(x))[:, torch.from_numpy(cols).to(DEV)].double()
        ref = dev(x).double() @ dev(w[cols]).double().t()
        # E4M3 codes: a relative 2^-4 an operand, independent over K
        assert float((y - ref).norm() / ref.norm()) <= 0.06
