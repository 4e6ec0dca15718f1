"""The K-wave and the ring GEMM kernels on tile edges: every tile of both, forced
through the planner overrides, on shapes that leave rows, columns and fragment
columns over (and on fewer of each than one tile)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_28003_amd import synth, w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

KWAVE = (32, 33, 34, 35, 36, 37, 38, 39, 40, 44, 45, 46)
KWAVE_GLU = (34, 39, 40, 41, 42, 43, 44, 45)
RING = (64, 65, 66, 67, 68)
# one row and column block, ragged in every direction (an odd column count has
# no aligned row stride), and several tiles of the largest shape
SHAPES = [(1, 16, 64), (77, 203, 1168), (300, 1000, 1152), (530, 520, 448)]


def dev_bf16(u16):
    return torch.from_numpy(np.ascontiguousarray(u16).view(np.int16)).view(torch.bfloat16).to(DEV)


def force(name, tile):
    w8a8.clear_plan_overrides()
    w8a8.set_plan_override("NO_STREAM", 1)
    w8a8.set_plan_override(name, tile)


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_int8_tiles_exact(m, n, k):
    rng = np.random.default_rng(m + n)
    qa = rng.integers(-127, 128, (m, k), dtype=np.int8)
    qb = rng.integers(-127, 128, (n, k), dtype=np.int8)
    acc_o = oracle.gemm_i32(qa, qb)
    A = torch.from_numpy(w8a8.rowmajor_to_frag(qa)).to(DEV)
    B = torch.from_numpy(w8a8.rowmajor_to_frag(qb)).to(DEV)
    x = synth.to_bf16_bits(rng.standard_normal((m, k)).astype(np.float32))
    w = synth.to_bf16_bits(rng.standard_normal((n, k)).astype(np.float32))
    layer = w8a8.LinearW8A8.from_weight(dev_bf16(w))
    wq, sw = oracle.quantize_weights(w, None)
    for tile in KWAVE + RING:
        print("int8 tile", tile, m, n, k, flush=True)
        force("GEMM_TILE", tile)
        acc = w8a8.gemm_i8_i32(A, m, B, n, k).cpu().numpy()
        np.testing.assert_array_equal(acc, acc_o, err_msg="tile %d" % tile)
        for dt, name in ((torch.float32, "f32"), (torch.bfloat16, "bf16")):
            y = w8a8.linear(layer, dev_bf16(x), dt).cpu()
            got = y.numpy() if name == "f32" else y.view(torch.int16).numpy().view(np.uint16)
            np.testing.assert_array_equal(got, oracle.w8a8_linear(x, wq, sw, None, name),
                                          err_msg="tile %d %s" % (tile, name))


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
@pytest.mark.parametrize("m,n,k", [(1, 16, 128), (77, 203, 1152), (300, 1000, 640)])
def test_float_tiles(dt, m, n, k):
    """Against binary64 products of the same operands.  bf16: binary32 sums and
    one rounding of the output.  E4M3: the matrix instruction keeps at least 15
    bits below the largest product of a 128-wide block, the blocks add in
    binary32 (the allowance of the FP8 parity tests)."""
    g = torch.Generator().manual_seed(m)
    x, w = (torch.randn(r, k, generator=g).bfloat16().to(DEV) for r in (m, n))
    if dt == "bf16":
        wp, a, b = w8a8.pack_bf16(w), x.double(), w.double()
        call = lambda: w8a8.bf16_linear(x, wp, n, k)
        allowed = 2.0 ** -8 * (a @ b.t()).abs() + k * 2.0 ** -24 * (a.abs() @ b.abs().t())
    else:
        (qx, _), (qw, _) = w8a8.fp8_quantize_act(x), w8a8.fp8_quantize_weights(w)
        dec = lambda q, r: torch.from_numpy(w8a8.frag_to_rowmajor(q.cpu().numpy(), r, k).view(np.uint8).copy()) \
            .view(torch.float8_e4m3fn).double().to(DEV)
        a, b = dec(qx, m), dec(qw, n)
        call = lambda: w8a8.fp8_gemm_f32(qx, m, qw, n, k)
        big = sum(a[:, i:i + 128].abs().amax(1)[:, None] * b[:, i:i + 128].abs().amax(1)[None]
                  for i in range(0, k, 128))
        allowed = 2.0 ** -8 * big + (k + 8) * 2.0 ** -24 * (a.abs() @ b.abs().t())
    ref = a @ b.t()
    for tile in KWAVE + (RING if dt == "bf16" else RING[-1:]):
        print(dt, "tile", tile, m, n, k, flush=True)
        force("GEMM_TILE", tile)
        over = (call().double() - ref).abs() - allowed
        assert float(over.max()) <= 0.0, tile


@pytest.mark.parametrize("m,d,f", [(1, 64, 16), (77, 1152, 208), (300, 448, 1008), (530, 1088, 464)])
def test_gated_tiles_bit_identical(m, d, f):
    """Every gated tile gives the h of the LDS tile (exact sums, one epilogue)."""
    cfg = synth.ffn_config(m=m, d=d, f=f)
    one = lambda n: torch.ones(n, device=DEV)
    layer = w8a8.FfnW8A8.from_weights(dev_bf16(cfg["w_gate"]), dev_bf16(cfg["w_up"]),
                                      dev_bf16(cfg["w_down"]), one(d), one(f))
    qx, sx = w8a8.quantize_act(dev_bf16(cfg["x"]))
    force("GLU_TILE", 5)
    ref = w8a8.ffn_gate_up(layer, qx, sx, m).cpu().view(torch.int16)
    for tile in KWAVE_GLU + RING:
        print("gated tile", tile, m, d, f, flush=True)
        force("GLU_TILE", tile)
        h = w8a8.ffn_gate_up(layer, qx, sx, m).cpu().view(torch.int16)
        assert torch.equal(h, ref), tile


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
def test_gated_float_tiles(dt):
    """The same for float sums, which differ in order and so in the last bits of
    h: both are within half a bf16 ulp (2^-9) of one value but for sums that
    differ by a few 1e-5, hence rel-L2 within 2^-8 of each other."""
    m, d, f = 77, 1152, 256
    cfg = synth.ffn_config(m=m, d=d, f=f)
    w = [dev_bf16(cfg[n]) for n in ("w_gate", "w_up", "w_down")]
    x = dev_bf16(cfg["x"])
    if dt == "bf16":
        layer = w8a8.FfnBF16.from_weights(*w)
        call = lambda: w8a8.bf16_ffn_gate_up(layer, x)
    else:
        layer = w8a8.fp8_ffn_layer(*w, torch.ones(d, device=DEV), torch.ones(f, device=DEV))
        qx, sx = w8a8.fp8_quantize_act(x)
        call = lambda: w8a8.fp8_ffn_gate_up(layer, qx, sx, m)
    force("GLU_TILE", 9)
    ref = call().double()
    for tile in KWAVE_GLU + (RING if dt == "bf16" else RING[-1:]):
        print(dt, "gated tile", tile, flush=True)
        force("GLU_TILE", tile)
        h = call().double()
        assert float((h - ref).norm() / ref.norm()) <= 2.0 ** -8, tile


@pytest.mark.parametrize("m,d,f", [(33, 64, 96), (77, 1152, 6912), (300, 640, 2048), (1021, 1152, 6912)])
def test_bf16_block_packed_activations(m, d, f):
    """h in whole packed fragments (rows past m uninitialised) against h in rows,
    which a workspace of the plain size keeps: one K-wave or ring kernel each way,
    sums in another order, so within a bf16 rounding of h and of the output."""
    print("bf16 block", m, d, f, flush=True)
    cfg = synth.ffn_config(m=m, d=d, f=f)
    layer = w8a8.FfnBF16.from_weights(*(dev_bf16(cfg[n]) for n in ("w_gate", "w_up", "w_down")))
    x = dev_bf16(cfg["x"])
    need, plain = w8a8.bf16_ffn_workspace_bytes(m, d, f), m * f * 2
    assert need >= -(-m // 16) * 16 * f * 2
    y, y_rows = (w8a8.bf16_ffn(layer, x, ws=torch.full((n,), 255, dtype=torch.uint8, device=DEV)).double()
                 for n in (need, (plain + 255) // 256 * 256))
    h = w8a8.bf16_ffn_gate_up(layer, x).double()
    ref = h @ torch.from_numpy(cfg["w_down"].astype(np.uint32) << 16).to(torch.int32).view(torch.float32).to(DEV).double().t()
    for name, got in (("packed", y), ("rows", y_rows)):
        assert float((got - ref).norm() / ref.norm()) <= 2.0 ** -8, name


@pytest.mark.parametrize("m", [33, 100, 300])
def test_stack_down_splits(m):
    """K-wave tiles over parts of K, added by the glue: int8 sums are exact, so the
    stack's logits have the same bits for every tile and split (ragged last splits
    among them)."""
    d, f, v = 208 * 4, 2112, 512
    g = torch.Generator().manual_seed(m)
    rnd = lambda *s: (torch.randn(s, generator=g) * 0.05).bfloat16().to(DEV)
    ws = [(rnd(f, d), rnd(f, d), rnd(d, f)) for _ in range(2)]
    one = lambda n: torch.ones(n, device=DEV)
    head = w8a8.LinearW8A8.from_weight(rnd(v, d), one(d))
    stack = w8a8.Stack([w8a8.FfnW8A8.from_weights(*w, one(d), one(f)) for w in ws],
                       [w8a8.FfnBF16.from_weights(*w) for w in ws], head, None, v)
    x = torch.randn(m, d, generator=g).bfloat16().to(DEV)

    def run(prec):
        buf = torch.full((w8a8.stack_workspace_bytes(m, d, f, v),), 255, dtype=torch.uint8, device=DEV)
        return stack.run(x, np.array(prec, np.uint8), True, ws=buf).double()

    w8a8.set_plan_override("DOWN_TILE", 34)
    w8a8.set_plan_override("DOWN_SPLITS", 1)
    ref = run([1, 1])
    for tile in (None,) + KWAVE:
        for splits in (2, 3, 4):
            print("down splits", m, tile, splits, flush=True)
            w8a8.clear_plan_overrides()
            if tile is not None:
                w8a8.set_plan_override("DOWN_TILE", tile)
                w8a8.set_plan_override("DOWN_SPLITS", splits)
            assert torch.equal(run([1, 1]), ref), (tile, splits)
