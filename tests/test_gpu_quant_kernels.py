"""The tiled weight quantiser, the wide column maximum and the many-row E4M3
quantiser at the edges of their launch rules, bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_2608_28003_amd import synth, w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to(DEV)
    return torch.from_numpy(a).to(DEV)


# 16, 8 and 4 rows a workgroup (by length, then by row count), ragged rows and
# columns, one unit, the longest rows of the kernel and the first past it
@pytest.mark.parametrize("n,k", [(8197, 1168), (4099, 2560), (8200, 1552), (37, 1152), (5, 16), (50, 12288),
                                 (20, 12304)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_weight_codes(n, k, dtype):
    print("weights", n, k, dtype, flush=True)
    rng = np.random.default_rng(n + k)
    w = (rng.standard_normal((n, k)) * 0.02).astype(np.float32)
    w[0] = 0.0
    w[1] *= np.float32(1e-37)  # subnormal products and scales
    w[2] *= np.float32(1e30)
    w[3, 1:] *= np.float32(1e-38)  # tiny values under an ordinary maximum
    if dtype == "bf16":
        w = synth.to_bf16_bits(w)
    for delta in (None, np.exp(rng.uniform(-2, 2, k)).astype(np.float32)):
        d = None if delta is None else dev(delta)
        for ref, got in ((oracle.quantize_weights, w8a8.quantize_weights),
                         (oracle.quantize_weights_fp8, w8a8.fp8_quantize_weights)):
            q_o, s_o = ref(w, delta)
            wq, s = got(dev(w), d)
            full = w8a8.frag_to_rowmajor(wq.cpu().numpy(), -(-n // 16) * 16, -(-k // 64) * 64)
            np.testing.assert_array_equal(s.cpu().numpy(), s_o)
            np.testing.assert_array_equal(full[:n, :k].view(q_o.dtype), q_o)
            assert not full[n:].any() and not full[:, k:].any()


@pytest.mark.parametrize("rows,k", [(1, 8), (13, 16), (1000, 1152), (25000, 1160), (300, 2056), (77, 6912), (50, 1001)])
def test_col_absmax(rows, k):
    print("col_absmax", rows, k, flush=True)
    rng = np.random.default_rng(rows + k)
    x = rng.standard_normal((rows, k)).astype(np.float32)
    x[rng.integers(0, rows, 5), rng.integers(0, k, 5)] = np.float32([np.nan, np.inf, -np.inf, 3e38, -1e-40])
    start = np.abs(rng.standard_normal(k)).astype(np.float32) * 2
    for a in (x, synth.to_bf16_bits(x)):
        got = w8a8.col_absmax(dev(a), dev(start)).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.col_absmax(a, start))


@pytest.mark.parametrize("m,k,r", [(257, 1152, 2), (320, 6912, 4), (300, 2048, 1)])
def test_fp8_many_rows(m, k, r):
    """Rows on both sides of 2^-107, where the IEEE divisions take over."""
    print("fp8 act", m, k, r, flush=True)
    rng = np.random.default_rng(m)
    delta = np.exp2(rng.uniform(20, 40, k)).astype(np.float32)
    target = rng.standard_normal((m, k))
    target[0::4] = np.exp2(rng.uniform(-150, -108, (len(target[0::4]), k)))
    target[1::4] = np.exp2(rng.uniform(-160, -127, (len(target[1::4]), k)))
    target[1::4, 7] = 2.0 ** -107 * (1 + 2.0 ** -6)
    target[2::8] = np.exp2(rng.uniform(-130, -107.5, (len(target[2::8]), k)))
    target[2::8, 3] = 2.0 ** -107 * (1 - 2.0 ** -6)
    sign = np.where(rng.random((m, k)) < 0.5, -1.0, 1.0)
    x = synth.to_bf16_bits((sign * target * delta).astype(np.float32))
    x[4] = 0
    q_o, s_o = oracle.quantize_act_fp8(x, delta)
    w8a8.set_plan_override("QROWS_R", r)
    qx, s = w8a8.fp8_quantize_act(dev(x), dev(delta))
    got = w8a8.frag_to_rowmajor(qx.cpu().numpy(), m, k).view(np.uint8)
    np.testing.assert_array_equal(s.cpu().numpy(), s_o)
    np.testing.assert_array_equal(got, q_o)


# both sides of the row counts from which the tiles and the many-row kernel are taken
@pytest.mark.parametrize("n,k", [(496, 1152), (512, 1168), (300, 448), (300, 512), (515, 12288), (600, 6912)])
def test_weight_codes_rule(n, k):
    test_weight_codes(n, k, "bf16")


@pytest.mark.parametrize("m,k", [(1264, 640), (1265, 640), (272, 1920), (257, 2048), (40, 10240), (257, 10240)])
def test_fp8_act_rule(m, k):
    print("fp8 act rule", m, k, flush=True)
    rng = np.random.default_rng(m + k)
    x = synth.to_bf16_bits(rng.standard_normal((m, k)).astype(np.float32))
    delta = np.exp(rng.uniform(-2, 2, k)).astype(np.float32)
    q_o, s_o = oracle.quantize_act_fp8(x, delta)
    qx, s = w8a8.fp8_quantize_act(dev(x), dev(delta))
    np.testing.assert_array_equal(s.cpu().numpy(), s_o)
    np.testing.assert_array_equal(w8a8.frag_to_rowmajor(qx.cpu().numpy(), m, k).view(np.uint8), q_o)


@pytest.mark.parametrize("rows,k", [(4, 1152), (5, 1152), (4, 8), (5, 10240)])
def test_col_absmax_rule(rows, k):
    test_col_absmax(rows, k)
