"""The bf16 block gives the same bits with every workspace that it accepts, and
one byte less than the smallest is refused."""

import pytest
import torch

from paper_2608_28003_amd import w8a8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,d,f", [(1, 64, 96), (33, 64, 96), (77, 1152, 6912), (200, 1536, 4608), (257, 1152, 6912),
                                   (300, 640, 2048), (1021, 1152, 6912), (130, 2560, 10240)])
def test_same_bits(m, d, f):
    print("bf16 block workspace", m, d, f, flush=True)
    g = torch.Generator(device=DEV).manual_seed(m + d)
    rnd = lambda *s: (torch.randn(s, generator=g, device=DEV) * 0.05).bfloat16()
    layer = w8a8.FfnBF16.from_weights(rnd(f, d), rnd(f, d), rnd(d, f))
    x = (rnd(m, d) * 20).contiguous()
    need = w8a8.bf16_ffn_workspace_bytes(m, d, f)
    rows = (2 * m * f + 255) // 256 * 256
    call = lambda n: w8a8.bf16_ffn(layer, x, ws=torch.full((n,), 255, dtype=torch.uint8, device=DEV))
    y = call(need)
    ref = w8a8.bf16_ffn_gate_up(layer, x).double() @ layer_down(layer, d, f).t()
    assert float((y.double() - ref).norm() / ref.norm()) <= 2.0 ** -7  # two bf16 roundings
    if need > rows:
        for n in (need - 1, need - 256, rows):
            if n >= rows:
                assert torch.equal(call(n).view(torch.int16), y.view(torch.int16)), n
    with pytest.raises(w8a8.W8A8Error):
        call(rows - 1)


def layer_down(layer, d, f):
    """W_down from its packed form: 16 x 32 fragments, lane l row l % 16, columns 8 (l / 16) .. + 7."""
    p = layer.wp_down.view(torch.bfloat16)[:-(-d // 16) * 16 * f].view(-1, f // 32, 4, 16, 8)
    return p.permute(0, 3, 1, 2, 4).reshape(-1, f)[:d].double()
