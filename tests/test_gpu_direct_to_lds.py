"""The direct-to-LDS main loop (conv_kernel.h) at the edges of its tiles and of its ring: one, two
and more chunks of K, ragged filter and pixel tiles, taps outside the map on every side, strides and
non-square kernels, against eq. (1) in float64 on integer data (every sum exact, so bit for bit)."""
import pytest
import torch

import paper_2003_12203_amd as ft

pytestmark = pytest.mark.gpu

# (n, ch, h, w, m, r, s, stride, pad)
SHAPES = [
    (1, 64, 5, 5, 64, 1, 1, 1, 0),       # one chunk, one partial pixel tile
    (2, 128, 9, 7, 65, 1, 1, 1, 0),      # two chunks, a filter past one tile
    (3, 64, 8, 8, 130, 1, 3, 1, 1),      # three chunks
    (2, 64, 11, 13, 96, 3, 3, 2, 1),     # stride, odd map
    (2, 64, 12, 10, 257, 5, 2, 3, 4),    # padding beyond the kernel's reach: whole windows of zeros
    (1, 64, 20, 20, 70, 16, 16, 1, 3),   # the largest kernel of the tap masks
    (1, 64, 24, 24, 70, 17, 3, 1, 3),    # one past it: another loop
    (9, 192, 14, 14, 256, 3, 3, 1, 1),   # several filter and pixel tiles, the last ones ragged
]


def exact_conv(D, W, stride, pad):
    return torch.nn.functional.conv2d(D.double(), W.double(), stride=stride, padding=pad)


@pytest.mark.parametrize("dtype", ["bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_edges_bit_for_bit(shape, dtype):
    print(f"[direct-to-lds] {dtype} {shape}", flush=True)
    n, ch, h, w, m, r, s, u, p = shape
    g = torch.Generator().manual_seed(sum(shape))
    D = torch.randint(0, 4, (n, ch, h, w), generator=g).float()
    # one nonzero tap in eight: bf16 outputs stay below 2^8, exact
    W = torch.randint(-1, 2, (m, ch, r, s), generator=g).float()
    W *= (torch.rand(W.shape, generator=g) < min(1.0, 24.0 / (ch * r * s))).float()
    ref = exact_conv(D, W, u, p)
    assert ref.abs().max() < 256
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    lay = ft.Layer(n, ch, h, w, m, r, s, u, p, dtype)
    Dd, Wd, O = D.to(dt).cuda(), W.to(dt).cuda(), lay.empty_output()
    lay.encode_weights(Wd)
    lay.conv_ws(Dd, Wd, O)
    assert torch.equal(O.double().cpu(), ref)
    O.zero_()
    lay.protected(Dd, Wd, O)
    rep = lay.read_report()
    assert not rep.detected
    assert torch.equal(O.double().cpu(), ref)
