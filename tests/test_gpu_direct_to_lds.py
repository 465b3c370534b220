"""The direct-to-LDS main loop (conv_kernel.h), bf16 and fp32 on split copies, at the edges of its
tiles and of its ring: one, two and more chunks of K, ragged filter and pixel tiles, taps outside the
map on every side, strides and non-square kernels, against eq. (1) in float64 on integer data (every
sum exact, so bit for bit); and what the split must not change: 24-bit operands, the error of long
sums, and infinite, NaN and overflowing operands."""
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
    (1, 64, 20, 20, 70, 16, 16, 1, 3),   # large kernels
    (1, 64, 24, 24, 70, 17, 3, 1, 3),
    (1, 64, 40, 33, 40, 32, 3, 1, 9),    # the largest kernel of the tap masks
    (2, 64, 9, 40, 66, 3, 37, 2, 18),    # past them: wider than the map, few and many filters
    (1, 64, 70, 66, 64, 33, 33, 1, 20),
    (2, 128, 50, 7, 130, 48, 1, 1, 11),
    (1, 64, 1, 70000, 64, 1, 9, 3, 4),   # a map wider than 16 bits
    (9, 192, 14, 14, 256, 3, 3, 1, 1),   # several filter and pixel tiles, the last ones ragged
]
# enough outputs for the larger tiles, the last ones ragged both ways
SHAPES += [(5, 64, 50, 51, 130, 3, 3, 1, 1), (5, 64, 50, 51, 130, 2, 2, 1, 0), (11, 64, 50, 51, 150, 1, 2, 1, 0),
           (10, 64, 50, 50, 257, 1, 3, 1, 0), (14, 64, 50, 51, 61, 1, 3, 1, 1)]
# the tiles of few filters, and one of few outputs and many chunks (shared by stream-K workgroups)
FEW_FILTERS = [(2, 32, 9, 9, 31, 3, 3, 1, 1), (4, 96, 30, 31, 33, 3, 3, 1, 1), (1, 512, 7, 7, 512, 3, 3, 1, 1)]
# 1x1 layers that one type has on the loop (fp32: few products an input value, fp32 copies), and a packed one in bf16
OTHERS = [(5, 64, 50, 51, 130, 1, 1, 1, 0), (10, 64, 50, 50, 257, 1, 1, 1, 0), (31, 96, 50, 51, 130, 3, 1, 1, 1)]
# packed copies, with the tiles of fp32 and bf16: stems (a kernel row a tap; four or eight channels a column by the
# stride; padding past the kernel), channels that fill no block of eight, kernels up to the largest, units that end
# inside a chunk, ragged tiles of every kind (None: fp32 gathers)
PACKED = {
    (16, 3, 43, 40, 64, 9, 9, 2, 4): ("64x128", "64x128"),
    (6, 3, 61, 60, 96, 11, 11, 4, 0): ("64x64", "64x64"),
    (2, 3, 43, 40, 96, 11, 11, 4, 0): ("64x64", "64x64"),
    (24, 20, 53, 53, 90, 3, 3, 1, 1): ("96x256", "128x128"),
    (11, 3, 224, 222, 61, 7, 7, 2, 3): (None, "64x256"),
    (16, 6, 41, 40, 65, 7, 7, 2, 3): ("64x64", "64x64"),
    (8, 8, 40, 40, 64, 7, 7, 2, 3): ("64x128", "64x128"),
    (8, 2, 60, 60, 96, 15, 15, 2, 7): ("64x64", "64x64"),
    (8, 1, 80, 80, 70, 9, 9, 4, 6): (None, "64x64"),
    (16, 6, 31, 32, 33, 7, 5, 3, 2): ("64x128", "64x128"),
    (16, 3, 60, 61, 40, 5, 5, 1, 2): (None, "64x128"),
    (2, 17, 29, 28, 100, 3, 3, 1, 1): ("64x64", "64x64"),
    (3, 100, 25, 26, 70, 3, 3, 2, 1): ("64x64", "64x64"),
    (6, 105, 22, 23, 200, 1, 1, 1, 0): (None, "64x64"),
    (2, 9, 20, 20, 64, 15, 15, 1, 7): ("64x128", "64x128"),
    (8, 40, 17, 19, 300, 2, 3, 1, 1): ("64x64", "64x64"),
    (16, 40, 17, 19, 300, 2, 3, 1, 1): ("128x128", "64x64"),
    (4, 65, 24, 24, 31, 3, 3, 1, 1): ("32x128", "64x128"),
    (16, 12, 40, 41, 60, 5, 4, 1, 2): ("64x128", "64x128"),
    (24, 105, 30, 30, 130, 3, 3, 1, 1): ("128x128", "128x128"),
}
# short sums, small layers and kernels past 15 rows stay on the gather
GATHERED = [(2, 3, 40, 41, 40, 7, 7, 2, 3), (3, 3, 40, 41, 130, 3, 3, 1, 1), (4, 5, 30, 31, 33, 5, 3, 3, 2),
            (4, 8, 30, 31, 65, 3, 3, 2, 1), (8, 1, 40, 40, 70, 5, 5, 1, 6), (16, 3, 97, 97, 96, 3, 3, 1, 0),
            (1, 65, 24, 24, 65, 16, 3, 1, 3)]


def exact_conv(D, W, stride, pad):
    return torch.nn.functional.conv2d(D.double(), W.double(), stride=stride, padding=pad)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES + FEW_FILTERS + OTHERS + list(PACKED) + GATHERED, ids=lambda s: "-".join(map(str, s)))
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


def run_f32(D, W, u=1, p=1, scale=None):
    n, ch, h, w = D.shape
    m, _, r, s = W.shape
    lay = ft.Layer(n, ch, h, w, m, r, s, u, p, "f32")
    O = lay.empty_output()
    lay.conv_ws(D.cuda(), W.cuda(), O)
    return O.cpu()


def test_split_holds_every_bit():
    # products of 24-bit values by powers of two, one a filter: exact only if all three planes are whole
    g = torch.Generator().manual_seed(5)
    D = (torch.randint(1 << 23, 1 << 24, (2, 32, 6, 6), generator=g).float()
         * torch.where(torch.rand(2, 32, 6, 6, generator=g) < 0.5, -1.0, 1.0))
    W = torch.zeros(64, 32, 1, 1)
    for m in range(64):
        W[m, m % 32] = 2.0 ** (m // 32 - 3)
    ref = exact_conv(D, W, 1, 0)
    assert torch.equal(run_f32(D, W, p=0).double(), ref)
    Wm = torch.randint(1 << 23, 1 << 24, (64, 32, 1, 1), generator=g).float() * (W != 0)
    one = torch.zeros_like(D)
    one[:, :, 2, 3] = 4.0
    assert torch.equal(run_f32(one, Wm, p=0).double(), exact_conv(one, Wm, 1, 0))


def test_split_error_is_an_fp32_sum_s():
    # fp32 accumulation of K terms in any order: below 2^-24 K of the sum of magnitudes, and far below
    # it in the mean (2^-24 sqrt(K) of the root sum of squares); So5 must not add the errors up
    g = torch.Generator().manual_seed(6)
    n, ch, hw, m = 8, 256, 14, 128
    D, W = torch.rand(n, ch, hw, hw, generator=g), torch.randn(m, ch, 3, 3, generator=g) * 0.03
    ref = exact_conv(D, W, 1, 1)
    O = run_f32(D, W).double()
    mag = exact_conv(D, W.abs(), 1, 1)
    assert ((O - ref).abs() <= 2.0 ** -24 * ch * 9 * mag).all()
    rel = ((O - ref).norm() / ref.norm()).item()
    assert rel <= 2.0 ** -24 * (ch * 9) ** 0.5, rel
    bias = (O - ref).sum((0, 1)).norm() / ((O - ref).norm() * (n * m) ** 0.5)
    # independent errors give about (n m)^-1/2 = 0.03; errors of one sign 1
    assert bias < 0.25, bias


# long sums of few and of many filters, the first AlexNet layer, 1x1, packed channels
ERROR_SHAPES = [(8, 512, 14, 14, 1, 3, 3, 1, 1), (8, 256, 14, 14, 128, 3, 3, 1, 1), (4, 3, 115, 115, 96, 11, 11, 4, 0),
                (4, 512, 26, 26, 64, 1, 1, 1, 0), (4, 105, 28, 28, 128, 3, 3, 1, 1)]


@pytest.mark.parametrize("weights", ["random", "positive", "one parity"])
@pytest.mark.parametrize("shape", ERROR_SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_split_is_no_further_from_float64_than_fp32_instructions(shape, weights):
    n, ch, h, w, m, r, s, u, p = shape
    g = torch.Generator().manual_seed(11)
    D, W = torch.rand(n, ch, h, w, generator=g), torch.randn(m, ch, r, s, generator=g) * 0.03
    if weights == "positive":
        W = W.abs()
    if weights == "one parity":
        W[1::2] = 0
    lay = ft.Layer(*shape, "f32")
    assert ft.conv_tile(lay.desc, 1)["loop"] >= 3 and ft.conv_tile(lay.desc, 0)["loop"] < 3
    Dd, Wd, O, O32 = D.cuda(), W.cuda(), lay.empty_output(), lay.empty_output()
    lay.encode_weights(Wd)
    lay.protected(Dd, Wd, O)
    lay.conv(Dd, Wd, O32)
    ref = exact_conv(D, W, u, p)
    err, err32 = O.double().cpu() - ref, O32.double().cpu() - ref
    assert err.norm() <= err32.norm(), (err.norm(), err32.norm())
    # the errors of the outputs that are not zero must not lean to one side: their mean is that of
    # independent ones, below 6 deviations of rms / sqrt(count)
    live = err[:, ::2] if weights == "one parity" else err
    lean = (live.mean().abs() / live.square().mean().sqrt() * live.numel() ** 0.5).item()
    assert lean < 6, lean


def test_split_zeros_are_positive():
    # as the fp32 instructions give them: the sign of a filter's copy must not reach its outputs
    for ch, k in ((64, 3), (40, 3)):
        lay = ft.Layer(8, ch, 30, 30, 64, k, k, 1, k // 2, "f32")
        assert ft.conv_tile(lay.desc, 1)["loop"] >= 3
        D, W, O = torch.zeros(8, ch, 30, 30).cuda(), torch.ones(64, ch, k, k).cuda(), lay.empty_output()
        lay.conv_ws(D, W, O)
        assert not torch.signbit(O).any()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(6, 3, 61, 60, 96, 11, 11, 4, 0), (16, 3, 43, 40, 64, 9, 9, 2, 4), (8, 40, 17, 19, 300, 2, 3, 1, 1)],
                         ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_packed_padding_meets_no_infinite_value(value, shape, dtype):
    # a run of a kernel row reads on past its last column (stems: to the twelfth of eleven, the tenth of nine),
    # against zero weights
    n, ch, h, w, m, r, s, u, p = shape
    g = torch.Generator().manual_seed(10)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    D, W = torch.rand(n, ch, h, w, generator=g) + 0.5, torch.rand(m, ch, r, s, generator=g) + 0.1
    D[1, 2, 10, 11 - p] = value   # just past the first output's run
    D[0, 0, 0, w - 1] = value
    lay = ft.Layer(*shape, dtype)
    assert ft.conv_tile(lay.desc, 1)["loop"] in (5, 6)
    O = lay.empty_output()
    lay.conv_ws(D.to(dt).cuda(), W.to(dt).cuda(), O)
    ref = torch.nn.functional.conv2d(torch.nn.functional.pad(D, (p,) * 4), W, stride=u)
    assert torch.equal(torch.isfinite(O.cpu()), torch.isfinite(ref))
    assert torch.equal(torch.isnan(O.cpu()), torch.isnan(ref))


@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan"), 3.4028234e38])
@pytest.mark.parametrize("where", ["D", "W", "both"])
def test_nonfinite_operands_give_what_fp32_gives(value, where):
    g = torch.Generator().manual_seed(7)
    D, W = torch.rand(2, 64, 9, 9, generator=g) + 0.5, torch.randn(96, 64, 3, 3, generator=g)
    W = torch.where(W.abs() < 0.1, torch.full_like(W, 0.1), W)
    if where in ("D", "both"):
        D[1, 5, 4, 4] = value
        D[0, 63, 0, 0] = value
    if where in ("W", "both"):
        W[17, 40, 1, 1] = value
        if abs(value) < float("inf") and where == "both":
            W[17, 5] = W[17, 63] = 0.1   # overflow of both signs in one sum would depend on its order
    ref = torch.nn.functional.conv2d(D, W, padding=1)
    O = run_f32(D, W)
    assert torch.equal(torch.isnan(O), torch.isnan(ref))
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(O), inf) and torch.equal(O[inf], ref[inf])
    ok = torch.isfinite(ref)
    assert ok.any()
    torch.testing.assert_close(O[ok], ref[ok], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("ch,k,dtype", [(64, 3, "f32"), (64, 3, "bf16"), (40, 3, "f32"), (8, 7, "f32"), (8, 7, "bf16"), (40, 3, "bf16")])
def test_nonfinite_weight_meets_the_padding(ch, k, dtype, value):
    # zero padding is zeros that the filter multiplies: an infinite tap gives NaN there, as the gather does
    g = torch.Generator().manual_seed(12)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    D, W = torch.rand(4, ch, 30, 30, generator=g) + 0.5, torch.rand(96, ch, k, k, generator=g) + 0.1
    W[17, 1, 0, 0] = value
    W[18, 2, k - 1, 1] = value
    lay = ft.Layer(4, ch, 30, 30, 96, k, k, 1, k // 2, dtype)
    assert ft.conv_tile(lay.desc, 1)["loop"] >= 3 and ft.conv_tile(lay.desc, 0)["loop"] < 3
    Dd, Wd, O, Og = D.to(dt).cuda(), W.to(dt).cuda(), lay.empty_output(), lay.empty_output()
    lay.conv_ws(Dd, Wd, O)
    lay.conv(Dd, Wd, Og)
    ref = torch.nn.functional.conv2d(torch.nn.functional.pad(D, (k // 2,) * 4), W)
    for got in (O.cpu(), Og.cpu()):
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))


def test_nonfinite_operands_stay_inside_their_group():
    # two groups of 48 channels: the middle block of 32 channels holds both groups'
    g = torch.Generator().manual_seed(8)
    D, W = torch.rand(1, 96, 5, 5, generator=g) + 0.5, torch.rand(64, 48, 3, 3, generator=g) + 0.1
    D[0, 40, 2, 2] = float("inf")
    lay = ft.Layer(1, 96, 5, 5, 64, 3, 3, 1, 1, "f32", groups=2)
    O = lay.empty_output()
    lay.conv_ws(D.cuda(), W.cuda(), O)
    ref = torch.nn.functional.conv2d(D, W, padding=1, groups=2)
    assert torch.equal(torch.isinf(O.cpu()), torch.isinf(ref)) and not torch.isnan(O).any()


# (shape, groups): ragged tiles of several waves, groups that share a block of filters, strides, packed
# stems and channels, sums that end inside a step of the redo (bf16: on packed copies)
REDO_SHAPES = [((3, 64, 19, 21, 150, 3, 3, 1, 1), 1), ((2, 96, 20, 20, 48, 3, 3, 1, 1), 4), ((9, 192, 14, 14, 256, 3, 3, 2, 1), 1),
               ((4, 32, 45, 45, 33, 5, 2, 2, 3), 1), ((16, 6, 41, 40, 65, 7, 7, 2, 3), 1), ((6, 105, 22, 23, 200, 3, 3, 1, 1), 1),
               ((4, 3, 60, 60, 96, 11, 11, 4, 0), 1), ((4, 42, 24, 24, 60, 3, 3, 1, 1), 2)]


REDO_CASES = [(s, g, d) for s, g in REDO_SHAPES for d in ("f32", "bf16") if d == "f32" or s[1] % 64 and not (s[1] % 32 == 0 and g > 1)]


@pytest.mark.parametrize("shape,groups,dtype", REDO_CASES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_redone_outputs(shape, groups, dtype):
    # beside infinities and NaN, values whose outputs are finite but past the split copies' scale
    n, ch, h, w, m, r, s, u, p = shape
    g = torch.Generator().manual_seed(13)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    D, W = torch.rand(n, ch, h, w, generator=g) + 0.5, torch.rand(m, ch // groups, r, s, generator=g) + 0.1
    D[0] *= 2.0 ** 104
    D[n - 1, ch - 1, h - 1, w - 1] = float("inf")
    D[n - 1, 0, 0, 0] = float("nan")
    W[m - 1, 0, r // 2, s // 2] = -float("inf")
    D, W = D.to(dt).float(), W.to(dt).float()
    lay = ft.Layer(*shape, dtype, groups=groups)
    assert ft.conv_tile(lay.desc, 1)["loop"] >= 3, ft.conv_tile(lay.desc, 1)
    O = lay.empty_output()
    lay.conv_ws(D.to(dt).cuda(), W.to(dt).cuda(), O)
    Dp = torch.nn.functional.pad(D, (p,) * 4).double()
    ref = torch.nn.functional.conv2d(Dp, W.double(), stride=u, groups=groups)
    got = O.double().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isinf(got), torch.isinf(ref)) and torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    # positive terms: an fp32 sum of them is within 2^-24 of itself a term; bf16 outputs round once more
    K = ch // groups * r * s
    torch.testing.assert_close(got[ok], ref[ok], rtol=2.0 ** -24 * K + (2.0 ** -8 if dtype == "bf16" else 0.0), atol=0.0)


def test_one_large_value_costs_a_few_blocks():
    # 9 x 256 outputs are redone, all in few tiles: one lane an output took 110 times the clean layer here
    lay = ft.Layer(4, 256, 28, 28, 256, 3, 3, 1, 1, "f32")
    g = torch.Generator().manual_seed(14)
    D, W, O = torch.rand(4, 256, 28, 28, generator=g).cuda(), torch.randn(256, 256, 3, 3, generator=g).cuda(), lay.empty_output()

    def best():
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ts = []
        for _ in range(6):
            e0.record()
            lay.conv_ws(D, W, O)
            e1.record()
            e1.synchronize()
            ts.append(e0.elapsed_time(e1))
        return min(ts)

    clean = best()
    D[1, 2, 10, 10] = 3e38
    assert best() < 20 * clean


@pytest.mark.parametrize("d_exp,w_exp", [(-125, 0), (0, -125), (-140, 0), (-70, -60), (100, 0), (60, 30), (0, 100)])
def test_split_over_the_range_of_fp32(d_exp, w_exp):
    # operands down to subnormal numbers and up to where their sums still fit
    g = torch.Generator().manual_seed(9)
    D = torch.rand(2, 64, 9, 9, generator=g) * 2.0 ** d_exp
    W = torch.randn(64, 64, 3, 3, generator=g) * 0.05
    W = W * 2.0 ** w_exp if w_exp > -126 else W
    ref = exact_conv(D, W, 1, 1)
    O = run_f32(D, W).double()
    # an fp32 sum's error, and half of the smallest subnormal for its rounding
    bound = 2.0 ** -24 * 576 * exact_conv(D.abs(), W.abs(), 1, 1) + 2.0 ** -149
    assert ((O - ref).abs() <= bound).all()
    if ref.abs().max() > 1e-30:
        assert (O - ref).norm() <= 2.0 ** -24 * 24 * ref.norm()
