"""Host-only: which kernel a layer's workspace calls take (ftcnn_conv_tile) where the choice once cost time.  Every
case was measured on an MI355X; the time of the route that must not come back, against the one asserted, stands
beside it (protected layer, us)."""
import pytest

import paper_2003_12203_amd as ft

# (n, ch, h, w, m, r, s, stride, pad), tile rows, pixels
SHARED_TILES = [
    ((16, 512, 14, 14, 512, 3, 3, 1, 1), 128, 128),     # 64 x 64 tiles 141, 116 (128 x 256: 119)
    ((3, 608, 43, 43, 448, 11, 11, 4, 5), 128, 128),    # 64 x 64 tiles 438, 363 (128 x 256: 371)
    ((9, 352, 74, 74, 320, 11, 11, 4, 5), 128, 256),    # 64 x 64 tiles 1031, 697
    ((32, 512, 14, 14, 512, 3, 3, 1, 1), 128, 256),     # (VGG-19 v14: as before)
    ((1, 512, 7, 7, 512, 3, 3, 1, 1), 64, 64),          # (few outputs: as before)
    ((64, 256, 13, 13, 256, 3, 3, 1, 1), 128, 128),     # 128 x 256 106, 92
    ((6, 960, 58, 19, 160, 11, 11, 4, 0), 128, 128),    # two 128 x 256 tiles of 113 parts 354, 258
]


@pytest.mark.parametrize("shape,tm,tp", SHARED_TILES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_shared_tiles_count_the_bytes_they_fetch(shape, tm, tp):
    t = ft.conv_tile(ft.make_desc(*shape, "f32"), 1)
    assert (t["tm"], t["tp"]) == (tm, tp), t


def _loop(shape, dtype, groups=1):
    return ft.conv_tile(ft.make_desc(*shape, dtype, groups=groups), 1)


# padded copies that cost more than they saved: the gather, or in bf16 channels-last copies
NOT_PACKED = [
    ((32, 1, 256, 256, 32, 9, 9, 1, 4), "f32"),       # eight values a column: 632, 301
    ((8, 1, 256, 256, 96, 9, 9, 1, 4), "f32"),        # 316, 154
    ((8, 1, 128, 128, 128, 15, 15, 1, 7), "f32"),     # 252, 123
    ((32, 2, 112, 112, 64, 7, 7, 1, 3), "f32"),       # 133, 103
    ((32, 3, 112, 112, 96, 5, 5, 1, 2), "f32"),       # 142, 108
    ((32, 100, 28, 28, 100, 1, 1, 1, 0), "f32"),      # 30.5, 25.7
    ((46, 87, 85, 85, 144, 1, 1, 1, 0), "f32"),       # 354, 258
    ((32, 1, 256, 256, 32, 9, 9, 1, 4), "bf16"),      # 285, 194
    ((24, 143, 151, 151, 32, 1, 1, 1, 0), "bf16"),    # 228, 140
    ((54, 32, 199, 199, 7, 3, 3, 1, 1), "bf16"),      # 339, 270
    ((36, 288, 80, 80, 144, 1, 1, 1, 0), "bf16"),     # 231, 192
]
# ... and those that pay
STAY_PACKED = [
    ((64, 3, 227, 227, 96, 11, 11, 4, 0), "f32"),     # AlexNet conv1: gather 192, 157
    ((32, 105, 56, 56, 128, 3, 3, 1, 1), "f32"),      # 423, 210
    ((128, 3, 224, 224, 64, 7, 7, 2, 3), "bf16"),     # ResNet-18 stem: 261, 161
    ((64, 160, 28, 28, 320, 1, 1, 1, 0), "bf16"),     # 72, 49
    ((32, 96, 28, 28, 128, 3, 3, 1, 1), "bf16"),      # 41, 30
]


@pytest.mark.parametrize("shape,dtype", NOT_PACKED + STAY_PACKED, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else v)
def test_packed_copies_where_they_pay(shape, dtype):
    assert (_loop(shape, dtype)["loop"] in (5, 6)) == ((shape, dtype) in STAY_PACKED)


def test_loop_test_shapes_run_their_loops():
    """The shapes of test_gpu_direct_to_lds.py run what their lists say."""
    import test_gpu_direct_to_lds as t
    for s in t.SHAPES:
        for dtype in ("f32", "bf16"):
            assert _loop(s, dtype)["loop"] in ((7,) if max(s[5:7]) > 32 else (3, 4)), (s, dtype)
    for s, tiles in t.PACKED.items():
        for dtype, want in zip(("f32", "bf16"), tiles):
            got = _loop(s, dtype)
            assert (got["loop"] in (5, 6)) == (want is not None), (s, dtype, got)
            assert want is None or want == f"{got['tm']}x{got['tp']}", (s, dtype, got)
    for s in t.GATHERED:
        assert _loop(s, "f32")["loop"] < 3 and _loop(s, "bf16")["loop"] < 3 and not _loop(s, "f32")["nhwc"], s
    # every packed tile has a shape
    have = {(d, w) for tiles in t.PACKED.values() for d, w in zip(("f32", "bf16"), tiles) if w}
    assert have == {("f32", w) for w in ("32x128", "64x128", "96x256", "128x128", "64x64")} | \
                   {("bf16", w) for w in ("64x128", "64x256", "128x128", "64x64")}


# fp32 layers of few products an input value: the half larger split copies cost more than the faster products save
NOT_SPLIT = [((17, 320, 86, 86, 6, 1, 1, 1, 0), 1),       # 187, 149
             ((16, 128, 104, 104, 64, 1, 1, 1, 0), 1),    # Darknet-19 c4: 115, 90
             ((11, 992, 80, 50, 16, 1, 1, 1, 0), 2),      # 199, 166
             ((60, 192, 73, 73, 3, 1, 1, 1, 0), 1)]       # 283, 189
SPLIT = [((16, 256, 52, 52, 128, 1, 1, 1, 0), 1),         # Darknet-19 c7: fp32 copies 62, split 56
         ((16, 512, 26, 26, 256, 1, 1, 1, 0), 1),         # 56, 44
         ((32, 256, 56, 56, 256, 3, 3, 1, 1), 1),         # VGG-19 v6: 1010, 640
         ((64, 96, 27, 27, 256, 5, 5, 1, 2), 2)]          # AlexNet conv2: 271, 200


@pytest.mark.parametrize("shape,groups", NOT_SPLIT + SPLIT, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else f"g{v}")
def test_split_copies_where_they_pay(shape, groups):
    t = _loop(shape, "f32", groups)
    assert t["nhwc"] and (t["loop"] in (3, 4)) == ((shape, groups) in SPLIT), t


def test_grouped_tiles_count_both_groups_they_straddle():
    # 192 filters a group: every third tile of 128 walks two groups' channels (AlexNet conv4, 141 us against 134)
    t = _loop((64, 384, 13, 13, 384, 3, 3, 1, 1), "f32", 2)
    assert (t["tm"], t["tp"], t["group_skip"]) == (64, 64, True), t
    t = _loop((64, 384, 13, 13, 256, 3, 3, 1, 1), "f32", 2)   # 128 a group: none straddles
    assert t["tm"] == 128, t
