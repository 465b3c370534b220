"""Host-only: which kernel a layer's workspace calls take (ftcnn_conv_tile) where the choice once cost time.  Every
case was measured on an MI355X; the time of the route that must not come back, against the one asserted, stands
beside it (protected layer, us)."""
import pytest

import paper_2003_12203_amd as ft

# (n, ch, h, w, m, r, s, stride, pad), tile rows, pixels
SHARED_TILES = [
    ((16, 512, 14, 14, 512, 3, 3, 1, 1), 128, 256),     # 64 x 64 tiles 141, 117
    ((3, 608, 43, 43, 448, 11, 11, 4, 5), 128, 256),    # 64 x 64 tiles 438, 376
    ((9, 352, 74, 74, 320, 11, 11, 4, 5), 128, 256),    # 64 x 64 tiles 1031, 697
    ((32, 512, 14, 14, 512, 3, 3, 1, 1), 128, 256),     # (VGG-19 v14: as before)
    ((1, 512, 7, 7, 512, 3, 3, 1, 1), 64, 64),          # (few outputs: as before)
]


@pytest.mark.parametrize("shape,tm,tp", SHARED_TILES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_shared_tiles_count_the_bytes_they_fetch(shape, tm, tp):
    t = ft.conv_tile(ft.make_desc(*shape, "f32"), 1)
    assert (t["tm"], t["tp"]) == (tm, tp), t
