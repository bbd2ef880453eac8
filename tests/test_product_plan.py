"""Plans of the convolutions' products (pcpp_conv3x3_plan; host only): which
tile a size takes, and that no tile reaches further than the 32-bit offsets
its kernel addresses X with."""

import numpy as np
import pytest

from paper_2412_02962_amd import pcpp


def _plan(H, W, n, i, c_in, c_out, batch=1, mode=0, cus=256, enabled=256):
    return pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(H, W, n, i, c_in, c_out, batch, mode), cus, enabled)


# 3840 px images: the level-0 960 -> 320 and level-1 1920 -> 640 ResNets'
# first convolutions, whole images and low ones; wider images and larger
# channel counts; stride 2 and upsampling
@pytest.mark.parametrize("geo", [(480, 480, 8, 3, 960, 320), (480, 472, 8, 3, 960, 320), (240, 240, 4, 1, 1920, 640),
                                 (240, 240, 8, 0, 1920, 640, 2), (48, 240, 8, 2, 1920, 640), (768, 768, 8, 1, 640, 320),
                                 (384, 384, 8, 1, 2560, 1280), (960, 960, 8, 1, 320, 320, 1, 1),
                                 (240, 480, 4, 1, 1280, 640, 1, 2)])
def test_wide_images_take_wide_tiles(geo):
    tokens, outputs, pieces = _plan(*geo)
    assert tokens * outputs >= 128 * 128 or pieces > 1, (geo, tokens, outputs, pieces)


def _span(H, W, n, c_in, batch, mode, tile_tokens):
    """Largest distance in bytes between the first and any other row of X of one tile."""
    u, st = (2 if mode == 2 else 1), (2 if mode == 1 else 1)
    Hf, Wf = H // n * u, W * u
    b, y, x = np.meshgrid(np.arange(batch), np.arange(Hf // st), np.arange(Wf // st), indexing="ij")
    off = (((b * (Hf + 2) + st * y) * (Wf + 2) + st * x).astype(np.int64) * c_in * 2).reshape(-1)
    first = off[np.arange(off.size) // tile_tokens * tile_tokens]
    return int((off - first).max())


def test_no_tile_reaches_past_32_bits():
    rng = np.random.default_rng(5)
    geos = [(2, 200000, 1, 0, 64, 640, 1, 0), (2, 200000, 1, 0, 2560, 1280, 1, 0), (2, 104000, 1, 0, 2560, 640, 1, 0),
            (2, 110000, 1, 0, 2560, 640, 1, 0), (4, 90000, 1, 0, 2560, 640, 1, 1), (1, 1, 1, 0, 2560, 1280, 4000, 0),
            (2, 2, 1, 0, 2560, 1280, 4000, 1), (600, 1, 1, 0, 2560, 1280, 1, 0), (2, 3, 1, 0, 1920, 640, 900, 2)]
    for _ in range(60):
        W = int(np.exp(rng.uniform(0, np.log(4000))))
        geos.append((2 * int(np.exp(rng.uniform(0, np.log(64)))), 2 * W, 1, 0, 64 * int(rng.integers(1, 41)),
                     int(rng.choice([320, 640, 1280])), int(rng.integers(1, 4)), int(rng.integers(0, 3))))
    wide = 0
    for geo in geos:
        H, W, n, i, c_in, c_out, batch, mode = geo
        tokens, outputs, pieces = _plan(*geo)
        if (tokens, outputs) != (64, 64):
            wide += 1
            assert _span(H, W, n, c_in, batch, mode, tokens) < 2 ** 31, (geo, tokens, outputs, pieces)
    assert wide >= 30


def test_k_is_split_only_on_whole_unmasked_xcds():
    geo = (48, 240, 8, 2, 1920, 640)
    assert _plan(*geo)[2] > 1
    for cus, enabled in ((256, 255), (250, 250), (80, 80)):
        assert _plan(*geo, cus=cus, enabled=enabled)[2] == 1
    with pytest.raises(pcpp.PcppError):
        _plan(*geo, cus=-1)
    with pytest.raises(pcpp.PcppError):
        _plan(48, 240, 8, 2, 1920, 65)


def _geglu(tokens, heads, ff=None, cus=256, enabled=256):
    return pcpp.pcpp_geglu_plan(pcpp.make_geom(1, tokens, 1, 0, 0.0, heads), ff or 256 * heads, cus, enabled)


def test_geglu_tiles():
    """Three 64 x 64 tiles to a compute unit where K is short and the tiles
    come to several rounds; the largest ones for long K and many tokens."""
    for tokens, heads in ((2072, 5), (8219, 4), (23864, 8), (1157, 8), (11610, 1), (546, 16)):
        assert _geglu(tokens, heads) == (64, 64, 3), (tokens, heads)
    assert _geglu(65, 1) == (64, 64, 2)
    assert _geglu(2048, 10) == _geglu(1024, 20) == _geglu(12639, 20) == (256, 80, 1)
    assert _geglu(512, 20) == _geglu(504, 20) == (128, 80, 1)
    assert _geglu(500, 8, 2560) == (128, 64, 1)
    assert _geglu(2048, 10, 2496)[1] == 64  # 2496 = 39 x 64
    with pytest.raises(pcpp.PcppError):
        _geglu(64, 5, 100)
