"""The wide-tile products (256 x 160, 128 x 160, 128 x 128 and 64 x 128
outputs per workgroup) at the edges of their tiles: ragged token counts, K
split into two to eight pieces, stride 2 and upsampling, tiles over several
images, through pcpp_conv3x3; GEGLU and the products with residuals through
pcpp_transformer_block.  Bounds as for the other convolutions and blocks."""

import numpy as np
import pytest

from paper_2412_02962_amd import synth
from tests import gpu_util as gu
from tests import test_gpu_conv as conv

pytestmark = pytest.mark.gpu

# (H, W, n, i, c_in, c_out, batch, mode), and the tile the plan takes on 256
# compute units (tokens x outputs, pieces of K)
CASES = [
    (141, 142, 1, 0, 64, 320, 1, 0),    # 256 x 160, 79 ragged token tiles, unsplit
    (40, 50, 1, 0, 1280, 1280, 1, 0),   # 256 x 160 in 4 pieces, 208 tokens in the last tile
    (100, 100, 2, 1, 64, 320, 1, 0),    # 128 x 160, unsplit
    (13, 10, 1, 0, 320, 320, 1, 0),     # 128 x 160 in 8 pieces, 2 tokens in the last tile
    (64, 64, 1, 0, 64, 640, 1, 0),      # 128 x 128, unsplit
    (26, 5, 2, 0, 640, 640, 1, 0),      # 128 x 128 in 8 pieces of 11 or 12 k-tiles, one ragged tile
    (6, 3, 1, 0, 640, 640, 3, 0),       # three images in one tile
    (26, 10, 1, 0, 320, 320, 2, 1),     # stride 2
    (7, 9, 1, 0, 320, 640, 2, 2),       # upsampling, two images
    (15, 20, 1, 0, 128, 640, 1, 0),     # 64 x 128, 44 tokens in the last tile
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_wide_convolution(case):
    conv._say("wide conv", case)
    got, want = conv._run(*case, seed=90 + CASES.index(case))
    conv._check(got, want, str(case))


# rows so wide that a tile spans a few of them (3840 px images): (tokens,
# outputs, pieces) with a ragged last tile
@pytest.mark.parametrize("case,plan", [((36, 240, 6, 2, 1920, 640, 1, 0), (128, 128, 4)),
                                       ((27, 480, 9, 1, 960, 320, 1, 0), (128, 160, 8)),
                                       ((10, 480, 5, 4, 1920, 640, 1, 1), (128, 128, 8))],
                         ids=lambda c: "x".join(map(str, c)))
def test_wide_images(case, plan):
    from paper_2412_02962_amd import pcpp
    conv._say("wide image", case, plan)
    assert pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(*case)) == plan
    got, want = conv._run(*case, seed=110)
    conv._check(got, want, str(case))


def test_split_pieces_give_the_same_bits_again():
    """The pieces of a tile are added in order, whichever arrives last."""
    case = CASES[1]
    first, _ = conv._run(*case, seed=91)
    for _ in range(3):
        again, _ = conv._run(*case, seed=91)
        assert np.array_equal(first, again)


# (H, W, n, i, heads, ff_inner, batch): ragged bands and feed-forward widths
# that take every tile (outputs per GEGLU tile: 80 or 64)
BLOCKS = [(18, 28, 2, 1, 4, 640, 1), (10, 13, 1, 0, 5, 320, 3), (50, 50, 1, 0, 2, 448, 2), (40, 64, 2, 0, 10, 2560, 2), (64, 64, 2, 1, 10, 2560, 2),
          (35, 49, 1, 0, 1, 1280, 1)]


@pytest.mark.parametrize("shape", BLOCKS, ids=lambda c: "x".join(map(str, c)))
def test_block_on_wide_tiles(shape):
    from tests import test_gpu_block as blk
    H, W, n, i, heads, ff, batch = shape
    bc = synth.BlockConfig("wide", synth.AttnConfig(name="wide", H=H, W=W, n=n, i=i, p=0.5, heads=heads, d=64,
                                                    dtype="bf16", seed_id=0),
                           n_text=9, text_dim=128, ff_inner=ff, gn_groups=32, seed_id=70)
    blk._say("block on wide tiles", shape)
    inp = synth.block_inputs(bc, batch=batch)
    y, k, v = blk._run_block(bc, inp, batch)
    want_y, want_k, want_v = blk._oracle_block(bc, inp)
    # stored roundings behind each output, added in quadrature
    # (gu.composition_bound): six for the block, four for K and V (GroupNorm,
    # the stream's LayerNorm and the operands of proj_in and Q/K/V)
    gu.check_composition(gu.to_f64(y), want_y, 6, "y")
    gu.check_composition(gu.to_f64(k), want_k, 4, "k export")
    gu.check_composition(gu.to_f64(v), want_v, 4, "v export")


def test_geglu_on_three_tiles_a_compute_unit():
    """The last of the blocks above: 540 tiles of 64 x 64, the last row of them with 51 tokens."""
    from paper_2412_02962_amd import pcpp
    H, W, n, i, heads, ff, batch = BLOCKS[-1]
    assert pcpp.pcpp_geglu_plan(pcpp.make_geom(H, W, n, i, 0.5, heads, 64, batch), ff) == (64, 64, 3)
