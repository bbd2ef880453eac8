"""The wide-tile products (256 x 160, 128 x 160, 128 x 128 and 64 x 128
outputs per workgroup) at the edges of their tiles: ragged token counts, K
split into four to eight pieces, stride 2 and upsampling, tiles over several
images, through pcpp_conv3x3 and pcpp_resnet_block; GEGLU and the products
with residuals through pcpp_transformer_block.  Every case states the plan
that it is meant to run on.  Bounds as for the other convolutions and blocks."""

import numpy as np
import pytest

from paper_2412_02962_amd import synth
from tests import gpu_util as gu
from tests import test_gpu_conv as conv

pytestmark = pytest.mark.gpu

# (H, W, n, i, c_in, c_out, batch, mode) and the plan on 256 compute units
# (tokens and outputs of a tile, pieces of K); the cases on 64 x 64 tiles lie
# next to the line
CASES = [
    ((141, 142, 1, 0, 64, 320, 1, 0), (256, 160, 1)),    # 79 token tiles, the last of 54
    ((40, 50, 1, 0, 1280, 1280, 1, 0), (256, 160, 4)),   # 208 tokens in the last tile
    ((100, 100, 2, 1, 64, 320, 1, 0), (64, 64, 1)),
    ((13, 10, 1, 0, 320, 320, 1, 0), (64, 64, 1)),
    ((64, 64, 1, 0, 64, 640, 1, 0), (64, 64, 1)),
    ((26, 5, 2, 0, 640, 640, 1, 0), (128, 128, 8)),      # pieces of 11 or 12 k-tiles, one ragged tile
    ((6, 3, 1, 0, 640, 640, 3, 0), (128, 128, 8)),       # three images in one tile
    ((26, 10, 1, 0, 320, 320, 2, 1), (64, 64, 1)),
    ((7, 9, 1, 0, 320, 640, 2, 2), (128, 128, 8)),       # upsampling, two images
    ((15, 20, 1, 0, 128, 640, 1, 0), (64, 64, 1)),
    ((141, 26, 1, 0, 64, 320, 3, 0), (128, 160, 1)),     # tiles over two images
    ((13, 10, 1, 0, 640, 320, 1, 0), (128, 160, 8)),     # 2 tokens in the last tile
    ((30, 26, 1, 0, 64, 1280, 3, 0), (128, 128, 1)),
    ((90, 13, 1, 0, 64, 640, 1, 2), (128, 128, 1)),      # upsampling
    ((90, 5, 1, 0, 128, 1280, 3, 0), (64, 128, 1)),      # 6 tokens in the last tile
    ((26, 13, 1, 0, 128, 1280, 1, 2), (64, 128, 1)),
    ((90, 20, 1, 0, 128, 1280, 3, 1), (64, 128, 1)),     # stride 2
    ((90, 100, 1, 0, 64, 640, 3, 1), (128, 160, 1)),
    ((50, 64, 1, 0, 64, 1280, 3, 1), (128, 128, 1)),
    ((2, 10, 1, 0, 640, 320, 2, 1), (128, 160, 8)),      # stride 2, ten tokens
    ((26, 20, 1, 0, 640, 1280, 2, 0), (256, 160, 6)),
]


def _id(c):
    return "x".join(map(str, c))


@pytest.mark.parametrize("case,plan", CASES, ids=_id)
def test_wide_convolution(case, plan):
    from paper_2412_02962_amd import pcpp
    conv._say("wide conv", case, plan)
    assert pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(*case)) == plan
    got, want = conv._run(*case, seed=90 + CASES.index((case, plan)))
    conv._check(got, want, str(case))


# (c_in, c_out, H, W, batch) of ResNets whose tiles cover two images or more
# (each image its own time embedding), and the plans of their convolutions:
# split and not, with the shortcut in bf16 and from a product in float32
RESNETS = [(640, 640, 6, 3, 3, (128, 128, 8), (128, 128, 8)), (320, 640, 7, 9, 2, (128, 128, 8), (128, 128, 8)),
           (64, 320, 141, 26, 3, (128, 160, 1), (128, 160, 1))]


@pytest.mark.parametrize("shape", RESNETS, ids=lambda c: _id(c[:5]))
def test_resnet_tiles_over_images(shape):
    from paper_2412_02962_amd import pcpp
    from tests import test_gpu_resnet as res
    ci, co, H, W, B, plan1, plan2 = shape
    res._say("resnet on wide tiles", shape)
    assert pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(H, W, 1, 0, ci, co, B)) == plan1
    assert pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(H, W, 1, 0, co, co, B)) == plan2
    rc = synth.ResnetConfig("r_wide", H, W, 1, 0, ci, co, temb_dim=64, groups=32, batch=B, seed_id=91)
    inp = synth.resnet_inputs(rc)
    y, e1, e2, _, _ = res._run(rc, {k: gu.to_dev(v, "bf16") for k, v in inp.items()})
    want, w1, w2 = res._oracle(rc, inp)
    res._check(gu.to_f64(y), want, 4, "y")
    res._check(gu.to_f64(e2), w2, 2, "edges2", res._silu_gn_scale(inp, "gn2"), res._h1_rounding_term(rc, inp))


# rows so wide that a tile spans a few of them (3840 px images): (tokens,
# outputs, pieces) with a ragged last tile
@pytest.mark.parametrize("case,plan", [((36, 240, 6, 2, 1920, 640, 1, 0), (128, 128, 4)),
                                       ((27, 480, 9, 1, 960, 320, 1, 0), (128, 160, 8)),
                                       ((10, 480, 5, 4, 1920, 640, 1, 1), (128, 128, 8))],
                         ids=_id)
def test_wide_images(case, plan):
    from paper_2412_02962_amd import pcpp
    conv._say("wide image", case, plan)
    assert pcpp.pcpp_conv3x3_plan(pcpp.make_conv_geom(*case)) == plan
    got, want = conv._run(*case, seed=110)
    conv._check(got, want, str(case))


def test_split_pieces_give_the_same_bits_again():
    """The pieces of a tile are added in order, whichever arrives last."""
    case, _ = CASES[1]
    first, _ = conv._run(*case, seed=91)
    for _ in range(3):
        again, _ = conv._run(*case, seed=91)
        assert np.array_equal(first, again)


@pytest.mark.parametrize("case,plan", [CASES[1], CASES[11], CASES[5], CASES[20]], ids=_id)
def test_pieces_that_give_up_waiting(case, plan):
    """A piece that does not see the others arrive leaves its share of the tile
    to the last of them.  With no look at the arrivals every piece but the last
    gives up at once: the same bits, and the counters back at zero."""
    import ctypes
    import torch
    from paper_2412_02962_amd import pcpp
    H, W, n, i, ci, co, B, mode = case
    conv._say("pieces that give up", case, plan)
    g = pcpp.make_conv_geom(*case)
    assert pcpp.pcpp_conv3x3_plan(g) == plan and plan[2] > 1
    d = {k: gu.to_dev(v, "bf16") for k, v in synth.conv_inputs(H, W, n, i, ci, co, B, 95).items()}
    ptr = lambda t: None if t is None else t.data_ptr()
    wsb = pcpp.pcpp_conv3x3_workspace_size(g)
    ws = torch.full((wsb,), 0x7F, dtype=torch.uint8, device=gu.DEV)
    fn = pcpp.lib().pcpp_internal_conv3x3
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.POINTER(pcpp.pcpp_conv_geom_t)] + [ctypes.c_void_p] * 9 + [ctypes.c_size_t, ctypes.c_int32,
                                                                                   ctypes.c_void_p]
    framed = (B * (H // n + 2) * (W + 2) * ci * 2 + 255) // 256 * 256  # the split region follows, its counters first
    outs = []
    for polls in (-1, 0, 0, 1, -1):
        y = torch.full((B, H // n * W, co), float("nan"), dtype=torch.bfloat16, device=gu.DEV)
        st = fn(ctypes.byref(g), ptr(d["x"]), ptr(d["row_up"]), ptr(d["row_dn"]), ptr(d["w"]), ptr(d["b"]), ptr(y), None,
                None, ptr(ws), wsb, polls, torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        outs.append(y)
        assert not ws[framed:framed + 4 * 4096].view(torch.int32).any()
    assert not torch.isnan(outs[0]).any()
    assert all(torch.equal(outs[0], y) for y in outs[1:])


# (H, W, n, i, heads, ff_inner, batch) and the plan of GEGLU on 256 compute
# units (tokens and outputs of a tile, workgroups on a compute unit): ragged
# bands on every tile
BLOCKS = [
    ((18, 28, 2, 1, 4, 640, 1), (64, 64, 2)), ((10, 13, 1, 0, 5, 320, 3), (64, 64, 2)),
    ((50, 50, 1, 0, 2, 448, 2), (64, 64, 3)), ((40, 64, 2, 0, 10, 2560, 2), (128, 80, 1)),
    ((64, 64, 2, 1, 10, 2560, 2), (256, 80, 1)),
    ((35, 49, 1, 0, 1, 1280, 1), (64, 64, 3)),  # 540 tiles, the last row of them with 51 tokens
    ((25, 20, 1, 0, 8, 2560, 1), (128, 64, 1)), ((41, 45, 1, 0, 5, 1280, 1), (128, 80, 1)),
    ((42, 41, 1, 0, 2, 2560, 1), (256, 80, 1)),
]


@pytest.mark.parametrize("shape,plan", BLOCKS, ids=_id)
def test_block_on_wide_tiles(shape, plan):
    from paper_2412_02962_amd import pcpp
    from tests import test_gpu_block as blk
    H, W, n, i, heads, ff, batch = shape
    bc = synth.BlockConfig("wide", synth.AttnConfig(name="wide", H=H, W=W, n=n, i=i, p=0.5, heads=heads, d=64,
                                                    dtype="bf16", seed_id=0),
                           n_text=9, text_dim=128, ff_inner=ff, gn_groups=32, seed_id=70)
    blk._say("block on wide tiles", shape, plan)
    assert pcpp.pcpp_geglu_plan(pcpp.make_geom(H, W, n, i, 0.5, heads, 64, batch), ff) == plan
    inp = synth.block_inputs(bc, batch=batch)
    y, k, v = blk._run_block(bc, inp, batch)
    want_y, want_k, want_v = blk._oracle_block(bc, inp)
    # stored roundings behind each output, added in quadrature
    # (gu.composition_bound): six for the block, four for K and V (GroupNorm,
    # the stream's LayerNorm and the operands of proj_in and Q/K/V)
    gu.check_composition(gu.to_f64(y), want_y, 6, "y")
    gu.check_composition(gu.to_f64(k), want_k, 4, "k export")
    gu.check_composition(gu.to_f64(v), want_v, 4, "v export")
