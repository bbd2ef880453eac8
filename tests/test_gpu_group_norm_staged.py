"""Transformer modules whose proj_in applies the GroupNorm while staging its
operand (whole 64-token tiles, up to 640 channels, at most two 64 x 64 tiles a
compute unit), and their neighbours past each of these lines, with every
band's statistics as exchanged, against the float64 oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_2412_02962_amd import synth
from tests import gpu_util as gu
from tests import test_gpu_block as blk

pytestmark = pytest.mark.gpu

# (H, W, n, i, heads, groups, text_dim, batch)
CASES = [
    (8, 16, 2, 1, 1, 32, 64, 1),      # one token tile, one k-tile, two channels a group
    (8, 16, 2, 0, 1, 1, 64, 3),       # three images, one group
    (24, 16, 3, 1, 5, 64, 128, 2),    # two token tiles an image, five k-tiles
    (12, 32, 2, 1, 10, 32, 2048, 1),  # 640 channels, beside a text product of 32 k-tiles
    (12, 32, 2, 1, 10, 128, 96, 2),   # text_dim no multiple of 64: proj_in in a launch of its own
    (8, 17, 2, 0, 2, 32, 64, 1),      # 68 tokens: not staged
    (8, 16, 2, 0, 11, 32, 64, 1),     # 704 channels: not staged
    (64, 51, 1, 0, 10, 32, 64, 1),    # 510 tiles on 256 compute units: staged
    (64, 52, 1, 0, 10, 32, 64, 1),    # 520: not staged
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_module_around_staging(case):
    H, W, n, i, heads, groups, text_dim, batch = case
    blk._say("module around GroupNorm staging", case)
    attn = synth.AttnConfig(name="staged", H=H, W=W, n=n, i=i, p=0.25, heads=heads, d=64, dtype="bf16", seed_id=83)
    bc = synth.BlockConfig("staged", attn, n_text=5, text_dim=text_dim, ff_inner=128, gn_groups=groups, seed_id=83)
    x, text, module, blocks, stale = synth.module_inputs(bc, 1, batch=batch)
    rng = np.random.default_rng(9)
    st = np.stack([oracle.group_stats(0.3 * rng.standard_normal() + rng.standard_normal((batch, attn.h * W, attn.C)),
                                      groups) for _ in range(n)])
    bands = torch.from_numpy(st.astype(np.float32)).to(gu.DEV)
    y, ko, vo, own = blk._run_module(bc, x, text, module, blocks, stale, batch, gn_bands=bands, want_own=True)
    want_y, want_k, want_v = blk._oracle_module(bc, x, text, module, blocks, stale, gn_band_stats=st)
    blk._check_module(bc, 1, y, ko, vo, want_y, want_k, want_v)
    want_own = oracle.group_stats(oracle.from_bf16_bits(x), groups)
    got_own = own.double().cpu().numpy()
    assert np.array_equal(got_own[..., 0], want_own[..., 0])
    # float32 sums of values of order 1: the mean to 1e-5, M2 to 1e-4 of itself
    assert np.allclose(got_own[..., 1], want_own[..., 1], rtol=0, atol=1e-5)
    assert np.allclose(got_own[..., 2], want_own[..., 2], rtol=1e-4, atol=0)
