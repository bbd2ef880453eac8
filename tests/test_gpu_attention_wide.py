"""bf16 attention in blocks of 256 queries (four wavefronts of two blocks of
32), which launches with many blocks take: its tile edges, its split over
pieces of the keys and its late rescale, against the float64 oracle."""

import numpy as np
import pytest

from paper_2412_02962_amd import synth
from tests import gpu_util as gu
from tests.test_gpu_attention import _monotone_score_inputs

pytestmark = pytest.mark.gpu


def _check(geo, pieces, inputs):
    from paper_2412_02962_amd import pcpp
    H, W, n, i, p, heads, batch = geo
    cfg = synth.AttnConfig(name="wide", H=H, W=W, n=n, i=i, p=p, heads=heads, d=64, dtype=synth.DTYPE_BF16, seed_id=91,
                           batch=batch)
    assert pcpp.pcpp_partial_attention_plan(gu.geom(cfg))[:2] == (256, pieces)
    print("[case]", geo, flush=True)
    inp = inputs(cfg)
    got = gu.to_f64(gu.run_attention(cfg, inp))
    gu.assert_close(cfg, got, gu.oracle_attention(cfg, inp).reshape(got.shape), str(geo))


# whole blocks: one query past 128, a full block, one past it (a second block
# of one query), sources that end inside a tile; three pieces: 12 or 13 of 38
# tiles, six blocks of which the last has 220 queries
@pytest.mark.parametrize("geo,pieces", [((1, 129, 1, 0, 0.0, 20, 16), 1), ((16, 16, 1, 0, 0.0, 20, 16), 1),
                                        ((1, 257, 1, 0, 0.0, 20, 20), 1), ((30, 25, 3, 1, 0.5, 20, 16), 1),
                                        ((30, 25, 3, 0, 0.26, 20, 17), 1), ((90, 50, 3, 1, 0.3, 2, 24), 3)])
@pytest.mark.parametrize("variant", ["unit", "sharp"])
def test_edges(geo, pieces, variant):
    _check(geo, pieces, lambda cfg: synth.attention_inputs(cfg, variant))


@pytest.mark.parametrize("geo,pieces", [((30, 25, 3, 1, 0.5, 20, 16), 1), ((90, 50, 3, 1, 0.3, 2, 24), 3)])
@pytest.mark.parametrize("slope", [10.0, -10.0])
def test_scores_rise_along_the_keys(geo, pieces, slope):
    """The running maximum moves in every tile (rises) or never (falls), in
    both blocks of a wavefront, and pieces merge maxima far apart."""
    _check(geo, pieces, lambda cfg: _monotone_score_inputs(cfg, slope, np.random.default_rng(17)))


# (first, last) of the keys with an infinite component: the first half-tile of
# all, the first tile of the second of three pieces (23 or 24 of 71 tiles), a
# half-tile in the middle of a piece, and a whole piece
@pytest.mark.parametrize("first,last", [(0, 32), (1472, 1536), (2016, 2048), (1472, 3008)])
def test_scores_of_minus_infinity(first, last):
    """Half of the queries score -inf on some keys (the others, in the same
    wavefronts, +inf, so no number): the other keys' share stays as it is."""
    from paper_2412_02962_amd import pcpp
    cfg = synth.AttnConfig(name="wide", H=82, W=100, n=2, i=0, p=0.1, heads=1, d=64, dtype=synth.DTYPE_BF16,
                           seed_id=92, batch=8)
    assert pcpp.pcpp_partial_attention_plan(gu.geom(cfg))[:2] == (256, 3)
    print("[case]", cfg, first, last, flush=True)
    inp = {k: (None if v is None else v.copy()) for k, v in synth.attention_inputs(cfg, "unit").items()}
    inp["k_fresh"][:, first:last, 0] = 0x7F80  # +inf in one dimension; the band's own keys come first
    got = gu.to_f64(gu.run_attention(cfg, inp))
    with np.errstate(invalid="ignore"):
        want = gu.oracle_attention(cfg, inp).reshape(got.shape)
    finite = np.isfinite(want).all(-1)
    assert 0.3 < finite.mean() < 0.7
    assert np.isfinite(got[finite]).all() and np.isnan(got[~finite]).all()
    gu.assert_close(cfg, got[finite], want[finite], f"{first} {last}")
