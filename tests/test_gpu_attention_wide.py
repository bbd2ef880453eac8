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
