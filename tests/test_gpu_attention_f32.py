"""float32 attention at the edges of its tiles (16 queries, 16 keys, four
wavefronts that share a block's keys), against the float64 oracle."""

import numpy as np
import pytest

from paper_2412_02962_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(cfg, inp):
    got = gu.to_f64(gu.run_attention(cfg, inp)).reshape(cfg.batch, cfg.n_q, cfg.C)
    want = gu.oracle_attention(cfg, inp).reshape(got.shape)
    # one rounding to float32 (half an ulp is 2^-24 of the value); the float64
    # sums and exponentials of scores up to 10^3 are off by about 1e-12
    bound = 2.0 ** -23 * np.abs(want) + 1e-9 * np.sqrt(np.mean(want ** 2))
    worst = float((np.abs(got - want) / bound).max())
    print(f"{cfg.name}: worst error / bound {worst:.3f}", flush=True)
    assert np.isfinite(got).all() and worst <= 1.0


def _cfg(H, W, n, i, p, heads, batch=1):
    return synth.AttnConfig(name=f"f32 {H}x{W} n{n} i{i} p{p} b{batch}", H=H, W=W, n=n, i=i, p=p, heads=heads, d=64,
                            dtype=synth.DTYPE_F32, seed_id=77, batch=batch)


# queries 1, 15, 16, 17, 33; keys from one (three wavefronts idle) through one
# tile more or less than the wavefronts share evenly, with sources that end
# inside a tile
@pytest.mark.parametrize("geo", [(1, 1, 1, 0, 0.0, 2), (1, 15, 1, 0, 0.0, 1), (1, 16, 1, 0, 0.0, 3),
                                 (2, 17, 2, 0, 1.0, 2), (3, 11, 1, 0, 0.0, 1, 2), (12, 5, 4, 2, 0.4, 2, 2),
                                 (16, 16, 4, 1, 0.25, 2), (9, 23, 3, 1, 0.7, 1)])
def test_f32_tile_edges(geo):
    cfg = _cfg(*geo)
    _check(cfg, synth.attention_inputs(cfg))


@pytest.mark.parametrize("order", [1, -1])
def test_f32_scores_far_apart(order):
    """Scores that rise (fall) along the keys over about 1000, so that the
    weights' reference moves several times in every wavefront and the
    wavefronts merge references hundreds apart."""
    cfg = _cfg(9, 23, 3, 1, 0.7, 1)
    inp = {k: (None if v is None else v.copy()) for k, v in synth.attention_inputs(cfg).items()}
    # one dimension carries a ramp over the context rows; the query's weight on it is constant
    inp["q"][..., 0] = 8.0
    up, own, dn = inp["k_up"], inp["k_fresh"], inp["k_dn"]
    ramp = order * np.linspace(-500.0, 500.0, 3 * own.shape[1], dtype=np.float32)
    for j, t in enumerate((up, own, dn)):
        t[..., 0] = ramp[j * own.shape[1]:(j + 1) * own.shape[1]]
    _check(cfg, inp)


def test_f32_value_rows_past_the_end_weigh_nothing():
    """The last tile is padded with copies of the last row; an infinite value
    there must come through with that row's weight only."""
    cfg = _cfg(1, 17, 1, 0, 0.0, 1)
    inp = {k: (None if v is None else v.copy()) for k, v in synth.attention_inputs(cfg).items()}
    inp["v_fresh"][0, 16, 5] = np.inf
    out = gu.to_f64(gu.run_attention(cfg, inp)).reshape(cfg.n_q, cfg.C)
    assert np.isposinf(out[:, 5]).all()
    assert np.isfinite(np.delete(out, 5, axis=1)).all()


# keys whose scores are -inf for half of the queries (and +inf, so no number,
# for the others, which share their workgroups): the first tile of the second
# wavefront's keys, all of its keys, tiles in the middle of a wavefront's
@pytest.mark.parametrize("first,last", [(64, 80), (64, 128), (144, 176)])
def test_f32_scores_of_minus_infinity(first, last):
    """Keys of weight 0 leave the other keys' share as it is."""
    cfg = _cfg(16, 16, 1, 0, 0.0, 2)
    inp = {k: (None if v is None else v.copy()) for k, v in synth.attention_inputs(cfg).items()}
    inp["k_fresh"][:, first:last, ::64] = np.inf        # dimension 0 of each head
    finite = inp["q"][..., ::64] < 0                    # [batch, query, head]
    assert finite.any() and not finite.all()
    got = gu.to_f64(gu.run_attention(cfg, inp)).reshape(cfg.n_q, cfg.heads, 64)
    with np.errstate(invalid="ignore"):
        want = gu.oracle_attention(cfg, inp).reshape(got.shape)
    finite = finite.reshape(cfg.n_q, cfg.heads)
    assert np.isfinite(want[finite]).all() and np.isnan(want[~finite]).all()
    assert np.isnan(got[~finite]).all() and np.isfinite(got[finite]).all()
    # the bound of _check
    assert (np.abs(got - want)[finite] <= 2.0 ** -23 * np.abs(want[finite]) + 1e-9).all()
