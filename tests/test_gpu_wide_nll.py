"""Scoring with more than 192 rows in a pass: without logits the LM head's tiles leave maxima, sums and best entries only.  Every
position's cross entropy and greedy choice against those of the same engine's logits (which take the other route), in 64 bits.

Tolerance: the logits of both routes are the same sums; the cross entropy adds fp32 exponentials (1e-6 of each, relative) and a logarithm,
so 1e-5 covers them at values of a few units; the best entry's logit is the largest up to the last bits of a logit.
"""
import numpy as np
import pytest

import dmtd_inputs as di
from oracle import dmtd_oracle as O
from parity_util import engine_config
import paper_2510_11958_amd as pkg

pytestmark = pytest.mark.gpu

S = di.ModelShape
CASES = {
    # name: (shape, batch, length): rows of a pass, entries of a tile's 256 that exist
    "193_rows_vocab_130": (S(1, 64, 2, 1, 64, 128, 130), 1, 193),
    "400_rows_vocab_256": (S(2, 128, 2, 1, 64, 128, 256), 2, 200),
    "300_rows_vocab_257": (S(1, 128, 4, 2, 64, 192, 257), 3, 100),
    "700_rows_vocab_20000": (S(2, 256, 4, 2, 64, 256, 20000), 7, 100),
    "two_passes_vocab_4100": (S(1, 128, 2, 1, 64, 128, 4100), 3, 900),          # 2046 rows, then 654
    "tiny_vocab_20": (S(1, 64, 2, 1, 64, 128, 20), 1, 250),                     # too few entries for the scratch: the other route
}


@pytest.mark.parametrize("name", list(CASES))
def test_cross_entropy_without_logits(name):
    sh, batch, n = CASES[name]
    blob = di.make_weight_blob(sh, seed=21, std=0.05, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, batch, n, seed=9)
    mask = O.training_mask(n, 3)
    eng = pkg.Engine(engine_config(sh, n + 3, batch), blob)
    want = eng.masked_forward(toks, mask, 1, want_logits=True)
    for _ in range(2):
        got = eng.masked_forward(toks, mask, 1)
        z = want["logits"].astype(np.float64)
        top = z.max(-1)
        nll = np.log(np.exp(z - top[..., None]).sum(-1)) + top
        nll[:, :-1] -= np.take_along_axis(z[:, :-1], toks[:, 1:, None].astype(np.int64), -1)[..., 0]
        nll[:, -1] = 0
        assert np.abs(got["nll"] - nll).max() < 1e-5 * max(1.0, np.abs(z).max()), np.abs(got["nll"] - nll).max()
        assert (got["nll"][:, -1] == 0).all()
        picked = np.take_along_axis(z, got["best"][..., None].astype(np.int64), -1)[..., 0]
        assert (top - picked <= 1e-6 * np.abs(top)).all()
        assert np.allclose(got["loss"], nll[:, :-1].mean(1), rtol=1e-5)


def test_equal_and_infinite_logits():
    """A head whose rows are all equal (the lowest entry is the best), then one with an entry that makes logits infinite."""
    sh = S(1, 64, 2, 1, 64, 128, 700)
    blob = di.make_weight_blob(sh, seed=21, std=0.05)
    table = blob[:sh.vocab * sh.hidden].reshape(sh.vocab, sh.hidden)
    table[:] = table[5]
    toks = di.make_prompts(sh.vocab, 1, 230, seed=9)
    mask = np.ones(230, np.uint8)
    eng = pkg.Engine(engine_config(sh, 240, 1), blob)
    got = eng.masked_forward(toks, mask, 1)
    assert (got["best"] == 0).all()
    assert np.abs(got["nll"][:, :-1] - np.log(700)).max() < 1e-4
    big = table.copy()
    big[650] = (table[5] & 0x8000) | 0x7F00          # the signs of the row, values of 1.7e38: sums beyond the largest float
    table[:] = big
    eng = pkg.Engine(engine_config(sh, 240, 1), blob)
    a, b = eng.masked_forward(toks[:, :230], mask, 1, want_logits=True), eng.masked_forward(toks, mask, 1)
    assert np.isinf(a["logits"]).any() or np.isnan(a["logits"]).any()
    assert np.array_equal(np.isnan(a["nll"]), np.isnan(b["nll"]))
    assert np.array_equal(a["best"], b["best"])
