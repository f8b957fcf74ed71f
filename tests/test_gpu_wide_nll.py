"""Scoring with more than 192 rows in a pass: without logits the LM head's tiles leave maxima, sums and best entries only.  Every
position's cross entropy and greedy choice against those of the same engine's logits (which take the other route), in 64 bits.

Tolerance: the logits of both routes are the same sums; the cross entropy adds fp32 exponentials (1e-6 of each, relative) and a logarithm,
so 1e-5 covers them at values of a few units; the best entry's logit is the largest up to the last bits of a logit.
"""
import ctypes as C

import numpy as np
import pytest

import dmtd_inputs as di
from oracle import dmtd_oracle as O
from parity_util import engine_config
import paper_2510_11958_amd as pkg

S = di.ModelShape
CASES = {
    # name: (shape, batch, length), rows of the first pass's tiles (0: the vocabulary is too small for their results, the other route):
    # rows of a pass, entries of a tile's 256 that exist
    "193_rows_vocab_130": (S(1, 64, 2, 1, 64, 128, 130), 1, 193, 128),
    "400_rows_vocab_256": (S(2, 128, 2, 1, 64, 128, 256), 2, 200, 128),
    "300_rows_vocab_257": (S(1, 128, 4, 2, 64, 192, 257), 3, 100, 128),
    "700_rows_vocab_20000": (S(2, 256, 4, 2, 64, 256, 20000), 7, 100, 256),
    "900_rows_k1024_vocab_10000": (S(1, 1024, 4, 2, 64, 128, 10000), 3, 300, 256),
    "two_passes_vocab_4100": (S(1, 128, 2, 1, 64, 128, 4100), 3, 900, 256),          # 2046 rows, then 654
    "250_rows_vocab_12": (S(1, 64, 2, 1, 64, 128, 12), 1, 250, 128),
    "250_rows_vocab_11": (S(1, 64, 2, 1, 64, 128, 11), 1, 250, 0),
    "2048_rows_vocab_48": (S(1, 64, 2, 1, 64, 128, 48), 4, 512, 128),                 # logits of 512 rows are what the place is for
    "2048_rows_vocab_47": (S(1, 64, 2, 1, 64, 128, 47), 4, 512, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_cases_reach_the_routes_they_are_there_for(name):
    """Runs without a GPU."""
    sh, batch, n, bm = CASES[name]
    cfg, lib, score, wide = engine_config(sh, n + 3, batch).to_c(), pkg.load_library(), (C.c_int32 * 2)(), (C.c_int32 * 5)()
    assert lib.dmtd_score_plan(C.byref(cfg), batch, n, score) == pkg.DMTD_OK
    assert score[1] == (bm > 0) and score[0] == min(n, 2048 // batch)
    assert lib.dmtd_wide_plan(C.byref(cfg), 4, batch * score[0], 256, wide) == pkg.DMTD_OK
    assert bm in (0, wide[1]) and wide[3] == 0


def test_score_plan_of_other_passes():
    lib, plan = pkg.load_library(), (C.c_int32 * 2)()
    bf16, fp32 = (engine_config(S(1, 64, 2, 1, 64, 128, 1000, dtype=t), 400, 4).to_c() for t in ("bf16", "fp32"))
    for cfg, batch, n, want in ((bf16, 1, 192, (192, 0)), (bf16, 1, 193, (193, 1)), (bf16, 4, 400, (400, 1)), (fp32, 2, 400, (64, 0))):
        assert lib.dmtd_score_plan(C.byref(cfg), batch, n, plan) == pkg.DMTD_OK and tuple(plan) == want
    for cfg, batch, n, out in ((None, 1, 9, plan), (C.byref(bf16), 0, 9, plan), (C.byref(bf16), 5, 9, plan), (C.byref(bf16), 1, 0, plan),
                               (C.byref(bf16), 1, 401, plan), (C.byref(bf16), 1, 9, None)):
        assert lib.dmtd_score_plan(cfg, batch, n, out) == pkg.DMTD_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_cross_entropy_without_logits(name):
    sh, batch, n, _ = CASES[name]
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


@pytest.mark.gpu
@pytest.mark.parametrize("vocab,batch,n,bm", [(700, 1, 230, 128), (20000, 7, 100, 256)])
def test_equal_and_infinite_logits(vocab, batch, n, bm):
    """A head whose rows are all equal (the lowest entry is the best), then one with an entry that makes logits infinite."""
    sh = S(1, 64, 2, 1, 64, 128, vocab)
    blob = di.make_weight_blob(sh, seed=21, std=0.05)
    table = blob[:sh.vocab * sh.hidden].reshape(sh.vocab, sh.hidden)
    table[:] = table[5]
    toks = di.make_prompts(sh.vocab, batch, n, seed=9)
    mask = np.ones(n, np.uint8)
    cfg, wide = engine_config(sh, n + 10, batch), (C.c_int32 * 5)()
    assert pkg.load_library().dmtd_wide_plan(C.byref(cfg.to_c()), 4, batch * n, 256, wide) == pkg.DMTD_OK and wide[1] == bm
    eng = pkg.Engine(cfg, blob)
    got = eng.masked_forward(toks, mask, 1)
    assert (got["best"] == 0).all()
    assert np.abs(got["nll"][:, :-1] - np.log(vocab)).max() < 1e-4
    big = table.copy()
    big[650] = (table[5] & 0x8000) | 0x7F00          # the signs of the row, values of 1.7e38: sums beyond the largest float
    table[:] = big
    eng = pkg.Engine(cfg, blob)
    a, b = eng.masked_forward(toks, mask, 1, want_logits=True), eng.masked_forward(toks, mask, 1)
    assert np.isinf(a["logits"]).any() or np.isnan(a["logits"]).any()
    assert np.array_equal(np.isnan(a["nll"]), np.isnan(b["nll"]))
    assert np.array_equal(a["best"], b["best"])
