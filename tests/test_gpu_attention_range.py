"""The prefill attention over values near the largest that 32 bits hold: a row's result is a mean of the values it sees, so it is finite and
right while they are, also where a later tile's score exceeds the largest so far (the sums are kept against the largest score there is; against an
older one, lower by up to 8 powers of two, they would overflow).

Three tokens, embeddings one entry each, so that the layer's projections pick columns: "first" (position 0) and "later" (a tile further on, of the same
parity) hold values of up to 2^124, all others 0.  Keys and queries lie in the two pairs of dims that rotary embedding turns least (1e-4 over
these positions), at angles that put the scores, in powers of two, at 0, 29 and 35.5.  The O projection brings values back by 2^-120.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit)."""
import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

S = di.ModelShape
V, AT, OTHER, FIRST, LATER = 300, 150, 0, 1, 2
CASES = {
    # name: (query heads, KV heads, head dim, positions)
    "hd128_two_groups": (32, 8, 128, 257),       # 72 blocks
    "hd128_one_group": (32, 8, 128, 1100),       # 280 blocks
    "hd64_two_groups": (16, 8, 64, 600),
    "hd64_one_group": (32, 16, 64, 1100),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_values_near_the_largest_stay_finite(name):
    nh, nkv, hd, n = CASES[name]
    width = 128
    sh = S(1, width, nh, nkv, hd, 64, V, tied_embeddings=False)
    rng = np.random.RandomState(3)
    embed = np.zeros((V, width), np.float32)
    embed[np.arange(width), np.arange(width)] = 1.0
    gain = 2.0
    unit = gain * gain * np.sqrt(hd) * np.log2(np.e)      # a score in powers of two: unit times the cosine between query and key
    q, k, v = np.zeros((nh, hd, width), np.float32), np.zeros((nkv, hd, width), np.float32), np.zeros((nkv, hd, width), np.float32)
    a, c = hd // 2 - 2, hd // 2 - 1                       # the slowest pairs' first dims
    q[:, a, :] = 1.0
    for t, score in ((OTHER, 0.0), (FIRST, 29.0), (LATER, 35.5)):
        k[:, a, t], k[:, c, t] = score / unit, np.sqrt(1.0 - (score / unit) ** 2)
    for t in (FIRST, LATER):
        v[:, :, t] = rng.uniform(-1, 1, (nkv, hd)) * 2.0 ** 124 / np.sqrt(width)
    o = rng.normal(size=(width, nh * hd)) * 2.0 ** -120
    one = np.ones(width)
    zero = np.zeros((64, width))
    parts = [embed, one, q, k, v, np.full(hd, gain), np.full(hd, gain), o, one, zero, zero, np.zeros((width, 64)), one, rng.normal(size=(V, width)) * 0.05]
    blob = di.f32_to_bf16_bits(np.concatenate([np.asarray(p, np.float32).ravel() for p in parts]))
    assert blob.size == di.blob_elems(sh)
    toks = np.full((1, n), OTHER, np.int32)
    toks[0, 0], toks[0, AT] = FIRST, LATER
    eng = pkg.Engine(engine_config(sh, n + 2), blob)
    mask = np.ones(n, np.uint8)
    got = eng.masked_forward(toks, mask, 1, want_logits=True)["logits"][0]
    ocfg = oracle_config(sh)
    ref = O.masked_forward(toks[0], mask, 1, O.unpack_weights(blob, ocfg, np.float64), ocfg)
    assert np.isfinite(ref).all()
    for i in range(n):
        assert norm_err(got[i], ref[i]) < 2e-2, i
