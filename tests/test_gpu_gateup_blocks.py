"""GPU parity of gate/up with 8 to 16 rows around the line between blocks of two and of four waves (64 to 128 blocks of four waves on 256
compute units, rows that do not fit the one-tile-per-block kernel), against the CPU oracle.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit); a wrong row or weight tile is an error of order one.
"""
import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

S = di.ModelShape
CASES = {
    # name: (width, SwiGLU width, sequences)
    "65_blocks": (2048, 64 * 65, 8),        # the fewest that take two waves
    "128_blocks": (2048, 64 * 128, 13),     # the most
    "64_blocks": (2048, 64 * 64, 16),       # four waves
    "129_blocks": (2048, 64 * 129, 8),      # four waves
    "96_blocks": (2048, 64 * 96, 16),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_gateup_blocks_against_oracle(name):
    width, ffn, batch = CASES[name]
    sh = S(1, width, 2, 1, 64, ffn, 300)
    blob = di.make_weight_blob(sh, seed=43, std=0.02, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, batch, 3, seed=5)
    eng = pkg.Engine(engine_config(sh, 8, batch), blob)
    eng.prefill(toks[:, :2])
    eng.decode(1, 1, 1, forced=toks[:, 2:])      # one row per sequence
    z = eng.logits()
    ocfg = oracle_config(sh)
    w = O.unpack_weights(blob, ocfg, np.float64)
    for b in range(batch):
        ref = O.masked_forward(toks[b], np.ones(3, np.uint8), 1, w, ocfg)[-1]
        assert norm_err(z[b], ref) < 2e-2, b
