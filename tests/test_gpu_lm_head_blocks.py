"""GPU parity of the LM head with 17 to 32 rows where it runs in blocks of ten waves (131073 to 163840 entries at a width of 512 or more in whole
rounds of its pipeline, and 262145 to 327680 at widths of whole 1024s) and next to that, against the CPU oracle.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit); a wrong row or weight tile is an error of order one.  The token is
the largest of the reported logits, the first of equal ones.
"""
import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

S = di.ModelShape
CASES = {
    # name: (width, entries, sequences)
    "fewest_entries": (512, 131073, 17),          # one entry in the last tile
    "most_entries": (512, 163840, 32),            # 512 full blocks
    "ragged": (640, 151936, 25),                  # the last block has 16 of 20 tiles
    "odd_steps": (576, 151936, 25),               # nine steps: blocks of eight waves
    "narrow": (128, 131073, 17),                  # blocks of eight waves, as in the next two
    "one_round_more": (512, 163841, 18),
    "two_rounds": (512, 262145, 18),
    "two_rounds_1024": (1024, 262145, 18),        # blocks of ten
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_lm_head_against_oracle(name):
    width, vocab, batch = CASES[name]
    sh = S(1, width, 2, 1, 64, 64, vocab)
    blob = di.make_weight_blob(sh, seed=41, std=0.04, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, batch, 2, seed=5)
    eng = pkg.Engine(engine_config(sh, 8, batch), blob)
    first = eng.prefill(toks)
    z = eng.logits()
    ocfg = oracle_config(sh)
    w = O.unpack_weights(blob, ocfg, np.float32)
    for b in range(batch):
        ref = O.masked_forward(toks[b], np.ones(2, np.uint8), 1, w, ocfg)[-1]
        assert norm_err(z[b], ref) < 2e-2, b
        assert int(first[b]) == int(np.argmax(z[b])), b
