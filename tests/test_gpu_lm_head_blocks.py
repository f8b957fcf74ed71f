"""GPU parity of the LM head with 17 to 32 rows where it runs in blocks of ten waves (131073 to 163840 entries and a width of whole rounds of
its pipeline) and next to that, against the CPU oracle.

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
    "fewest_entries": (128, 131073, 17),          # one entry in the last tile; the first steps are the last
    "most_entries": (256, 163840, 32),            # 512 full blocks
    "ragged": (320 + 64, 151936, 25),             # the last block has 16 of 20 tiles
    "odd_steps": (192, 151936, 25),               # three steps: blocks of eight waves
    "two_rounds": (128, 163841, 18),              # blocks of eight waves
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
