"""GPU parity of the prefill attention where its launch has more blocks than compute units but no more than two per unit (the second
round then starts with the shortest blocks), where gains spread scores so far that a later tile often has a row's largest, and where blocks
have one tile of keys, against the CPU oracle.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit).  A score's error from the rounded keys is 2^-9.8 of its
spread, 0.4 % of a probability at the spread of 3 that gains of 1 + N(0, 1) give; a block that took another block's rows, or a sum
left at the wrong scale, is an error of order one.
"""
import ctypes as C

import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

S = di.ModelShape
CASES = {
    # name: (shape, batch, positions, spread of the gains)
    "blocks_280_hd64_gq4": (S(1, 128, 32, 8, 64, 64, 300), 1, 1100, 0.2),        # 35 slices of 8 blocks, 32 of them from the longest down; 12 rows in the last
    "blocks_510_hd64_gq1": (S(1, 128, 34, 34, 64, 64, 300), 3, 600, 0.2),        # 5 slices of 102, three down and two up
    "growing_hd128_gq4": (S(1, 128, 32, 8, 128, 64, 300), 1, 1100, 1.0),
    "growing_hd64_gq2": (S(1, 128, 8, 4, 64, 64, 300), 2, 900, 1.0),             # 120 blocks: even and odd tiles apart
    # blocks whose groups of waves have one tile of 64 keys, next to blocks with one key more
    "one_tile_hd128": (S(1, 128, 32, 8, 128, 64, 300), 40, 30, 0.2),             # 320 blocks, one group
    "one_and_two_tiles_hd64": (S(1, 128, 16, 2, 64, 64, 300), 31, 65, 0.2),      # 310 blocks, one group; the last row sees 65 keys
    "one_to_three_tiles_hd128": (S(1, 128, 32, 8, 128, 64, 300), 3, 129, 0.2),   # 120 blocks, two groups; the last row sees 129 keys
}

# On 256 compute units: (blocks of a slice of 128 query vectors per KV head and sequence, slices, slices from the longest down)
ORDERS = {
    "blocks_280_hd64_gq4": (8, 35, 32),
    "blocks_510_hd64_gq1": (102, 5, 3),
    "growing_hd128_gq4": (8, 35, 32),
}


@pytest.mark.parametrize("name", list(ORDERS))
def test_cases_reach_the_order_they_are_there_for(name):
    """Runs without a GPU: all positions are in one pass, its launch has 257 to 512 blocks, and some slices start from the shortest up."""
    sh, batch, n, _ = CASES[name]
    plan = (C.c_int32 * 2)()
    assert pkg.load_library().dmtd_score_plan(C.byref(engine_config(sh, n + 2, batch).to_c()), batch, n, plan) == pkg.DMTD_OK
    assert plan[0] == n
    rows = 128 // (sh.n_q_heads // sh.n_kv_heads)
    per_slice, slices = sh.n_kv_heads * batch, -(-n // rows)
    down = min(slices, -(-256 // per_slice))
    assert 256 < per_slice * slices <= 512 and down < slices
    assert (per_slice, slices, down) == ORDERS[name]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_prefill_attention_against_oracle(name):
    sh, batch, n, sigma = CASES[name]
    blob = di.make_weight_blob(sh, seed=37, std=0.04, gain_sigma=sigma)
    toks = di.make_prompts(sh.vocab, batch, n, seed=5)
    eng = pkg.Engine(engine_config(sh, n + 2, batch), blob)
    mask = np.ones(n, np.uint8)
    got = eng.masked_forward(toks, mask, 1, want_logits=True)["logits"]
    ocfg = oracle_config(sh)
    w = O.unpack_weights(blob, ocfg)
    for b in range(batch):
        ref = O.masked_forward(toks[b], mask, 1, w, ocfg)
        worst = max(norm_err(got[b, i], ref[i]) for i in range(n))
        print(f"{name} {b}: {worst:.2e}")
        assert worst < 2e-2, (b, worst)
