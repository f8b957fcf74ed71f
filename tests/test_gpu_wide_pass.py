"""GPU parity of passes that carry many rows (more than 192 activation rows, more than 16 positions per sequence): the wide
projection GEMM (tiles of 128 or 256 rows x 256 outputs, K optionally split over blocks) and the prefill attention kernel (128
query vectors x 64 keys per tile), at the edges of their tiles, against the CPU oracle.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit: the bf16 KV cache's rounding through the layers);
a wrong row, key or output of a tile is an error of order one.
"""
import ctypes as C

import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

TOL_BF16 = 2e-2

S = di.ModelShape
CASES = {
    # name: (shape, batch, positions)
    "rows_129_hd128_gq4": (S(2, 256, 8, 2, 128, 512, 1000), 1, 129),             # the LDS-tiled kernel's two passes below the wide GEMM's least rows
    "rows_193_hd128_gq4": (S(2, 256, 8, 2, 128, 512, 1000), 1, 193),             # the wide GEMM's least rows; one row in a group of 16
    "rows_385_hd128_gq2": (S(2, 1024, 8, 4, 128, 1600, 2000), 1, 385),           # one row in the fourth tile of 128; K split over blocks
    "rows_3x83_hd64_gq1": (S(2, 192, 3, 3, 64, 320, 203), 3, 83),                # K = 192, outputs not multiples of 128 or 256
    "rows_256_hd64_gq7": (S(2, 128, 7, 1, 64, 448, 515), 1, 256),                # 18 rows per attention block; full row tiles
    "rows_2x257_hd128_gq2": (S(2, 320, 4, 2, 128, 960, 129), 2, 257),            # 514 rows: two blocks of logits; 64-key tiles + 1
    "rows_17x17_hd64_gq16": (S(1, 128, 16, 1, 64, 64, 300), 17, 17),             # fewest positions of a wide pass, 8 rows per attention block
    "rows_5x450_hd64_gq4": (S(1, 64, 4, 1, 64, 128, 97), 5, 450),                # 2250 rows: two passes, the second reads the first's keys
    # more than 512 blocks of 16 query vectors, from which on the prefill attention kernel takes a pass
    "vectors_8224_hd128_gq4": (S(2, 256, 32, 8, 128, 512, 1000), 1, 257),        # 513 blocks of 16; one row in the ninth tile of 32
    "vectors_8106_hd64_gq7": (S(2, 128, 21, 3, 64, 448, 515), 2, 193),           # 18 rows per block, 13 rows in the last
    "vectors_9600_hd64_gq1": (S(2, 192, 16, 16, 64, 320, 203), 3, 200),          # 128 rows per block
    "vectors_8224_hd128_gq2": (S(2, 320, 16, 8, 128, 960, 129), 2, 257),         # one row in the fifth tile of 64
    "vectors_19200_hd64_gq8": (S(1, 128, 8, 1, 64, 128, 97), 48, 50),            # 192 blocks of 128, two groups of waves
    # the layouts that the plan of a projection reaches at these sizes: LAYOUTS below
    "tiles_256_whole_and_tail": (S(2, 896, 14, 2, 64, 8896, 17000), 8, 256),
    "tiles_256_qkv_ragged": (S(1, 512, 66, 22, 64, 704, 300), 4, 505),            # 2020 rows: the last row tile has 228, nqkv is 27.5 tiles
    "tiles_256_qkv_tail_ragged": (S(1, 768, 78, 26, 64, 704, 300), 4, 505),       # nqkv is 32.5 tiles
    "tiles_128_qkv_tail_ragged": (S(1, 1024, 93, 31, 64, 704, 300), 4, 449),      # the last row tile has 4 rows, nqkv is 38.75 tiles
    "resid_in_two_launches": (S(2, 1024, 4, 2, 64, 128, 300), 5, 400),
    "vectors_38400_hd64_gq8": (S(1, 128, 16, 2, 64, 128, 97), 48, 50),           # 384 blocks of 128, more than a block per CU: one group of waves
}


# What the cases above are there for, on 256 compute units: (rows per launch, rows of a tile, whole tiles, tiles of the second launch,
# parts of K).  The kinds a case does not name run tiles of 128 rows without a whole round before a tail.
KINDS = {"qkv": 0, "oproj": 1, "gateup": 2, "down": 3, "lmhead": 4}
LAYOUTS = {
    "tiles_256_whole_and_tail": {"gateup": (2048, 256, 512, 48, 3), "down": (2048, 256, 0, 32, 8), "lmhead": (512, 256, 134, 0, 1)},
    "tiles_256_qkv_ragged": {"qkv": (2020, 256, 224, 0, 1)},
    "tiles_256_qkv_tail_ragged": {"qkv": (2020, 256, 256, 8, 3)},
    "tiles_128_qkv_tail_ragged": {"qkv": (1796, 128, 512, 73, 3)},
    "resid_in_two_launches": {"oproj": (1536, 128, 0, 48, 1), "down": (1536, 128, 0, 48, 1)},
}


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_cases_reach_the_layouts_they_are_there_for(name):
    """Runs without a GPU: the cases that cover the tiles of 256 rows, split tails and launches in parts really reach them."""
    sh, batch, n = CASES[name]
    cfg = engine_config(sh, n + 2, batch).to_c()
    for kind, want in LAYOUTS[name].items():
        plan = (C.c_int32 * 5)()
        rows = batch * n if kind != "lmhead" else min(batch * n, 512)      # a scoring pass that is asked for logits, as here, holds those of 512 rows at a time
        assert pkg.load_library().dmtd_wide_plan(C.byref(cfg), KINDS[kind], rows, 256, plan) == pkg.DMTD_OK
        assert tuple(plan) == want, kind


def test_wide_plan_refuses_what_the_wide_kernel_does_not_take():
    lib, plan = pkg.load_library(), (C.c_int32 * 5)()
    bf16, fp32 = (engine_config(S(2, 256, 8, 2, 128, 512, 1000, dtype=t), 64, 8).to_c() for t in ("bf16", "fp32"))
    assert lib.dmtd_wide_plan(C.byref(bf16), 0, 193, 256, plan) == pkg.DMTD_OK
    for cfg, kind, rows, cus, out in ((bf16, 0, 192, 256, plan), (bf16, 5, 193, 256, plan), (bf16, -1, 193, 256, plan), (bf16, 0, 193, 0, plan),
                                      (bf16, 0, 193, 256, None), (fp32, 0, 193, 256, plan)):
        assert lib.dmtd_wide_plan(C.byref(cfg), kind, rows, cus, out) == pkg.DMTD_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_wide_pass_against_oracle(name):
    sh, batch, n = CASES[name]
    blob = di.make_weight_blob(sh, seed=31, std=0.04, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, batch, n, seed=5)
    mask = O.inference_mask(n, n // 2, 3)
    eng = pkg.Engine(engine_config(sh, n + 2, batch), blob)
    got = eng.masked_forward(toks, mask, 1, want_logits=True)
    ocfg = oracle_config(sh)
    w = O.unpack_weights(blob, ocfg)
    worst = 0.0
    for b in range(batch):
        ref = O.masked_forward(toks[b], mask, 1, w, ocfg)
        worst = max(worst, max(norm_err(got["logits"][b, i], ref[i]) for i in range(n)))
        err = np.abs(got["nll"][b, :n - 1] - O.next_token_nll(ref, toks[b])).max()
        assert err < 2 * TOL_BF16 * np.abs(ref).max(), (b, err)
    assert worst < TOL_BF16, worst
    # prefill takes the same passes: its logits are the last position's, with every position full
    eng.prefill(toks)
    full = np.ones(n, np.uint8)
    for b in range(batch):
        assert norm_err(eng.logits()[b], O.masked_forward(toks[b], full, 1, w, ocfg)[-1]) < TOL_BF16
    print(f"{name}: worst logit error {worst:.2e}")


@pytest.mark.gpu
@pytest.mark.parametrize("n,limit", [(1003, 2.6e-4), (2048, 1.8e-4)])
def test_few_cached_values_round_the_other_way(n, limit):
    """How near the QKV projection's sums are to 64 bits decides how many keys and values round to the other bf16 neighbour: of 2.05 million
    values 2.3e-4 with K = 2560 summed in five parts (passes of 128 rows), 3.2e-4 to 3.6e-4 in one fp32 chain, 1.4e-4 in chains of
    4 k-steps of 32.  2.6e-4 is three standard deviations of the count above the first.  Of 4.19 million values at 2048 rows 1.67e-4 and 1.51e-4
    (keys, values) in chains of 4 k-steps; 1.8e-4 is two standard deviations above, and chains of one step in tiles of 192 weight rows leave 1.87e-4."""
    import torch
    sh = S(1, 2560, 32, 8, 128, 128, 300)
    blob = di.make_weight_blob(sh, seed=31, std=0.02, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, 1, n, seed=5)
    eng = pkg.Engine(engine_config(sh, n + 2), blob)
    eng.prefill(toks)
    ocfg = oracle_config(sh)
    o = O.DmtdOracle(ocfg, O.unpack_weights(blob, ocfg, np.float64), n + 2, np.float64)
    o.prefill(toks[0])
    got = eng.read_kv(0, 0, n)
    for which, ref in ((0, o.K[0]), (1, o.V[0])):
        want = torch.from_numpy(np.ascontiguousarray(np.transpose(ref[:n], (1, 0, 2)))).to(torch.bfloat16).float().numpy()
        share = float((got[which] != want).mean())
        print(("keys", "values")[which], f"{share:.2e}")
        assert share < limit, (which, share)


@pytest.mark.gpu
@pytest.mark.parametrize("name,at", [("vectors_8224_hd128_gq4", 40), ("vectors_8224_hd128_gq4", 95), ("vectors_9600_hd64_gq1", 100),
                                     ("vectors_19200_hd64_gq8", 13), ("vectors_38400_hd64_gq8", 41), ("vectors_8106_hd64_gq7", 192)])
def test_a_value_that_is_not_finite_stays_behind_its_position(name, at):
    """Passes through the prefill attention, one token's embedding NaN (the LM head is a table of its own): its row and the later ones,
    which see it, are NaN, the rows before it are bit for bit those of the same sequence with another token there."""
    sh, batch, n = CASES[name]
    sh = S(sh.n_layers, sh.hidden, sh.n_q_heads, sh.n_kv_heads, sh.head_dim, sh.intermediate, sh.vocab, tied_embeddings=False)
    blob = di.make_weight_blob(sh, seed=31, std=0.04, gain_sigma=0.2)
    bad, good = 7, 8
    blob[bad * sh.hidden:(bad + 1) * sh.hidden] = 0x7FC0
    toks = di.make_prompts(sh.vocab, batch, n, seed=5)
    toks[toks == bad] = good
    eng = pkg.Engine(engine_config(sh, n + 2, batch), blob)
    mask = np.ones(n, np.uint8)
    clean = eng.masked_forward(toks, mask, 1, want_logits=True)["logits"]
    assert np.isfinite(clean).all()
    broken = toks.copy()
    broken[-1, at] = bad
    got = eng.masked_forward(broken, mask, 1, want_logits=True)["logits"]
    assert np.array_equal(got[:-1], clean[:-1])
    assert np.array_equal(got[-1, :at], clean[-1, :at])
    assert np.isnan(got[-1, at:]).all()
