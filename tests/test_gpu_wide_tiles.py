"""GPU parity of the wide GEMM's tiles of 192 weight rows (gate/up and QKV projections that fill the chip with them), where the last
tile along the rows and the last one along the outputs are partly empty, against the CPU oracle; and of gate/up launches whose tiles of 256
weight rows stay, the last of them summed in parts.

Tolerance: that of the other bf16 parity tests (2e-2 of the largest logit); a wrong row, output or gate/up pair is an error of order one.
"""
import ctypes as C

import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

S = di.ModelShape
# name: (shape, batch, positions), kind of projection, (rows per launch, rows of a tile, whole tiles, tiles of a second launch, parts of K), weight
# rows of a tile
CASES = {
    "gateup_in_parts": (S(1, 1024, 4, 2, 64, 4800, 300), 4, 505, 2, (2020, 256, 256, 48, 3), 256),
    "gateup_in_parts_ragged": (S(1, 704, 4, 2, 64, 4544, 300), 4, 449, 2, (1796, 256, 256, 32, 2), 256),      # 35.5 tiles; 4 rows in the last row tile
    "gateup_192": (S(1, 1088, 4, 2, 64, 2752, 300), 4, 505, 2, (2020, 256, 232, 0, 1), 192),            # 28.7 tiles of 96 outputs; K = 17 x 64
    "qkv_192_of_256": (S(1, 1024, 51, 17, 64, 64, 300), 4, 505, 0, (2020, 256, 232, 0, 1), 192),        # 28.3 tiles
    "gateup_192_a_round_not_full": (S(1, 1024, 4, 2, 64, 2560, 300), 4, 505, 2, (2020, 256, 216, 0, 1), 192),      # 26.7 tiles; 27 x 8 on 256
    "qkv_192_of_128_a_round_not_full": (S(1, 1024, 34, 17, 64, 64, 300), 1, 1003, 0, (1003, 128, 184, 0, 1), 192),
    "qkv_192_of_128": (S(1, 1600, 51, 17, 64, 64, 300), 1, 1003, 0, (1003, 128, 232, 0, 1), 192),       # a short last row tile of 107
}


@pytest.mark.parametrize("name", list(CASES))
def test_cases_reach_the_tiles_they_are_there_for(name):
    """Runs without a GPU."""
    sh, batch, n, kind, want, width = CASES[name]
    lib, cfg, plan = pkg.load_library(), engine_config(sh, n + 2, batch).to_c(), (C.c_int32 * 5)()
    assert lib.dmtd_wide_plan(C.byref(cfg), kind, batch * n, 256, plan) == pkg.DMTD_OK
    assert tuple(plan) == want
    assert lib.dmtd_wide_tile_width(C.byref(cfg), kind, batch * n, 256) == width


# (shape, kind, rows): launches whose 256-wide tiles are partly summed in parts of K, and where 192 or 320 weight rows would give whole tiles
IN_PARTS = {
    (S(1, 2560, 32, 8, 128, 9728, 300), 2, 1003): (1003, 256, 256, 48, 5),
    (S(1, 2560, 32, 8, 128, 9728, 300), 2, 2048): (2048, 256, 512, 96, 2),
    (S(1, 2560, 32, 8, 128, 9728, 300), 0, 2048): (2048, 128, 256, 128, 2),
    (S(1, 2048, 16, 8, 128, 6144, 300), 2, 1536): (1536, 256, 256, 32, 5),
    (S(1, 1536, 12, 2, 128, 8960, 300), 2, 1003): (1003, 256, 256, 24, 5),
    (S(1, 896, 14, 2, 64, 4864, 300), 2, 2048): (2048, 256, 256, 48, 3),
}


@pytest.mark.parametrize("case", list(IN_PARTS), ids=lambda c: f"{c[0].hidden}_kind{c[1]}_{c[2]}")
def test_another_width_keeps_the_parts_of_a_sum(case):
    """Runs without a GPU.  A sum in parts is nearer to 64 bits than one chain over all of K (2.0e-7 of its norm in five parts against 4.4e-7,
    K = 2560): a width that would turn the one into the other is not taken."""
    sh, kind, rows = case
    plan = (C.c_int32 * 5)()
    assert pkg.load_library().dmtd_wide_plan(C.byref(engine_config(sh, 2100).to_c()), kind, rows, 256, plan) == pkg.DMTD_OK
    assert tuple(plan) == IN_PARTS[case]


def test_tiles_of_another_width_are_whole():
    """Runs without a GPU: on any chip, and the tiles that the plan counts cover the launch."""
    lib, plan, rng, narrow = pkg.load_library(), (C.c_int32 * 5)(), np.random.RandomState(1), 0
    for _ in range(3000):
        sh = S(1, 64 * int(rng.randint(1, 65)), int(rng.randint(1, 9)) * 4, 4, 128, 64 * int(rng.randint(1, 193)), int(rng.randint(100, 200000)))
        rows, cus, kind = int(rng.randint(193, 2049)), int(rng.choice([64, 80, 228, 256, 304])), int(rng.randint(0, 5))
        cfg = engine_config(sh, 2100).to_c()
        width = lib.dmtd_wide_tile_width(C.byref(cfg), kind, rows, cus)
        assert lib.dmtd_wide_plan(C.byref(cfg), kind, rows, cus, plan) == pkg.DMTD_OK
        nqkv = (sh.n_q_heads + 2 * sh.n_kv_heads) * sh.head_dim
        outputs = {0: nqkv, 1: sh.hidden, 2: 2 * sh.intermediate, 3: sh.hidden, 4: sh.vocab}[kind]
        assert width in (192, 256) and plan[2] + plan[3] == -(-plan[0] // plan[1]) * -(-outputs // width)
        if width == 192:
            narrow += 1
            assert kind in (0, 2) and plan[3] == 0 and plan[4] == 1
    assert narrow > 30


def test_tile_width_refuses_what_the_plan_refuses():
    lib = pkg.load_library()
    bf16, fp32 = (engine_config(S(2, 256, 8, 2, 128, 512, 1000, dtype=t), 64, 8).to_c() for t in ("bf16", "fp32"))
    assert lib.dmtd_wide_tile_width(C.byref(bf16), 0, 193, 256) in (192, 256)
    for cfg, kind, rows, cus in ((bf16, 0, 192, 256), (bf16, 5, 193, 256), (bf16, -1, 193, 256), (bf16, 0, 193, 0), (fp32, 0, 193, 256)):
        assert lib.dmtd_wide_tile_width(C.byref(cfg), kind, rows, cus) == pkg.DMTD_EINVAL
    assert lib.dmtd_wide_tile_width(None, 0, 193, 256) == pkg.DMTD_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_wide_tiles_against_oracle(name):
    sh, batch, n, _, _, _ = CASES[name]
    blob = di.make_weight_blob(sh, seed=31, std=0.04, gain_sigma=0.2)
    toks = di.make_prompts(sh.vocab, batch, n, seed=5)
    mask = O.inference_mask(n, n // 2, 3)
    eng = pkg.Engine(engine_config(sh, n + 2, batch), blob)
    got = eng.masked_forward(toks, mask, 1, want_logits=True)["logits"]
    ocfg = oracle_config(sh)
    w = O.unpack_weights(blob, ocfg)
    for b in range(batch):
        ref = O.masked_forward(toks[b], mask, 1, w, ocfg)
        worst = max(norm_err(got[b, i], ref[i]) for i in range(n))
        assert worst < 2e-2, (b, worst)
