"""An output of the SwiGLU has the same bits whichever kernel its row went through: the wide GEMM's whole tiles (of 256 and 192 weight rows),
its tiles summed in parts, the tiled kernel, the kernels of few rows.  Tiles of 128 rows round the low part of outputs 1 and 2 of four from the
rounded product: there one in some 70 may differ by a unit of the low part.

The models make every sum exact, so that only the activation itself is left to differ.  Embeddings are small whole numbers and one
entry of 2^20, which alone decides every norm's scale; gate and up weights are small whole numbers times 2^8; attention adds nothing (its
weights are 0); the down projection and the LM head each pick one element.  A logit is then one SwiGLU output (its two bf16 parts) times
a power of two.  v_rcp_f32 in place of the division on one route changes 1 in 110 of them."""
import ctypes as C

import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from parity_util import engine_config

S = di.ModelShape
V, INPUTS = 300, 64
CASES = {
    # name: (width, SwiGLU width, rows of the long pass), its gate/up launch (rows, rows of a tile, whole tiles, tiles in parts, parts)
    "tiles_of_128": (256, 448, 400, (400, 128, 16, 0, 1)),
    "tiles_of_256": (256, 6144, 1100, (1100, 256, 240, 0, 1)),
    "tiles_of_256_by_192": (1024, 3072, 2046, (2046, 256, 256, 0, 1)),       # 256 weight rows a tile would be 192 tiles
    "tiles_in_parts": (1024, 1024, 400, (400, 128, 0, 32, 3)),
}


def _model(width, ffn):
    """Shape, weight blob (bf16 bits), and which SwiGLU outputs are picked."""
    sh = S(1, width, 2, 1, 64, ffn, V, tied_embeddings=False)
    rng = np.random.RandomState(7)
    f32 = {"embed": np.zeros((V, width), np.float32)}
    f32["embed"][:, 0] = 2.0 ** 20
    f32["embed"][:, 1:INPUTS] = rng.randint(-15, 16, (V, INPUTS - 1))
    gate, up = np.zeros((2, ffn, width), np.float32)
    for t in (gate, up):
        t[:, 1:INPUTS] = rng.randint(-8, 9, (ffn, INPUTS - 1)) * 256.0
    picked = min(width - INPUTS, ffn, V)
    which = rng.permutation(ffn)[:picked]
    down, head = np.zeros((width, ffn), np.float32), np.zeros((V, width), np.float32)
    down[INPUTS + np.arange(picked), which] = 1.0
    head[np.arange(picked), INPUTS + np.arange(picked)] = 1.0
    qd, kd, one = 128, 64, np.ones(width, np.float32)
    parts = [f32["embed"], one, np.zeros((qd, width)), np.zeros((kd, width)), np.zeros((kd, width)), np.ones(64), np.ones(64), np.zeros((width, qd)),
             one, gate, up, down, one, head]
    blob = di.f32_to_bf16_bits(np.concatenate([np.asarray(p, np.float32).ravel() for p in parts]))
    assert blob.size == di.blob_elems(sh)
    return sh, blob, which


def _logits(eng, tokens):
    """[token id, entry] of a pass over these tokens; a row depends on nothing but its token."""
    eng.reset()
    z = eng.masked_forward(tokens[None], np.ones(tokens.size, np.uint8), 1, want_logits=True)["logits"][0]
    out = np.empty((V, V), np.float32)
    out[tokens] = z
    assert np.array_equal(z, out[tokens])
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_cases_reach_the_launches_they_are_there_for(name):
    width, ffn, rows, want = CASES[name]
    plan = (C.c_int32 * 5)()
    cfg = engine_config(S(1, width, 2, 1, 64, ffn, V, tied_embeddings=False), rows + 2).to_c()
    assert pkg.load_library().dmtd_wide_plan(C.byref(cfg), 2, rows, 256, plan) == pkg.DMTD_OK
    assert tuple(plan) == want


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_swiglu_has_the_same_bits_on_every_route(name):
    width, ffn, rows, plan = CASES[name]
    sh, blob, which = _model(width, ffn)
    picked = which.size
    eng = pkg.Engine(engine_config(sh, rows + 2), blob)
    ids = np.arange(V, dtype=np.int32)
    want = np.empty((V, V), np.float32)
    for t in range(0, V, 100):              # the tiled kernel
        want[t:t + 100] = _logits(eng, ids[t:t + 100])[t:t + 100]
    assert np.isfinite(want).all() and np.abs(want[:, :picked]).min() < np.abs(want[:, :picked]).max()
    wide = _logits(eng, np.resize(ids, rows))
    if plan[1] == 128 and plan[4] == 1:
        # a unit of the low part is 2^-8 of it, and it is at most 2^-8 of the value
        rounded = np.flatnonzero((which % 4 == 1) | (which % 4 == 2))
        differ = wide[:, rounded] != want[:, rounded]
        assert 0 < differ.mean() < 1 / 40
        assert (np.abs(wide[:, rounded] - want[:, rounded]) <= 2.0 ** -16 * np.abs(want[:, rounded])).all()
        wide[:, rounded] = want[:, rounded]
    assert np.array_equal(wide, want), f"{int((wide != want).sum())} of {V * picked} outputs"
    for t in range(0, V, 12):               # the kernels of few rows
        few = _logits(eng, ids[t:t + 12])[t:t + 12]
        assert np.array_equal(few, want[t:t + 12]), t
