"""A bf16 context in less workspace than dmtd_workspace_bytes asks for: prefill and whole-sequence passes get shorter instead of the
call being refused, down to passes of 128 rows, and the results stay within the parity tests' tolerance of the oracle."""
import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config, norm_err, oracle_config

pytestmark = pytest.mark.gpu

SH = di.ModelShape(2, 256, 8, 2, 128, 512, 1000)
# What these contexts needed when every pass carried at most 128 rows: (batch, positions, bytes)
SIZES = [(1, 638, 52525056), (3, 300, 53044480)]


def engine_in(monkeypatch, cfg, nbytes, blob):
    lib = pkg.load_library()
    monkeypatch.setattr(lib, "dmtd_workspace_bytes", lambda _: nbytes)
    return pkg.Engine(cfg, blob)


@pytest.mark.parametrize("batch,n,nbytes", SIZES)
def test_shorter_passes_in_a_smaller_workspace(monkeypatch, batch, n, nbytes):
    import ctypes as C
    cfg = engine_config(SH, n + 2, batch)
    full = pkg.load_library().dmtd_workspace_bytes(C.byref(cfg.to_c()))
    assert nbytes < full
    blob = di.make_weight_blob(SH, seed=31, std=0.04, gain_sigma=0.2)
    toks = di.make_prompts(SH.vocab, batch, n, seed=5)
    ocfg = oracle_config(SH)
    w = O.unpack_weights(blob, ocfg)
    mask = O.inference_mask(n, n // 2, 3)
    refs = [O.masked_forward(toks[b], mask, 1, w, ocfg) for b in range(batch)]
    last = [O.masked_forward(toks[b], np.ones(n, np.uint8), 1, w, ocfg)[-1] for b in range(batch)]
    for size in (nbytes, (nbytes + full) // 2, full):
        eng = engine_in(monkeypatch, cfg, size, blob)
        got = eng.masked_forward(toks, mask, 1, want_logits=True)
        eng.prefill(toks)
        z = eng.logits()
        for b in range(batch):
            assert max(norm_err(got["logits"][b, i], refs[b][i]) for i in range(n)) < 2e-2
            assert norm_err(z[b], last[b]) < 2e-2
        eng.set_sampling(0.8, 20, 5)
        assert eng.decode(2, 1, 1).shape == (batch, 1)
        eng.close()


def test_a_workspace_without_room_for_short_passes_is_refused(monkeypatch):
    batch, n, nbytes = SIZES[0]
    with pytest.raises(pkg.DmtdError) as e:
        engine_in(monkeypatch, engine_config(SH, n + 2, batch), nbytes - (4 << 20), di.make_weight_blob(SH, seed=31))
    assert e.value.code == pkg.DMTD_ECAPACITY
