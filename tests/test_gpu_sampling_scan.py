"""Sampled token selection at the edges of its two launches: list limits (top_k 64 and 65, more equal logits than the list
holds), slice ends (vocabularies around 2048 and 4096), no restriction.  The oracle's sampler on the very logits the GPU reports
must pick the GPU's token wherever its two best scores are more than 1e-3 apart (float32 rounding of z / T and of the
logarithms moves a score by about 1e-6 of its size); the top-k set is decided by exact comparisons on both sides."""
import numpy as np
import pytest

import dmtd_inputs as di
import paper_2510_11958_amd as pkg
from oracle import dmtd_oracle as O
from parity_util import engine_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,top_k,std", [
    (2047, 64, 0.05), (2049, 65, 0.05), (4097, 2, 0.05), (4097, 0, 0.05), (9000, 64, 0.05), (9000, 65, 0.05), (9000, 8999, 0.05),
    (151936, 64, 0.05), (151936, 0, 0.05),
    (9000, 3, 0.0),          # all logits equal: every entry stays in, more than the list holds
])
def test_draws_match_the_oracles_sampler(vocab, top_k, std):
    sh = di.ModelShape(1, 64, 2, 1, 64, 128, vocab, dtype="bf16")
    blob = di.make_weight_blob(sh, seed=13, std=std)
    B, P, T, seed = 3, 9, 0.8, 77
    eng = pkg.Engine(engine_config(sh, 32, B), blob)
    eng.set_sampling(T, top_k, seed)
    tokens, pos, decided = eng.prefill(di.make_prompts(vocab, B, P, seed=6)), P - 1, 0
    for _ in range(6):
        z = eng.logits()
        for b in range(B):
            s = O.sampling_scores(z[b].astype(np.float64), T, top_k, seed, b, pos)
            assert np.isfinite(s[int(tokens[b])])                 # the draw lies inside the top-k set
            best = np.sort(s[np.isfinite(s)])[-2:]
            if best[-1] - best[0] > 1e-3:
                assert int(tokens[b]) == int(np.argmax(s)), (b, pos)
                decided += 1
        pos = eng.state()["n_tok"]
        tokens = eng.decode_cycle(2, 1, max_new=1)[:, 0]
    assert decided >= 15
