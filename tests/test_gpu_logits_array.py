"""Arrays that Engine.logits() returns: each keeps its values whatever the engine does afterwards, as long as it or a view of it
is held, although the engine lends the same page-locked memory again once nobody holds it."""
import numpy as np
import pytest
import torch

import dmtd_inputs as di
from parity_util import engine_config
import paper_2510_11958_amd as pkg

pytestmark = pytest.mark.gpu


def test_logits_arrays_stay_as_they_were():
    sh = di.ModelShape(2, 64, 2, 1, 64, 96, 130, dtype="fp32")
    eng = pkg.Engine(engine_config(sh, 64, 3), di.make_weight_blob(sh, seed=3))
    prompts = di.make_prompts(sh.vocab, 3, 5, seed=5)

    def take(n):                               # logits after a prefill of n sequences
        eng.reset()
        eng.prefill(prompts[:n])
        return eng.logits()

    want = [take(n).copy() for n in (3, 2, 1)]
    whole, row = take(3), take(2)[1]           # the second array's memory is not the first's; a view of one row is all that is kept
    tensor = torch.from_numpy(take(1))
    assert not np.shares_memory(whole, row)
    for _ in range(3):
        take(3)
    assert np.array_equal(whole, want[0]) and np.array_equal(row, want[1][1]) and np.array_equal(tensor.numpy(), want[2])
    at = whole.ctypes.data
    del whole
    kept = take(2)[:, 3:7].T                   # lent again: no array of the first kind is left
    assert kept.base is not None and at <= kept.ctypes.data < at + want[0].nbytes
    later = take(3)
    assert np.array_equal(kept, want[1][:, 3:7].T) and np.array_equal(later, want[0])
    del eng
    assert np.array_equal(kept, want[1][:, 3:7].T)
