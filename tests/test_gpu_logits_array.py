"""Arrays that Engine.logits() returns: each keeps its values whatever the engine does afterwards, whoever still reads it - the host, or
an upload to the GPU that was started and not waited for."""
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
    whole, row = take(3), take(2)[1]           # a view of one row is all that is kept of the second
    tensor = torch.from_numpy(take(1))
    assert not np.shares_memory(whole, row)
    for _ in range(3):
        take(3)
    assert np.array_equal(whole, want[0]) and np.array_equal(row, want[1][1]) and np.array_equal(tensor.numpy(), want[2])
    del whole
    kept = take(2)[:, 3:7].T
    later = take(3)
    assert np.array_equal(kept, want[1][:, 3:7].T) and np.array_equal(later, want[0])
    del eng
    assert np.array_equal(kept, want[1][:, 3:7].T)


@pytest.mark.parametrize("rows", [slice(None), slice(1, 3)], ids=["whole", "some_rows"])
def test_an_upload_that_nobody_waited_for_keeps_its_values(rows):
    """The array is dropped while an upload of it waits behind other work of torch's stream; the next logits() must not reach it."""
    sh = di.ModelShape(1, 64, 2, 1, 64, 96, 20000, dtype="fp32")
    eng = pkg.Engine(engine_config(sh, 64, 4), di.make_weight_blob(sh, seed=3))
    prompts = di.make_prompts(sh.vocab, 4, 5, seed=5)
    eng.prefill(prompts)
    first = eng.logits().copy()
    eng.decode(1, 1, 1)
    second = eng.logits().copy()
    assert not np.array_equal(first, second)
    for _ in range(3):
        eng.reset()
        eng.prefill(prompts)
        torch.cuda._sleep(20_000_000)          # about 10 ms of torch's stream
        up = torch.from_numpy(eng.logits()[rows]).to("cuda", non_blocking=True)
        eng.decode(1, 1, 1)
        later = eng.logits()
        torch.cuda.synchronize()
        assert np.array_equal(up.cpu().numpy(), first[rows])
        assert np.array_equal(later, second)


def test_closed_engine_gives_its_staging_memory_back():
    sh = di.ModelShape(1, 64, 2, 1, 64, 96, 130, dtype="fp32")
    eng = pkg.Engine(engine_config(sh, 64, 1), di.make_weight_blob(sh, seed=3))
    eng.prefill(di.make_prompts(sh.vocab, 1, 5, seed=5))
    z = eng.logits()
    kept = z.copy()
    assert z.flags.owndata and z.flags.writeable
    eng.close()
    assert eng._stage is None and np.array_equal(z, kept)
