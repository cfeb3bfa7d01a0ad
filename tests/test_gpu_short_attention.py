"""Contexts of one page (two for one-row passes) run the attention in one kernel
that folds its own pages; longer ones, and captured steps, which are replayed at
any length, run the per-page partials and the combine.  An eager engine against
one that replays graphs, from inside the first page into the third: the same
bits in every record, every logit and the KV state."""
import numpy as np
import pytest

import lede_inputs as li
from tests.parity import say
from tests.test_gpu_decode import GQA_128, SMALL_128, SMALL_GQA, TINY, TINY_BF16

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("model", [TINY, TINY_BF16, SMALL_128, SMALL_GQA, GQA_128], ids=lambda m: m.name)
def test_short_contexts_equal_the_combined_pages(model):
    from paper_2606_03113_amd import Engine
    say("short attention", model.name)
    L = model.n_layers
    acts = [(1, 3), (L, 2), (1, 0), (L, 8), (1, 6)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        engines = []
        for graphs in (0, 1):
            eng = Engine(model, max_ctx=192, k_max=8)
            eng.load_weights(li.weights(model), li.qnet_weights(model))
            eng.lede_set_options(graphs, 1)
            eng.lede_prefill(li.uniform_int(1, 20, 11, 0, model.vocab - 1))
            engines.append(eng)
        a, b = engines
        for i in range(200):
            act = acts[i % len(acts)]
            ra, rb = a.lede_step(act, log_qnet=False), b.lede_step(act, log_qnet=False)
            assert (ra.emitted, ra.drafts, ra.seq_len) == (rb.emitted, rb.drafts, rb.seq_len), (i, act)
            for which in (0, 3) if act[1] else (0,):
                assert np.array_equal(a.logits(which), b.logits(which)), (i, act, which)
            assert a.lede_get_kv_state() == b.lede_get_kv_state()
            if ra.seq_len > 150:
                break
        assert a.lede_get_kv_state()[0] > 150
        side.synchronize()
    for eng in engines:
        eng.close()
