"""Top-k of the draft's LM head on tied logits: value descending, then id
ascending, whole numbers compared exactly.  The head's rows repeat, so every
value occurs several times, in one lane, wave, slice or in several slices."""
import dataclasses

import numpy as np
import pytest

import synth
from synth.configs import TINY

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("period", [1, 64, 256, 700, 2048])
@pytest.mark.parametrize("k", [1, 5, 16])
def test_ties_go_to_the_lowest_id(period, k):
    from paper_2505_14260_amd.msd import Engine, make_static_spec
    dims = dataclasses.replace(TINY.dims, n_layers=1)
    V = dims.vocab
    w = synth.make_target_weights(dims, TINY.seed)
    dr = synth.make_draft_weights(dims, w, TINY.seed, "random")
    w["lm_head"] = np.ascontiguousarray(w["lm_head"][np.arange(V) % period])
    n = 7
    tokens = np.arange(n, dtype=np.int32)
    eng = Engine(dims, w, dr, max_batch=1, max_seq=128, max_tree=64, max_prompt=n)
    try:
        print(f"case: period {period}, k {k}", flush=True)
        first = eng.prefill(0, tokens, np.zeros(n, dtype=np.uint8),
                            np.zeros((0, dims.d_model), dtype=np.uint16))
        assert first < period
        dev = eng.new_trees(1)
        spec = make_static_spec(np.zeros(k, dtype=np.int32), np.arange(k, dtype=np.int32))
        eng.draft_tree([0], spec, dev)
        got = [int(t) for t in eng.trees_to_host(dev, 1)[0].token[1:k + 1]]
        want = []
        while len(want) < k:  # every id of one value, then of the next
            j = got[len(want)] % period
            want += list(range(j, V, period))
        assert got == want[:k]
        assert len({t % period for t in got}) == -(-k // (V // period)) or V % period
    finally:
        eng.close()
