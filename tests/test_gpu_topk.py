"""Top-k of the draft's LM head on tied logits: value descending, then id
ascending, whole numbers compared exactly, the values with the oracle's logits.  The head's rows repeat, so every
value occurs several times, in one lane, wave, slice or in several slices."""
import dataclasses

import numpy as np
import pytest

import synth
from synth.configs import TINY
from oracle import msd as O
from parity import oracle_draft_static

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
    m = O.Models(dims, w, dr)
    n = 7
    none = np.zeros((0, dims.d_model), dtype=np.uint16)
    tokens = np.arange(n, dtype=np.int32)
    eng = Engine(dims, w, dr, max_batch=1, max_seq=128, max_tree=64, max_prompt=n)
    try:
        print(f"case: period {period}, k {k}", flush=True)
        first = eng.prefill(0, tokens, np.zeros(n, dtype=np.uint8), none)
        assert first < period
        dev = eng.new_trees(1)
        spec = make_static_spec(np.zeros(k, dtype=np.int32), np.arange(k, dtype=np.int32))
        eng.draft_tree([0], spec, dev)
        got = [int(t) for t in eng.trees_to_host(dev, 1)[0].token[1:k + 1]]
        # the oracle's logits of the period's rows: a group of ids per value,
        # best value first; values within its rounding may swap
        st, _, _, _ = O.prefill(m, tokens, np.zeros(n, dtype=np.uint8), none, n + 64)
        logits = oracle_draft_static(m, st, ["0"])[1][0]
        assert np.array_equal(logits[:period], logits[V - V % period - period:][:period])
        tol = 1e-3 * np.abs(logits).max()
        value = logits[[t % period for t in got]]
        assert np.all(value[1:] <= value[:-1] + tol)
        rest = np.delete(logits, got)
        assert rest.max() <= value[-1] + tol
        want = []
        while len(want) < k:  # every id of one value, ascending, then of the next
            j = got[len(want)] % period
            want += list(range(j, V, period))
        assert got == want[:k]
    finally:
        eng.close()
