"""The packed-weight GEMM at the edges of its tiles and splits, through prompts
of the C ABI: row counts on both sides of every row-tile height (32 to 160
rows), of the passes that run as several launches, and widths with partial
weight tiles and K blocks.  A row's keys and values depend on the rows before
it only, so one oracle run over the longest prompt is the reference of all.

Tolerance: keys and values are stored in bfloat16 (half a unit in the last
place is 2^-9 of the value); one more unit for values near a rounding boundary
gives 2^-7 of the row's largest magnitude.
"""
import dataclasses

import numpy as np
import pytest

import synth
from synth.configs import TINY, WIDE
from oracle import model as M
from oracle import msd as O
from parity import argmax_ok, compare_static_tree, oracle_draft_static, row_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RTOL = 2.0 ** -7


def text_prompt(wl, n):
    rng = np.random.default_rng(wl.seed)
    tokens = rng.integers(0, wl.dims.vocab, n).astype(np.int32)
    return tokens, np.zeros(n, dtype=np.uint8), np.zeros((0, wl.dims.d_model), dtype=np.uint16)


def rows_of(view, layer, n, transposed):
    a = view[layer, 0, :, :, :n] if transposed else view[layer, 0, :, :n, :].transpose(1, 2)
    bits = a.cpu().numpy().astype(np.int16).view(np.uint16)   # [KV, hd, n]
    return M.widen(bits).transpose(2, 0, 1).reshape(n, -1)


@pytest.mark.parametrize("dims_of, counts", [
    # a partial 64-row weight tile (F = 2880) and a half K block in the down projection
    (WIDE.dims, [1, 31, 32, 33, 64, 65, 95, 97, 128, 129, 160, 161, 255, 257, 319]),
    # q/k/v of 12 tiles, an FFN of 688 (10 tiles and 48 rows; K blocks cut at 48 columns)
    (TINY.dims, [5, 63, 66, 130, 192, 300]),
    # K smaller than a block, one 40-wide remainder
    (dataclasses.replace(WIDE.dims, d_model=168, n_heads=3, n_kv_heads=1, head_dim=64,
                         ffn_dim=296, vocab=512), [3, 32, 65, 161]),
    # long prompts of few heads: 32 queries a workgroup, keys in four chains
    (dataclasses.replace(TINY.dims, n_layers=2, n_heads=2, n_kv_heads=1, head_dim=128, ffn_dim=296,
                         vocab=512), [639, 640, 641, 672, 703, 705, 767, 769]),
    (dataclasses.replace(TINY.dims, n_layers=2, n_heads=3, n_kv_heads=3, head_dim=64, ffn_dim=296,
                         vocab=512), [640, 673, 704, 769]),
    # of many: from 640 rows on 128 queries a workgroup, 64 keys a block
    (dataclasses.replace(TINY.dims, n_layers=2, n_heads=32, n_kv_heads=4, head_dim=128,
                         ffn_dim=296, vocab=512), [639, 640, 641, 672, 703, 705, 767, 769]),
    (dataclasses.replace(TINY.dims, n_layers=2, n_heads=48, n_kv_heads=3, head_dim=64,
                         ffn_dim=296, vocab=512), [640, 673, 704, 769]),
], ids=["wide", "tiny", "narrow", "long-128", "long-64", "long-heads-128", "long-heads-64"])
def test_prompt_rows_at_tile_edges(dims_of, counts):
    from paper_2505_14260_amd.msd import Engine
    wl = dataclasses.replace(TINY, dims=dims_of)
    n_max = max(counts)
    w = synth.make_target_weights(dims_of, wl.seed)
    dr = synth.make_draft_weights(dims_of, w, wl.seed, "random")
    tokens, vis, rows = text_prompt(wl, n_max)
    st, _, _, _ = O.prefill(O.Models(dims_of, w, dr), tokens, vis, rows, n_max + 64)
    eng = Engine(dims_of, w, dr, max_batch=1, max_seq=(n_max + 128) // 64 * 64, max_tree=64,
                 max_prompt=n_max)
    try:
        tk, tv, _, _ = eng.kv_views()
        for n in counts:
            print(f"case: {n} rows, d {dims_of.d_model}", flush=True)
            eng.prefill(0, tokens[:n], vis[:n], rows)
            torch.cuda.synchronize()
            for l in range(dims_of.n_layers):
                for view, ref, tr in ((tk, st.kv.k, False), (tv, st.kv.v, True)):
                    ok, err = row_close(rows_of(view, l, n, tr), ref[l, :n].reshape(n, -1), RTOL)
                    assert ok, (n, l, tr, err)
    finally:
        eng.close()


def test_prompt_of_several_launches():
    """2,080 rows: two launches per product, the second shorter."""
    from paper_2505_14260_amd.msd import Engine
    dims = dataclasses.replace(TINY.dims, n_layers=2)
    wl = dataclasses.replace(TINY, dims=dims)
    n = 2080
    w = synth.make_target_weights(dims, wl.seed)
    dr = synth.make_draft_weights(dims, w, wl.seed, "random")
    tokens, vis, rows = text_prompt(wl, n)
    st, _, _, _ = O.prefill(O.Models(dims, w, dr), tokens, vis, rows, n + 64)
    eng = Engine(dims, w, dr, max_batch=1, max_seq=n + 96, max_tree=64, max_prompt=n)
    try:
        print(f"case: {n} rows", flush=True)
        eng.prefill(0, tokens, vis, rows)
        torch.cuda.synchronize()
        tk, tv, _, _ = eng.kv_views()
        for l in range(dims.n_layers):
            for view, ref, tr in ((tk, st.kv.k, False), (tv, st.kv.v, True)):
                ok, err = row_close(rows_of(view, l, n, tr), ref[l, :n].reshape(n, -1), RTOL)
                assert ok, (l, tr, err)
    finally:
        eng.close()


@pytest.mark.parametrize("mode", ["embedding", "feature"])
@pytest.mark.parametrize("runs, heads", [
    ([1, 4, 1], 4),              # text, visual, text, ...: one row on either side
    ([3, 70, 40, 33, 2], 4),     # tiles with both kinds, text between the visual rows
    ([0, 64, 96, 31, 1], 4),     # tiles of visual rows only; the last row alone
    ([33], 4),                   # no visual row
    ([300, 161, 380], 4),        # 680 rows wanted of 841
    ([300, 161, 380], 48),       # with tiles of 128 queries, some without a wanted one
], ids=["1-4-1", "3-70-40-33-2", "0-64-96-31-1", "33", "300-161-380", "300-161-380-48"])
def test_prompt_of_text_and_visual_runs(runs, heads, mode):
    """A prompt's last layer runs over the rows whose features are read: the
    text rows in any order, or all with the Visual Feature input.  The draft's
    rows carry features of the whole target: 2e-2, as in the parity tests."""
    from paper_2505_14260_amd.msd import Engine, make_static_spec
    dims = dataclasses.replace(TINY.dims, n_layers=2, n_heads=heads, n_kv_heads=4)
    n = sum(runs)
    vis = np.concatenate([np.full(r, i & 1, dtype=np.uint8) for i, r in enumerate(runs)])
    rng = np.random.default_rng(n)
    tokens = np.where(vis, 0, rng.integers(0, dims.vocab, n)).astype(np.int32)
    w = synth.make_target_weights(dims, TINY.seed)
    dr = synth.make_draft_weights(dims, w, TINY.seed, "random")
    rows = w["embed"][rng.integers(0, dims.vocab, int(vis.sum()))].copy()
    m = O.Models(dims, w, dr)
    st, first, _, logits = O.prefill(m, tokens, vis, rows, n + 64, visual_input=mode)
    eng = Engine(dims, w, dr, max_batch=1, max_seq=(n + 160) // 64 * 64, max_tree=64, max_prompt=n)
    try:
        print(f"case: runs {runs}, {mode} input", flush=True)
        eng.set_draft_input(mode)
        got = eng.prefill(0, tokens, vis, rows)
        assert got == first or argmax_ok(got, logits[n - 1])
        tk, tv, dk, dv = eng.kv_views()
        torch.cuda.synchronize()
        parent, rank, _ = synth.static_tree_arrays(TINY.tree.paths)
        spec = make_static_spec(parent[1:], rank[1:])
        ref, logs, ranks = oracle_draft_static(m, st, TINY.tree.paths)  # catch-up + tree
        caches = [(tk, tv, st.kv, dims.n_layers, RTOL), (dk, dv, st.dkv, 1, 2e-2)]
        for k, v, kv, nl, tol in caches:
            for l in range(nl):
                for view, r, tr in ((k, kv.k, False), (v, kv.v, True)):
                    ok, err = row_close(rows_of(view, l, n, tr), r[l, :n].reshape(n, -1), tol)
                    assert ok, (nl, l, tr, err)
        if got == first:
            dev = eng.new_trees(1)
            eng.draft_tree([0], spec, dev)
            assert compare_static_tree(eng.trees_to_host(dev, 1)[0], ref, logs, ranks) >= ref.n // 2
    finally:
        eng.close()


@pytest.mark.parametrize("n", [2, 33, 65, 130, 193])
def test_training_products_at_edges(n):
    """Gradients of sequences of 1 to 192 rows (the weight gradients' K, cut and
    padded to 64) on a model whose widths leave partial tiles and whose
    vocabulary is odd (padded logits rows), three query heads on one kv head.
    The features carry the target's bf16 key/value cache: 2e-2 of each
    parameter's largest gradient, as in the training parity tests."""
    from paper_2505_14260_amd.msd import Engine
    from oracle import train as TR
    dims = dataclasses.replace(WIDE.dims, d_model=168, n_heads=3, n_kv_heads=1, head_dim=64,
                               ffn_dim=296, vocab=1037, n_layers=1)
    wl = dataclasses.replace(TINY, dims=dims)
    w = synth.make_target_weights(dims, wl.seed)
    dr = synth.make_draft_weights(dims, w, wl.seed, "random")
    m = O.Models(dims, w, dr)
    tokens, vis, rows = text_prompt(wl, n)
    print(f"case: training sequence of {n} rows", flush=True)
    eng = Engine(dims, w, dr, max_batch=1, max_seq=256, max_tree=16, max_prompt=193)
    try:
        assert not np.any(eng.train_read(0)["wq"])     # no sums yet
        loss = eng.train_accumulate(0, tokens, vis, rows)
        g = eng.train_read(0)
        params = TR.draft_params(m.draft)
        h, e, pt = TR.sequence_inputs(m, tokens, vis, rows)
        ref_loss, _, _, gref = TR.batch_grads(m, params, [(h, e, vis, pt)])
        assert abs(loss[0] / (n - 1) - ref_loss) <= 1e-2 * abs(ref_loss)
        # one row attends to itself alone: its query and key gradients are zero
        # up to the rounding of the others
        floor = 1e-5 * max(np.abs(r).max() for r in gref.values())
        for k in TR.PARAM_KEYS:
            err = np.abs(g[k] / (n - 1) - gref[k]).max() / max(np.abs(gref[k]).max(), floor)
            assert err <= 2e-2, (k, err)
        # a second sequence adds to the sums; after an update they start again
        eng.train_accumulate(0, tokens, vis, rows)
        g2 = eng.train_read(0)
        eng.train_apply(0.0)
        assert not np.any(eng.train_read(0)["wd"])
        eng.train_accumulate(0, tokens, vis, rows)
        g3 = eng.train_read(0)
        for k in TR.PARAM_KEYS:
            scale = max(np.abs(g[k]).max(), floor * (n - 1))
            assert np.abs(g2[k] - 2 * g[k]).max() <= 1e-5 * scale, k
            assert np.abs(g3[k] - g[k]).max() <= 1e-5 * scale, k
    finally:
        eng.close()
