"""The error of a product's float32 sums, through the logits of msd_verify.

The layer's output and down projections are zero and the embeddings have a mean
square of exactly one (integers over 16 whose squares sum to 256 per feature), so
that the features are the embeddings times the gains: 16 significant bits, which
the bf16 pair of a split row holds exactly.  The LM head's products over K = d_model
are then compared with float64, and all of the difference is the sums' own.

Bound: an accumulator that takes n adds of 16 columns each is off by about
2.5e-8 sqrt(n) of the result's root mean square (one rounding of at most 2^-24 per
add, at the size that the sum has by then); a block of 128 columns is 16 adds, hi
and lo, and one accumulator takes a quarter of K and at most seven blocks.  A
quarter more is allowed.
"""
import dataclasses

import numpy as np
import pytest

import synth
from synth.configs import TINY
from oracle import model as M

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def bf16_bits(x):
    u = np.asarray(x, dtype=np.float32).view(np.uint32)
    assert not np.any(u & 0xFFFF)      # exact
    return (u >> 16).astype(np.uint16)


def unit_rows(rng, n, d):
    """n rows of d integers with squares that sum to 256 d, signs at random."""
    out = np.empty((n, d), dtype=np.int64)
    for row in out:
        r = 0
        while not 0 < r < 60000:
            row[:-4] = rng.integers(8, 23, d - 4)
            r = 256 * d - int((row[:-4] ** 2).sum())
        row[-4:] = four_squares(r)
    return out * rng.choice([-1, 1], size=out.shape)


def four_squares(r):
    for a in range(int(r ** 0.5 / 2), int(r ** 0.5) + 1):
        for b in range(a + 1):
            rest = r - a * a - b * b
            if rest < 0:
                break
            for c in range(int(rest ** 0.5), int((rest / 2) ** 0.5) - 1, -1):
                e = int(round((rest - c * c) ** 0.5))
                if c * c + e * e == rest and max(a, c) < 256:
                    return a, b, c, e
    raise AssertionError(r)


@pytest.mark.parametrize("d", [256, 4096])
@pytest.mark.parametrize("n_seq,nodes", [(1, 1), (1, 27), (1, 61), (2, 47), (5, 64), (8, 63)])
def test_sums_of_the_lm_head(d, n_seq, nodes):
    from paper_2505_14260_amd.msd import Engine, Tree
    dims = dataclasses.replace(TINY.dims, n_layers=1, d_model=d, n_heads=4, n_kv_heads=4,
                               head_dim=64, ffn_dim=256, vocab=576, norm_eps=1e-30)
    rng = np.random.default_rng(d + nodes)
    w = synth.make_target_weights(dims, 3)
    x = unit_rows(rng, dims.vocab, d) / 16.0
    g = rng.integers(128, 256, d) / 128.0
    w["embed"], w["final_norm"] = bf16_bits(x), bf16_bits(g)
    last = w["layers"][0]
    zero = [k for k in last if k in ("wo", "wd", "w_down")]
    assert len(zero) == 2
    for k in zero:
        last[k] = np.zeros_like(last[k])
    dr = synth.make_draft_weights(dims, w, 3, "random")
    eng = Engine(dims, w, dr, max_batch=8, max_seq=128, max_tree=64, max_prompt=4)
    try:
        print(f"case: {n_seq} trees of {nodes} nodes, K {d}", flush=True)
        raw, tokens = b"", []
        for b in range(n_seq):
            eng.prefill(b, np.arange(3, dtype=np.int32), np.zeros(3, dtype=np.uint8),
                        np.zeros((0, d), dtype=np.uint16))
            t = Tree()
            t.n_nodes = nodes
            ids = rng.choice(dims.vocab, nodes, replace=False)
            for i, tok in enumerate(ids):      # a root and its children
                t.token[i], t.parent[i], t.depth[i] = int(tok), 0 if i else -1, min(i, 1)
                t.anc[i] = 1 | (1 << i)
            raw += bytes(t)
            tokens += list(ids)
        trees = torch.frombuffer(bytearray(raw), dtype=torch.uint8).cuda()
        _, logits = eng.verify(list(range(n_seq)), trees, nodes, want_logits=True)
        got = logits.cpu().numpy().astype(np.float64).reshape(len(tokens), -1)
        ref = (x[tokens] * g) @ M.widen(w["lm_head"]).astype(np.float64).T
        err = np.sqrt(((got - ref) ** 2).mean() / (ref ** 2).mean())
        bound = 1.25 * 2.5e-8 * np.sqrt(16 * min(max(d // 128 // 4, 1), 7))
        print(f"error {err:.2e}, bound {bound:.2e}")
        assert err <= bound
    finally:
        eng.close()
