"""The work that users of this library have it do, as cases that can be timed.

A case is one call sequence through the C ABI's binding
(paper_2505_14260_amd.msd) on a model of one of the shapes the benchmark and
the tests use, with a few layers (a block of the stack) or all of them:

  verify   msd_verify: the target over the trees of a batch (one node per
           tree is the plain decode step), logits included
  draft    msd_set_state + msd_draft_tree: one draft tree per sequence
  cycle    a whole decode cycle: msd_set_state, msd_draft_tree, msd_verify,
           msd_accept_compact (or msd_accept_sample at temperature > 0)
  prefill  msd_prefill of a visual + text prompt
  train    one draft training step: msd_train_accumulate, msd_train_read of
           the gradients, msd_train_apply

Decode cases start from an imported cache of `prefix` slots (msd_set_state),
so that a pass can be repeated.  Inputs are drawn on the GPU from the seed.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2505_14260_amd import msd as B

# layers, d_model, query heads, kv heads, head_dim, ffn, vocab, rope theta, eps
MODELS = {
    "tiny-llama-4L-d256": (4, 256, 4, 4, 64, 688, 4096, 1e4, 1e-5),
    "wide-gqa-2L-d1024": (2, 1024, 8, 2, 128, 2880, 4096, 1e4, 1e-5),
    "llava-1.5-7b-shaped": (32, 4096, 32, 32, 128, 11008, 32000, 1e4, 1e-5),
    "llava-1.5-13b-shaped": (40, 5120, 40, 40, 128, 13824, 32000, 1e4, 1e-5),
    "qwen2.5-vl-7b-shaped": (28, 3584, 28, 4, 128, 18944, 152064, 1e6, 1e-6),
}
# rank paths of the static trees ("01": the root's best child's second-best)
TREES = {
    "static-14": ["0", "1", "00", "01", "10", "11", "000", "001", "010", "011", "100", "101",
                  "110", "111"],
    "static-26": ["0", "1", "2", "3", "00", "01", "02", "10", "11", "20", "30", "000", "001",
                  "010", "020", "100", "200", "0000", "0001", "0010", "0100", "1000", "00000",
                  "00001", "00010", "00100"],
}
DYN_TOPK, DYN_DEPTH = 10, 6  # the dynamic trees' breadth and depth
LR = 5e-5


class Dims:
    def __init__(self, model, layers):
        (_, self.d, self.H, self.KV, self.hd, self.F, self.V, self.theta, self.eps) = MODELS[model]
        self.n_layers = layers
        self.qd, self.kd = self.H * self.hd, self.KV * self.hd
        self.layer_params = self.d * (2 * self.qd + 2 * self.kd) + 3 * self.d * self.F


# --- the cases ---------------------------------------------------------------------------


def listed():
    tiny, seven = "tiny-llama-4L-d256", "llava-1.5-7b-shaped"
    thirteen, qwen = "llava-1.5-13b-shaped", "qwen2.5-vl-7b-shaped"
    return [
        # the smallest calls: a decode cycle of a toy model, all launches and latency
        dict(name="cycle-tiny", op="cycle", model=tiny, layers=4, batch=1, prefix=96,
             tree="static-14", temperature=0.0),
        # decoding without a draft: a root-only tree
        dict(name="step-7b", op="verify", model=seven, layers=4, batch=1, prefix=709, nodes=1,
             in_place=False),
        # one user, the 26-node static tree: the benchmark's verify, a block of it
        dict(name="verify-7b", op="verify", model=seven, layers=4, batch=1, prefix=650, nodes=27,
             in_place=False),
        # one user, a 60-node tree
        dict(name="verify-13b-tree61", op="verify", model=thirteen, layers=4, batch=1, prefix=911,
             nodes=61, in_place=False),
        # four users at once: the rows of several trees in one pass
        dict(name="verify-7b-batch4", op="verify", model=seven, layers=4, batch=4, prefix=650,
             nodes=27, in_place=False),
        # four users, grouped-query heads, large trees, a large vocabulary; the
        # caller keeps its row-major weights
        dict(name="verify-qwen-batch4", op="verify", model=qwen, layers=4, batch=4, prefix=1150,
             nodes=61, in_place=True),
        # the draft phase alone: a dynamic tree, six passes of the draft layer
        # and the large LM head
        dict(name="draft-qwen-dynamic", op="draft", model=qwen, layers=1, batch=1, prefix=1150,
             tree="dynamic-60"),
        # the whole decode cycle of the benchmark
        dict(name="cycle-7b-whole", op="cycle", model=seven, layers=32, batch=1, prefix=650,
             tree="static-26", temperature=0.0),
        # a short text-only turn
        dict(name="prefill-7b-short", op="prefill", model=seven, layers=4, rows=93, visual=0,
             in_place=False, feature=False),
        # the average multimodal prompt (576 visual rows), the whole model
        dict(name="prefill-7b-whole", op="prefill", model=seven, layers=32, rows=624, visual=576,
             in_place=True, feature=False),
        # a long visual prefix
        dict(name="prefill-7b-long", op="prefill", model=seven, layers=4, rows=3136, visual=2880,
             in_place=False, feature=False),
        # draft training on one sequence of that average length
        dict(name="train-7b", op="train", model=seven, layers=4, rows=640, visual=576),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    op = rng.choice(["verify", "verify", "verify", "draft", "cycle", "prefill", "prefill", "train"])
    model = rng.choice(sorted(MODELS))
    big = MODELS[model][1] > 2048
    layers = rng.randint(1, 4)
    if op == "verify":
        return dict(op=op, model=model, layers=layers, batch=rng.choice([1, 1, 2, 3, 4, 5, 8]),
                    prefix=_log_int(rng, 17, 3200 if big else 800),
                    nodes=rng.choice([1, 15, 27, 61, rng.randint(2, 64)]),
                    in_place=rng.random() < 0.4)
    tree = rng.choice(["static-14", "static-26", "dynamic-60", "dynamic-%d" % rng.randint(12, 63)])
    if op == "draft":
        return dict(op=op, model=model, layers=1, batch=rng.choice([1, 1, 2, 4]),
                    prefix=_log_int(rng, 17, 3200 if big else 800), tree=tree)
    if op == "cycle":
        return dict(op=op, model=model, layers=layers, batch=rng.choice([1, 1, 2, 4]),
                    prefix=_log_int(rng, 17, 3200 if big else 800), tree=tree,
                    temperature=rng.choice([0.0, 0.0, 0.7]))
    if op == "prefill":
        rows = _log_int(rng, 24, 3200 if big else 1200)
    else:
        rows = _log_int(rng, 48, 1100)
    visual = rng.choice([0, rows // 2, rows - 1 - rows // 10])
    if op == "prefill":
        return dict(op=op, model=model, layers=layers, rows=rows, visual=visual,
                    in_place=rng.random() < 0.5, feature=rng.random() < 0.25)
    return dict(op=op, model=model, layers=layers, rows=rows, visual=visual)


def draw(rng):
    top = [work(c) for c in listed()]
    flops, nbytes = max(w["flops"] for w in top), max(w["bytes"] for w in top)
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return case


# --- inputs ------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _normal(g, shape, sigma):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, sigma, generator=g)


def _ids(g, n, vocab):
    return torch.randint(0, vocab, (n,), generator=g, device="cuda").cpu().numpy().astype(np.int32)


def _layer(dims, g):
    d, F = dims.d, dims.F
    lw = {k: _normal(g, s, 0.02) for k, s in (
        ("wq", (dims.qd, d)), ("wk", (dims.kd, d)), ("wv", (dims.kd, d)), ("wo", (d, dims.qd)),
        ("w_gate", (F, d)), ("w_up", (F, d)), ("w_down", (d, F)))}
    for k in ("attn_norm", "ffn_norm"):
        lw[k] = 1.0 + _normal(g, (d,), 0.1)
    return lw


def _weights(dims, g):
    """Target of N(0, 0.02^2) matrices with norm gains near one; the draft head
    is a copy of the last layer behind an f_down that passes the feature
    through with a little noise, so that it agrees with the target at times."""
    w = {"embed": _normal(g, (dims.V, dims.d), 0.02), "lm_head": _normal(g, (dims.V, dims.d), 0.02),
         "final_norm": 1.0 + _normal(g, (dims.d,), 0.1),
         "layers": [_layer(dims, g) for _ in range(dims.n_layers)]}
    fc = _normal(g, (dims.d, 2 * dims.d), 0.004)
    i = torch.arange(dims.d, device="cuda")
    fc[i, i] += 1.0
    w["fc"], w["draft"] = fc, {k: v.clone() for k, v in w["layers"][-1].items()}
    return w


def _tree_nodes(tree):
    return int(tree.split("-")[1]) + 1


def _static_arrays(tree):
    paths = sorted(TREES[tree], key=lambda p: (len(p), p))
    index = {"": 0}
    for i, p in enumerate(paths, start=1):
        index[p] = i
    return [index[p[:-1]] for p in paths], [int(p[-1]) for p in paths], [len(p) for p in paths]


def _verify_trees(case, seed, vocab):
    """Random trees of `nodes` nodes, up to ten per depth, as msd_tree arrays."""
    r = np.random.default_rng(int(seed) + 3)
    T, trees = case["nodes"], []
    for _ in range(case["batch"]):
        token = r.choice(vocab, size=T, replace=False).astype(np.int32)
        parent, depth, level = [-1], [0], [0]
        while len(parent) < T:
            width = min(int(r.integers(3, 11)), T - len(parent))
            kids = list(range(len(parent), len(parent) + width))
            parent += sorted(int(p) for p in r.choice(level, size=width))
            depth += [depth[level[0]] + 1] * width
            level = kids
        trees.append((token, parent, depth))
    return trees


def _pack_trees(trees):
    raw = b""
    for token, parent, depth in trees:
        t = B.Tree()
        t.n_nodes = len(parent)
        anc = []
        for i, p in enumerate(parent):
            anc.append((anc[p] if p >= 0 else 0) | (1 << i))
            t.token[i], t.parent[i], t.depth[i], t.anc[i] = int(token[i]), p, depth[i], anc[i]
        raw += bytes(t)
    return torch.frombuffer(bytearray(raw), dtype=torch.uint8).cuda()


def _prompt(case, dims, g):
    n, nv = case["rows"], case["visual"]
    tokens = _ids(g, n, dims.V)
    is_visual = np.zeros(n, dtype=np.uint8)
    is_visual[:nv] = 1
    tokens[:nv] = 0
    return tokens, is_visual, _normal(g, (nv, dims.d), 1.0 / 64) if nv else None


def _inputs(case, seed):
    """The case's weights and call inputs, as plain tensors and arrays."""
    dims = Dims(case["model"], case["layers"])
    g = _gen(seed)
    s = {"dims": dims, "w": _weights(dims, g)}
    if case["op"] in ("prefill", "train"):
        s["prompt"] = _prompt(case, dims, g)
        return s
    nb, L = case["batch"], case["prefix"]
    s["kv"] = [_normal(g, (n, nb, dims.KV, L, dims.hd), 1.0)
               for n in (dims.n_layers, dims.n_layers, 1, 1)]
    if case["op"] == "verify":
        s["trees"] = _verify_trees(case, seed, dims.V)
    s["h"] = _normal(g, (nb, dims.d), 1.0)
    s["next"] = [int(t) for t in _ids(g, nb, dims.V)]
    return s


class _Session:
    """A context over device buffers, as a user's program holds it."""

    def __init__(self, dims, w, batch, max_seq, max_tree, max_prompt):
        desc = B.ModelDesc(dims.n_layers, dims.d, dims.H, dims.KV, dims.hd, dims.F, dims.V,
                           dims.theta, dims.eps)
        lim = B.Limits(batch, max_seq, max_tree, max_prompt)
        names = [n for n, _ in B.LayerWeights._fields_]
        layers = (B.LayerWeights * dims.n_layers)(
            *[B.LayerWeights(*[lw[n].data_ptr() for n in names]) for lw in w["layers"]])
        tw = B.TargetWeights(w["embed"].data_ptr(), layers, w["final_norm"].data_ptr(),
                             w["lm_head"].data_ptr())
        dw = B.DraftWeights(w["fc"].data_ptr(),
                            B.LayerWeights(*[w["draft"][n].data_ptr() for n in names]))
        tkv, dkv, ws, pw = B.msd_buffer_sizes(desc, lim)
        self.ctx = None
        self.bufs = [torch.empty(n, dtype=torch.uint8, device="cuda")
                     for n in (tkv, tkv, dkv, dkv, ws, pw)]
        self.w, self.layers = w, layers
        self.ctx = B.msd_create(desc, lim, tw, dw, B.Buffers(*[b.data_ptr() for b in self.bufs]),
                                torch.cuda.current_stream().cuda_stream)
        self.kv = []
        for i, nl in enumerate((dims.n_layers, dims.n_layers, 1, 1)):
            shape = (nl, batch, dims.KV) + ((max_seq, dims.hd) if i % 2 == 0 else (dims.hd, max_seq))
            self.kv.append(self.bufs[i].view(torch.bfloat16).view(shape))

    def __del__(self):
        if self.ctx:
            B.msd_destroy(self.ctx)


def _spec(tree):
    if tree.startswith("static"):
        parent, rank, _ = _static_arrays(tree)
        return B.make_static_spec(parent, rank)
    return B.make_dynamic_spec(DYN_TOPK, DYN_DEPTH, _tree_nodes(tree) - 1)


def prepare(case, seed):
    s = _inputs(case, seed)
    dims = s["dims"]
    st = {"op": case["op"], "case": case, "dims": dims}
    if case["op"] in ("prefill", "train"):
        n = case["rows"]
        e = _Session(dims, s["w"], 1, (n + 64 + 63) // 64 * 64, 64, n)
        st["prompt"] = s["prompt"]
        if case["op"] == "prefill":
            B.msd_use_caller_weights(e.ctx, case["in_place"])
            B.msd_set_draft_input(e.ctx, 1 if case["feature"] else 0)
        else:
            d, F = dims.d, dims.F
            n_par = 2 * d * d + dims.layer_params + 2 * d
            st["grads"] = torch.empty(n_par, dtype=torch.float32, device="cuda")
            # the trainer's state exists before its first step
            B.msd_train_read(e.ctx, 0, st["grads"].data_ptr(), n_par)
    else:
        nb, L = case["batch"], case["prefix"]
        T = case["nodes"] if case["op"] == "verify" else _tree_nodes(case["tree"])
        e = _Session(dims, s["w"], nb, (L + 128 + 63) // 64 * 64, 64, max(L, 8))
        if case.get("in_place"):
            B.msd_use_caller_weights(e.ctx, True)
        for i in range(4):
            if i % 2 == 0:
                e.kv[i][:, :, :, :L] = s["kv"][i]
            else:
                e.kv[i][:, :, :, :, :L] = s["kv"][i].transpose(3, 4)
        st["h"], st["next"], st["T"], st["seqs"] = s["h"], s["next"], T, list(range(nb))
        for b in range(nb):
            B.msd_set_state(e.ctx, b, L, s["h"][b].data_ptr(), s["next"][b])
        if case["op"] == "verify":
            st["trees"] = _pack_trees(s["trees"])
        else:
            st["spec"] = _spec(case["tree"])
            st["trees"] = torch.zeros(nb * ctypes.sizeof(B.Tree), dtype=torch.uint8, device="cuda")
        if case["op"] != "draft":
            st["argmax"] = torch.empty(nb * T, dtype=torch.int32, device="cuda")
            st["logits"] = torch.empty(nb * T, dims.V, dtype=torch.float32, device="cuda")
    st["session"] = e
    torch.cuda.synchronize()
    return st


def _draft_rows(tree):
    """Draft cache slots a tree's expansions take."""
    if tree.startswith("static"):
        parent, _, depth = _static_arrays(tree)
        return len({p for p in parent if p > 0})
    return DYN_TOPK * (DYN_DEPTH - 1)


def _draft_out(st):
    nb, L, T = len(st["seqs"]), st["case"]["prefix"], st["T"]
    words = st["trees"].view(nb, ctypes.sizeof(B.Tree))
    out = {"token": words.view(torch.int32)[:, 1:1 + T]}
    if st["case"]["tree"].startswith("dynamic"):
        o = B.Tree.score.offset // 4
        out["score"] = words.view(torch.float32)[:, o + 1:o + T]
    r = _draft_rows(st["case"]["tree"])
    _, _, dk, dv = st["session"].kv
    out["draft_k"], out["draft_v"] = dk[0, :, :, L - 1:L + r], dv[0, :, :, :, L - 1:L + r]
    return out


def run(st):
    c, op, ctx = st["case"], st["op"], st["session"].ctx
    if op == "verify":
        B.msd_verify(ctx, st["seqs"], st["trees"].data_ptr(), st["T"], st["argmax"].data_ptr(),
                     st["logits"].data_ptr())
        return {"logits": st["logits"], "argmax": st["argmax"]}
    if op in ("draft", "cycle"):
        for b in st["seqs"]:
            B.msd_set_state(ctx, b, c["prefix"], st["h"][b].data_ptr(), st["next"][b])
        B.msd_draft_tree(ctx, st["seqs"], st["spec"], st["trees"].data_ptr())
        if op == "draft":
            return _draft_out(st)
        B.msd_verify(ctx, st["seqs"], st["trees"].data_ptr(), st["T"], st["argmax"].data_ptr(),
                     st["logits"].data_ptr())
        if c["temperature"] > 0:
            B.msd_accept_sample(ctx, st["seqs"], st["trees"].data_ptr(), st["T"],
                                st["logits"].data_ptr(), c["temperature"], 7)
        else:
            B.msd_accept_compact(ctx, st["seqs"], st["trees"].data_ptr(), st["T"],
                                 st["argmax"].data_ptr())
        return {**_draft_out(st), "logits": st["logits"]}
    tokens, is_visual, visual = st["prompt"]
    vptr = visual.data_ptr() if visual is not None else None
    if op == "prefill":
        first = B.msd_prefill(ctx, 0, tokens, is_visual, vptr)
        tk, tv, dk, dv = st["session"].kv
        n = c["rows"]
        out = {"k": tk[:, 0, :, :n], "v": tv[:, 0, :, :, :n], "draft_k": dk[0, 0, :, :n],
               "draft_v": dv[0, 0, :, :, :n]}
        return {**out, "first": first} if c["layers"] <= 4 else out
    loss = B.msd_train_accumulate(ctx, 0, tokens, is_visual, vptr)
    g = st["grads"]
    B.msd_train_read(ctx, 0, g.data_ptr(), g.numel())
    B.msd_train_apply(ctx, LR)
    return {"loss": list(loss), "grads": g}


# --- work and tolerances -----------------------------------------------------------------


def _stack_work(dims, layers, rows, keys, with_head):
    """(bytes, flops) of `layers` layers over `rows` rows, each against `keys`
    cache slots per row (their bytes counted once per sequence by the caller)."""
    p = layers * dims.layer_params + (dims.V * dims.d if with_head else 0)
    attn = 4 * layers * rows * keys * dims.qd
    return 2 * p, 2 * rows * p + attn


def work(case):
    dims = Dims(case["model"], case["layers"])
    d, nl, kvb = dims.d, dims.n_layers, 4 * dims.kd  # bytes of one slot's K and V, one layer
    op = case["op"]
    nbytes = flops = 0
    if op in ("verify", "cycle"):
        nb, L = case["batch"], case["prefix"]
        T = case["nodes"] if op == "verify" else _tree_nodes(case["tree"])
        by, fl = _stack_work(dims, nl, nb * T, L + T / 2, True)
        nbytes += by + nb * (L + T) * nl * kvb + nb * T * (2 * d + 4 * dims.V)
        flops += fl
    if op in ("draft", "cycle"):
        nb, L = case["batch"], case["prefix"]
        rows = nb * (1 + _draft_rows(case["tree"]))
        static = case["tree"].startswith("static")
        passes = 1 + (max(_static_arrays(case["tree"])[2]) if static else DYN_DEPTH) - 1
        by, fl = _stack_work(dims, 1, rows, L, True)
        # f_down, the draft layer and the LM head are read in every pass
        nbytes += passes * (by + 4 * d * d + nb * L * kvb)
        flops += fl + 4 * rows * d * d
    if op in ("prefill", "train"):
        n = case["rows"]
        by, fl = _stack_work(dims, nl, n, n / 2, False)
        nbytes += by + n * (2 * d + nl * kvb)
        flops += fl
    if op == "prefill":
        by, fl = _stack_work(dims, 1, n, n / 2, False)
        nbytes += by + 4 * d * d + 2 * dims.V * d + n * kvb
        flops += fl + 4 * n * d * d + 2 * dims.V * d
    if op == "train":
        R = n - 1
        mats = 2 * R * (2 * d * d + dims.layer_params)
        attn = 2 * R * R * dims.qd
        flops += 3 * mats + 3 * attn + 3 * 2 * R * dims.V * d
        # float32 masters and moments read and written, gradients written and read
        nbytes += 2 * dims.V * d + (2 * d * d + dims.layer_params) * (3 * 8 + 2 + 3 * 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Each is about four times what the path shows against the 64-bit references
    # below.  Activations travel as bf16 pairs (about 17 bits) and the caches are
    # bf16: a value near a rounding boundary moves a cached key by up to 2^-8 of
    # itself, and that travels through the layers that follow.
    whole = case["layers"] > 4
    if case["op"] in ("verify", "cycle"):
        return {"rel": 5e-3 if whole else 2e-3, "max": 5e-2, "differ": 0.01}
    if case["op"] == "draft":
        return {"rel": 2e-3, "max": 5e-2, "differ": 0.01}
    if case["op"] == "prefill":
        return {"rel": 8e-3 if whole else 5e-3, "max": 0.1, "differ": 0.0}
    return {"rel": 1e-3, "max": 5e-2}


# --- 64-bit references -------------------------------------------------------------------


def _bf16(x):
    """What a bf16 cache holds of x."""
    return x.float().bfloat16().double()


def _mm(x, w):
    return x @ w.double().t()


def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, hd, theta):
    half = hd // 2
    inv = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / hd)
    ang = pos.double()[:, None] * inv
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    y = x.view(x.shape[0], -1, hd)
    a, b = y[..., :half], y[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(dims, q, kp, vp, k, v, see):
    """q [T,H,hd]; prefix kp, vp [KV,L,hd] (or None); the rows' own k, v
    [T,KV,hd], row i seeing row j where see[i,j]."""
    T, g, out = q.shape[0], dims.H // dims.KV, []
    for h in range(dims.KV):
        qh = q[:, h * g:(h + 1) * g].reshape(T * g, dims.hd)
        keys, vals = k[:, h], v[:, h]
        mask = see.repeat_interleave(g, 0)
        if kp is not None:
            keys = torch.cat([kp[h].double(), keys])
            vals = torch.cat([vp[h].double(), vals])
            mask = torch.cat([mask.new_ones(T * g, kp.shape[1]), mask], 1)
        s = (qh @ keys.t()) / math.sqrt(dims.hd)
        p = torch.softmax(s.masked_fill(~mask, -math.inf), -1)
        out.append((p @ vals).view(T, g, dims.hd))
    return torch.cat(out, 1).reshape(T, dims.qd)


def _layer_exact(dims, lw, x, pos, attend, cache=_bf16):
    """One decoder layer; attend(q, k, v) with the keys and values as cached.
    Returns (new rows, k, v)."""
    a = _norm(x, lw["attn_norm"], dims.eps)
    q = _rope(_mm(a, lw["wq"]), pos, dims.hd, dims.theta)
    k = cache(_rope(_mm(a, lw["wk"]), pos, dims.hd, dims.theta))
    v = cache(_mm(a, lw["wv"]).view(-1, dims.KV, dims.hd))
    x = x + _mm(attend(q, k, v), lw["wo"])
    a = _norm(x, lw["ffn_norm"], dims.eps)
    gate = _mm(a, lw["w_gate"])
    return x + _mm(gate * torch.sigmoid(gate) * _mm(a, lw["w_up"]), lw["w_down"]), k, v


def _tree_exact(dims, w, kv, b, L, token, parent, depth):
    """Logits of one tree's nodes."""
    T = len(parent)
    see = torch.zeros(T, T, dtype=torch.bool, device="cuda")
    for i in range(T):
        if parent[i] >= 0:
            see[i] = see[parent[i]]
        see[i, i] = True
    pos = L + torch.tensor(depth, device="cuda")
    x = w["embed"][torch.tensor(np.asarray(token, dtype=np.int64), device="cuda")].double()
    for l, lw in enumerate(w["layers"]):
        x, _, _ = _layer_exact(dims, lw, x, pos, lambda q, k, v: _attend(
            dims, q, kv[0][l, b], kv[1][l, b], k, v, see))
    return _mm(_norm(x, w["final_norm"], dims.eps), w["lm_head"])


class _DraftExact:
    """The draft head of one sequence: its cache prefix [0, L-1), the pending
    row at L-1, then expanded nodes at L, L+1, ..."""

    def __init__(self, dims, w, kv, b, L, h, nxt):
        self.dims, self.w, self.L = dims, w, L
        self.kp, self.vp = kv[2][0, b, :, :L - 1], kv[3][0, b, :, :L - 1]
        self.k, self.v, self.seen = [], [], {}
        self.feat = {None: self._pass(h.double()[None], [nxt], [L - 1], [[0]])[0]}

    def _pass(self, h, tokens, pos, sees):
        """sees[i]: the rows of self.k (this pass's included) that row i sees."""
        dims, w, n0, n = self.dims, self.w, len(self.k), len(tokens)
        e = w["embed"][torch.tensor(tokens, device="cuda")].double()
        x = _mm(torch.cat([h, e], 1), w["fc"])

        def attend(q, k, v):
            self.k += list(k)
            self.v += list(v)
            see = torch.zeros(n, n0 + n, dtype=torch.bool, device="cuda")
            for i, s in enumerate(sees):
                see[i, s] = True
            return _attend(dims, q, self.kp, self.vp, torch.stack(self.k), torch.stack(self.v), see)

        x, _, _ = _layer_exact(dims, w["draft"], x, torch.tensor(pos, device="cuda"), attend)
        return x

    def expand(self, keys, parents, tokens, depth):
        """Features of nodes `keys` of one depth; returns their logits rows."""
        sees = []
        for j, (key, par) in enumerate(zip(keys, parents)):
            self.seen[key] = (self.seen[par] if par is not None else [0]) + [len(self.k) + j]
            sees.append(self.seen[key])
        h = torch.stack([self.feat[p] for p in parents])
        out = self._pass(h, tokens, [self.L + depth - 1] * len(keys), sees)
        for j, key in enumerate(keys):
            self.feat[key] = out[j]
        return _mm(out, self.w["lm_head"])


def _draft_tree_exact(tree, ex, root):
    """(tokens, parents, depths, scores) of the tree that the draft builds."""
    logits = _mm(ex.feat[None][None], ex.w["lm_head"])
    if tree.startswith("static"):
        parent, rank, depth = ([-1] + v if i == 0 else [0] + v
                               for i, v in enumerate(_static_arrays(tree)))
        token, rows = [root] + [0] * (len(parent) - 1), {0: logits[0]}
        for dd in range(max(depth)):
            if dd:
                nodes = [u for u in range(len(parent)) if depth[u] == dd and u in parent]
                got = ex.expand(nodes, [parent[u] or None for u in nodes],
                                [token[u] for u in nodes], dd)
                rows = dict(zip(nodes, got))
            for c in range(1, len(parent)):
                if parent[c] in rows and depth[c] == dd + 1:
                    token[c] = int(torch.topk(rows[parent[c]], 16).indices[rank[c]])
        return token, parent, depth, None
    K, pool = DYN_TOPK, []  # (parent in pool or None, token, depth, score)

    def children(par, row, dep, base):
        lp = torch.log_softmax(row, -1)
        top = torch.topk(lp, K)
        for t, s in zip(top.indices.tolist(), top.values.tolist()):
            pool.append((par, t, dep, base + s))

    children(None, logits[0], 1, 0.0)
    front = list(range(K))
    for dep in range(2, DYN_DEPTH + 1):
        rows = ex.expand(front, [pool[u][0] for u in front], [pool[u][1] for u in front], dep - 1)
        first = len(pool)
        for j, u in enumerate(front):
            children(u, rows[j], dep, pool[u][3])
        front = sorted(sorted(range(first, len(pool)), key=lambda i: (-pool[i][3], i))[:K])
    keep = sorted(range(len(pool)), key=lambda i: (-pool[i][3], i))[:_tree_nodes(tree) - 1]
    keep.sort(key=lambda i: (pool[i][2], i))
    index = {None: 0, **{i: j for j, i in enumerate(keep, start=1)}}
    return ([root] + [pool[i][1] for i in keep], [-1] + [index[pool[i][0]] for i in keep],
            [0] + [pool[i][2] for i in keep], [pool[i][3] for i in keep])


def _prompt_exact(dims, w, prompt):
    """(input rows, features, [k of every layer], [v of every layer])."""
    tokens, is_visual, visual = prompt
    n = len(tokens)
    x = w["embed"][torch.tensor(tokens.astype(np.int64), device="cuda")].double()
    if visual is not None:
        x[:visual.shape[0]] = visual.double()
    e, see = x.clone(), torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
    pos = torch.arange(n, device="cuda")
    ks, vs = [], []
    for lw in w["layers"]:
        x, k, v = _layer_exact(dims, lw, x, pos,
                               lambda q, k, v: _attend(dims, q, None, None, k, v, see))
        ks.append(k)
        vs.append(v)
    return e, _norm(x, w["final_norm"], dims.eps), ks, vs


def _train_exact(dims, s):
    w, (tokens, is_visual, _) = s["w"], s["prompt"]
    e, h, _, _ = _prompt_exact(dims, w, s["prompt"])
    R = len(tokens) - 1
    names = [n for n, _ in B.LayerWeights._fields_]
    p = {"fc": w["fc"], **{n: w["draft"][n] for n in names}}
    p = {n: v.double().requires_grad_() for n, v in p.items()}
    vis = torch.tensor(is_visual[:R] != 0, device="cuda")[:, None]
    x = torch.where(vis, e[:R], torch.cat([h[:R], e[1:]], 1) @ p["fc"].t())
    see = torch.ones(R, R, dtype=torch.bool, device="cuda").tril()
    x, _, _ = _layer_exact(dims, p, x, torch.arange(R, device="cuda"), lambda q, k, v: _attend(
        dims, q, None, None, k, v, see), cache=lambda t: t)
    diff = x - h[1:]
    ad = diff.abs()
    reg = torch.where(ad < 1, 0.5 * diff * diff, ad - 0.5).mean(1).sum()
    ce = -(torch.softmax(_mm(h[1:], w["lm_head"]), -1)
           * torch.log_softmax(_mm(x, w["lm_head"]), -1)).sum()
    loss = reg + 0.1 * ce
    loss.backward()
    grads = torch.cat([p[n].grad.reshape(-1) for n in ["fc"] + names])
    return {"loss": [float(loss), float(reg), float(ce)], "grads": grads}


def exact(case, seed):
    s = _inputs(case, seed)
    dims, w, op = s["dims"], s["w"], case["op"]
    if op == "train":
        return _train_exact(dims, s)
    with torch.no_grad():
        if op == "verify":
            L = case["prefix"]
            logits = torch.cat([_tree_exact(dims, w, s["kv"], b, L, *t)
                                for b, t in enumerate(s["trees"])])
            return {"logits": logits, "argmax": logits.argmax(-1)}
        if op in ("draft", "cycle"):
            out = {"token": [], "score": [], "draft_k": [], "draft_v": [], "logits": []}
            for b in range(case["batch"]):
                L = case["prefix"]
                ex = _DraftExact(dims, w, s["kv"], b, L, s["h"][b], s["next"][b])
                token, parent, depth, score = _draft_tree_exact(case["tree"], ex, s["next"][b])
                out["token"].append(torch.tensor(token))
                if score is not None:
                    out["score"].append(torch.tensor(score, dtype=torch.float64))
                out["draft_k"].append(torch.stack(ex.k, 1))
                out["draft_v"].append(torch.stack(ex.v, 1).transpose(1, 2))
                if op == "cycle":
                    out["logits"].append(_tree_exact(dims, w, s["kv"], b, L, token, parent, depth))
            cat = {"logits"}
            return {k: torch.cat(v) if k in cat else torch.stack(v) for k, v in out.items() if v}
        e, h, ks, vs = _prompt_exact(dims, w, s["prompt"])
        tokens, is_visual, _ = s["prompt"]
        first = int(_mm(h[-1:], w["lm_head"]).argmax())
        vis = torch.tensor(is_visual != 0, device="cuda")[:, None]
        nxt = torch.cat([e[1:], w["embed"][first:first + 1].double()])
        x = torch.where(vis, h if case["feature"] else e, _mm(torch.cat([h, nxt], 1), w["fc"]))
        n = len(tokens)
        see = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
        _, dk, dv = _layer_exact(dims, w["draft"], x, torch.arange(n, device="cuda"),
                                 lambda q, k, v: _attend(dims, q, None, None, k, v, see))
        out = {"k": torch.stack(ks).transpose(1, 2), "v": torch.stack(vs).permute(0, 2, 3, 1),
               "draft_k": dk.transpose(0, 1), "draft_v": dv.permute(1, 2, 0)}
        return {**out, "first": first} if case["layers"] <= 4 else out
