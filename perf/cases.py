"""The work that users of this library have it do, as cases that can be prepared, run, checked and timed one at a time.

Two kinds of call make up a decoding step, and each has its cases: the forward pass of one model over the new rows of
a block (then the rollback of its cache), and the acceptance of the drafted tokens.  The forward cases are stacks of
one or two decoder layers of the model shapes in synth.py (embedding and head included, since every call has them);
one case is a whole 32-layer model.  Weights, cache contents, tokens and logits are drawn as synth.py draws them.
"""
import numpy as np
import torch

import paper_2510_26527_amd as psd
from paper_2510_26527_amd import runtime, synth

SHAPES = {"llama2_7b": synth.LLAMA2_7B, "llama3_8b": synth.LLAMA3_8B, "qwen2_7b": synth.QWEN2_7B,
          "chain_intermediate": synth.CHAIN_INTERMEDIATE, "chain_draft": synth.CHAIN_DRAFT}


# ---------------------------------------------------------------------------------------------------- the cases
def _forward(name, model, layers, batch, n_new, ctx, logit_rows, packed=True, w4=False, ragged=False, branch=0):
    return {"name": name, "kind": "forward", "model": model, "layers": layers, "batch": batch, "n_new": n_new, "ctx": ctx,
            "logit_rows": logit_rows, "packed": packed, "w4": w4, "ragged": ragged, "branch": branch}


def _accept(name, rows, gamma, vocab, dtype, bonus, temperature=1.0):
    return {"name": name, "kind": "accept", "rows": rows, "gamma": gamma, "vocab": vocab, "dtype": dtype, "bonus": bonus,
            "temperature": temperature}


def _tree_accept(name, rows, nodes, branch, vocab, dtype, temperature=1.0):
    return {"name": name, "kind": "tree_accept", "rows": rows, "nodes": nodes, "branch": branch, "vocab": vocab,
            "dtype": dtype, "temperature": temperature}


def listed():
    return [
        # one autoregressive step of a chain's one-layer draft model: the smallest forward, called most often
        _forward("draft_step", "chain_draft", 1, 1, 1, 389, 1),
        # the target's verify step of a chain: gamma + 1 = 11 rows, grouped-query heads, all rows with logits
        _forward("verify_gqa_11", "llama3_8b", 2, 1, 11, 521, 11),
        # the same step on the 4-bit copy that serves as the chain's intermediate level
        _forward("verify_w4_7", "llama3_8b", 2, 1, 7, 300, 7, w4=True),
        # a small serving batch: five sequences of different lengths, nine rows each
        _forward("verify_batch_5x9", "llama2_7b", 2, 5, 9, 1024, 9, ragged=True),
        # a large serving batch on long caches, row-major weights only
        _forward("verify_batch_16x16", "qwen2_7b", 2, 16, 16, 4096, 16, packed=False),
        # a prompt: many rows at once, an odd number of them, logits for the last only
        _forward("prefill_2001", "llama2_7b", 2, 1, 2001, 0, 1),
        # a drafted token tree: forward over its nodes, then the accepted path's rows move together
        _forward("tree_15", "llama2_7b", 2, 1, 15, 1024, 15, branch=2),
        # a whole model's verify step, the benchmark's headline
        _forward("whole_7b_8", "llama2_7b", 32, 1, 8, 1024, 8),
        # acceptance of one sequence's block by the logits a forward pass has just written (fp32, with the bonus row)
        _accept("accept_1x8", 1, 8, 32000, "float32", True),
        # acceptance for a batch of sequences on logits kept in bf16
        _accept("accept_64x8", 64, 8, 32000, "bfloat16", False),
        # acceptance for a serving batch with a large vocabulary
        _accept("accept_16x16", 16, 16, 152064, "float32", True),
        # acceptance down a token tree, a few sequences at a time
        _tree_accept("tree_accept_4x15", 4, 15, 2, 32000, "float32"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["verify", "verify", "batch", "batch", "prefill", "tree", "accept", "accept", "accept", "tree_accept"])
    if kind == "verify":
        model = rng.choice(["llama2_7b", "llama3_8b", "llama3_8b", "chain_intermediate", "chain_draft"])
        n = rng.randint(1, 16)
        c = _forward("", model, rng.randint(1, 2), 1, n, _log(rng, 40, 4000), n, w4=model == "llama3_8b" and rng.random() < 0.4)
    elif kind == "batch":
        model = rng.choice(["llama2_7b", "llama3_8b", "qwen2_7b"])
        b, n = rng.randint(2, 16), rng.randint(2, 16)
        w4 = model == "llama3_8b" and rng.random() < 0.25
        c = _forward("", model, rng.randint(1, 2), b, n, _log(rng, 40, 2000), n, packed=w4 or rng.random() < 0.5, w4=w4,
                     ragged=rng.random() < 0.7)
    elif kind == "prefill":
        model = rng.choice(["llama2_7b", "llama3_8b", "qwen2_7b"])
        most = {"llama2_7b": 1800, "llama3_8b": 1000, "qwen2_7b": 580}[model]     # query rows per KV head are limited
        c = _forward("", model, rng.randint(1, 2), 1, _log(rng, 40, most), rng.choice([0, 0, _log(rng, 40, 1000)]), 1)
    elif kind == "tree":
        model = rng.choice(["llama2_7b", "llama3_8b"])
        n = rng.randint(3, 32) if model == "llama2_7b" else rng.randint(3, 8)
        c = _forward("", model, rng.randint(1, 2), rng.randint(1, 2), n, _log(rng, 40, 2000), n, branch=rng.randint(1, 4))
    elif kind == "accept":
        gamma = rng.randint(0, 16)
        c = _accept("", _log(rng, 1, 64) if gamma <= 8 else _log(rng, 1, 16), gamma, rng.choice([32000, 128256, 152064, _log(rng, 1000, 100000)]),
                    rng.choice(["float32", "bfloat16"]), gamma == 0 or rng.random() < 0.6, rng.choice([1.0, 1.0, 0.7, 0.0]))
        if c["rows"] * max(1, gamma) * c["vocab"] > 16 * 16 * 152064:
            c["vocab"] = 32000
    else:
        c = _tree_accept("", _log(rng, 1, 16), rng.randint(2, 32), rng.randint(1, 4), rng.choice([32000, _log(rng, 1000, 60000)]),
                         rng.choice(["float32", "bfloat16"]), rng.choice([1.0, 1.0, 0.7, 0.0]))
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------- inputs
def _shape(case):
    s = SHAPES[case["model"]]
    return synth.Shape(case["layers"], s.d_model, s.n_q_heads, s.n_kv_heads, s.d_head, s.d_ffn, s.vocab, s.rope_theta, s.rms_eps)


def _parents(n, branch):
    return [-1] + [(i - 1) // branch for i in range(1, n)]


def _path(case, seed):
    """An accepted root-to-node path (root excluded) of the case's tree, as an acceptance call would return it."""
    parents, rng = _parents(case["n_new"], case["branch"]), np.random.default_rng(seed)
    node, path = int(rng.integers(case["n_new"] // 2, case["n_new"])), []
    while node > 0:
        path.append(node)
        node = parents[node]
    return path[::-1]


def _forward_inputs(case, seed):
    """(weights, quant, keys, values, lens, tokens): keys / values per layer [batch, n_kv_heads, ctx, d_head] bf16."""
    shape, dev = _shape(case), "cuda"
    weights, quant = synth.make_weights(shape, 7 * seed + 1, torch.bfloat16, device=dev), None
    if case["w4"]:
        weights, quant = synth.quantize_w4(weights)
    ks, vs = synth.make_kv_fill(shape, case["batch"], case["ctx"], 7 * seed + 2, torch.bfloat16, device=dev) if case["ctx"] else ([], [])
    lens = np.full(case["batch"], case["ctx"], np.int64)
    if case["ragged"]:
        lens -= np.random.default_rng(7 * seed + 3).integers(0, max(1, case["ctx"] // 2), case["batch"])
    tokens = torch.from_numpy(synth.make_tokens(shape.vocab, (case["batch"], case["n_new"]), 7 * seed + 4)).to(dev)
    return weights, quant, ks, vs, lens.tolist(), tokens


def _accept_inputs(case, seed):
    dtype = getattr(torch, case["dtype"])
    if case["kind"] == "accept":
        if case["gamma"] == 0:                      # plain sampling from one row per sequence
            gen = torch.Generator(device="cuda").manual_seed(seed)
            p = torch.empty((case["rows"], 1, case["vocab"]), device="cuda").normal_(0.0, 2.0, generator=gen).to(dtype)
            return {"p": p, "q": None, "tokens": None, "uniforms": synth.make_uniforms((case["rows"], 1), seed + 1, "cuda")}
        return synth.make_accept_inputs(case["rows"], case["gamma"], case["vocab"], seed, case["gamma"] + int(case["bonus"]),
                                        dtype=dtype, device="cuda")
    rows, n, V = case["rows"], case["nodes"], case["vocab"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.empty((rows, n, V), device="cuda").normal_(0.0, 2.0, generator=gen)
    q = (p + torch.empty_like(p).normal_(0.0, 0.5, generator=gen)).to(dtype)
    tokens = torch.zeros((rows, n), dtype=torch.int32, device="cuda")
    for i, parent in enumerate(_parents(n, case["branch"])):
        if parent >= 0:                             # a draw from the drafter's row at the parent (Gumbel-max)
            g = torch.empty((rows, V), device="cuda").exponential_(1.0, generator=gen)
            tokens[:, i] = torch.argmax(q[:, parent].float() - torch.log(g), dim=-1).to(torch.int32)
    return {"p": p.to(dtype), "q": q, "tokens": tokens, "uniforms": synth.make_uniforms((rows, n + 1), seed + 1, "cuda")}


class State:
    pass


def prepare(case, seed):
    s = State()
    s.case = case
    if case["kind"] != "forward":
        s.inputs = _accept_inputs(case, seed)
        s.acceptor = runtime.Acceptor("cuda")
        s.parents = _parents(case["nodes"], case["branch"]) if case["kind"] == "tree_accept" else None
        return s
    shape = _shape(case)
    weights, quant, ks, vs, lens, s.tokens = _forward_inputs(case, seed)
    s.model = runtime.Model(shape, weights, "cuda", quant=quant)
    if case["packed"]:
        s.model.pack()
    n = case["n_new"]
    max_len = (case["ctx"] + n + 63) // 64 * 64
    s.kv = runtime.KVCache(s.model, case["batch"], max_len)
    s.kv.k.zero_()
    s.kv.v.zero_()
    if case["ctx"]:
        s.kv.load(ks, vs, lens)
    s.bound = max(lens)
    s.base = torch.tensor(lens, dtype=torch.int32, device="cuda")
    s.keep = torch.zeros(case["batch"], dtype=torch.int32, device="cuda")
    s.logits = torch.empty((case["batch"], case["logit_rows"], shape.vocab), dtype=torch.float32, device="cuda")
    # what a pass writes into the cache: the new rows of every sequence, where they are stored
    s.k_new = [s.kv.k[:, b, :, l:l + n] for b, l in enumerate(lens)]
    s.v_new = [s.kv.v[:, b, :, :, l:l + n] for b, l in enumerate(lens)]
    if case["branch"]:
        s.parents = _parents(n, case["branch"])
        path = _path(case, seed)
        s.path = torch.tensor([path + [-1] * (n - len(path))] * case["batch"], dtype=torch.int32, device="cuda")
        s.path_len = torch.full((case["batch"],), len(path), dtype=torch.int32, device="cuda")
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s.case
    if case["kind"] == "accept":
        x = s.inputs
        return s.acceptor(x["p"], x["q"], x["tokens"], x["uniforms"], case["temperature"])
    if case["kind"] == "tree_accept":
        x = s.inputs
        return runtime.tree_accept(x["p"], x["q"], x["tokens"], s.parents, x["uniforms"], case["temperature"])
    if case["branch"]:
        runtime.forward_tree(s.model, s.kv, s.tokens, s.parents, logits_out=s.logits)
        psd.psd_kv_compact_tree(s.kv.handle, s.base, s.path, s.path_len, case["n_new"], case["n_new"])
    else:
        runtime.forward(s.model, s.kv, s.tokens, n_logit_rows=case["logit_rows"], logits_out=s.logits)
    psd.psd_kv_truncate(s.kv.handle, s.base, s.keep, 0, s.bound)      # the block is refused: back to the old lengths
    return {"logits": s.logits, "k": s.k_new, "v": s.v_new, "lens": s.kv.lens}


# ---------------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    if case["kind"] == "accept":
        size = 4 if case["dtype"] == "float32" else 2
        p_rows, q_rows = case["gamma"] + int(case["bonus"]), case["gamma"] if case["temperature"] > 0 else 0
        n = case["rows"] * case["vocab"] * (p_rows + q_rows)
        return {"bytes": n * size, "flops": 4 * n}
    if case["kind"] == "tree_accept":               # the root's two rows at least; how far a walk gets is up to the draws
        size = 4 if case["dtype"] == "float32" else 2
        n = case["rows"] * case["vocab"] * (2 if case["temperature"] > 0 else 1)
        return {"bytes": n * size, "flops": 4 * n}
    s, B, R = _shape(case), case["batch"], case["n_new"]
    hd, kvd = s.n_q_heads * s.d_head, s.n_kv_heads * s.d_head
    proj = s.n_layers * (s.d_model * (hd + 2 * kvd) + hd * s.d_model + 3 * s.d_model * s.d_ffn)
    head = s.vocab * s.d_model
    wbytes = proj * (0.5 + 3 / 128 if case["w4"] else 2) + head * 2
    cache = s.n_layers * B * 2 * kvd * 2 * (case["ctx"] + R)
    keys = case["ctx"] * R + R * (R + 1) / 2        # (query, key) pairs of one head of one sequence
    return {"bytes": wbytes + cache + B * R * s.d_model * 2 + 4 * B * case["logit_rows"] * s.vocab,
            "flops": 2.0 * B * (R * proj + case["logit_rows"] * head) + 4.0 * s.n_layers * B * hd * keys}


def tolerance(case):
    if case["kind"] != "forward":
        return "exact"                              # accepted lengths, tokens, flags: decided in 64 bits
    # four times the error against exact(): the rounding of the new keys and values to bf16 (2e-3) in one or two layers,
    # what 32 layers make of it (4e-3), and a prompt's last row (6e-3)
    if case["n_new"] > 32:
        return {"rel": 2.4e-2}
    return {"rel": 1.6e-2 if case["layers"] > 2 else 8e-3}


# ---------------------------------------------------------------------------------------------------- in 64 bits
def _dequant(weights, quant, name):
    w = weights[name]
    if not quant or name not in quant:
        return w.double()
    scale, zero = quant[name]
    q = torch.stack([w & 15, w >> 4], dim=-1).reshape(w.shape[0], -1).double()
    return (q.reshape(w.shape[0], -1, 128) - zero.double()[..., None]).mul_(scale.double()[..., None]).reshape(w.shape[0], -1)


def _norm(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, theta):
    """x [B, R, heads, d_head], pos [B, R]"""
    half = x.shape[-1] // 2
    freq = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[-1])
    ang = (pos.double()[..., None] * freq)[:, :, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * torch.cos(ang) - b * torch.sin(ang), b * torch.cos(ang) + a * torch.sin(ang)], dim=-1)


def exact(case, seed):
    if case["kind"] != "forward":
        return None                                 # whole numbers
    s, B, R = _shape(case), case["batch"], case["n_new"]
    weights, quant, ks, vs, lens, tokens = _forward_inputs(case, seed)
    w = lambda name: _dequant(weights, quant, name)
    dev, group = tokens.device, s.n_q_heads // s.n_kv_heads
    pos = torch.tensor(lens, device=dev)[:, None] + torch.arange(R, device=dev)
    seen = torch.ones(R, R, dtype=torch.bool, device=dev).tril()       # which new rows a new row sees
    if case["branch"]:
        seen.zero_()
        depth = [0] * R
        for i, parent in enumerate(_parents(R, case["branch"])):
            if parent >= 0:
                seen[i] = seen[parent]
                depth[i] = depth[parent] + 1
            seen[i, i] = True
        pos = torch.tensor(lens, device=dev)[:, None] + torch.tensor(depth, device=dev)
    x = weights["embed"][tokens.long()].double()
    k_new, v_new = [[] for _ in range(B)], [[] for _ in range(B)]
    for l in range(s.n_layers):
        n = _norm(x, weights[f"l{l}.attn_norm"], s.rms_eps)
        q = _rope((n @ w(f"l{l}.wq").t()).view(B, R, s.n_q_heads, s.d_head), pos, s.rope_theta)
        k = _rope((n @ w(f"l{l}.wk").t()).view(B, R, s.n_kv_heads, s.d_head), pos, s.rope_theta)
        v = (n @ w(f"l{l}.wv").t()).view(B, R, s.n_kv_heads, s.d_head)
        a = torch.empty(B, R, s.n_q_heads, s.d_head, dtype=torch.float64, device=dev)
        for b in range(B):
            k_new[b].append(k[b].transpose(0, 1))
            v_new[b].append(v[b].permute(1, 2, 0))
            for h in range(s.n_kv_heads):
                keys, vals = k[b, :, h], v[b, :, h]
                if case["ctx"]:
                    keys = torch.cat([ks[l][b, h, :lens[b]].double(), keys])
                    vals = torch.cat([vs[l][b, h, :lens[b]].double(), vals])
                qh = q[b, :, h * group:(h + 1) * group].transpose(0, 1).reshape(group * R, s.d_head)
                score = (qh @ keys.t().contiguous()).view(group, R, -1) / s.d_head ** 0.5
                score[:, :, lens[b]:].masked_fill_(~seen, float("-inf"))
                out = torch.softmax(score, -1).view(group * R, -1) @ vals.contiguous()
                a[b, :, h * group:(h + 1) * group] = out.view(group, R, s.d_head).transpose(0, 1)
        x = x + a.view(B, R, -1) @ w(f"l{l}.wo").t()
        n = _norm(x, weights[f"l{l}.ffn_norm"], s.rms_eps)
        g = n @ w(f"l{l}.w_gate").t()
        x = x + (g * torch.sigmoid(g) * (n @ w(f"l{l}.w_up").t())) @ w(f"l{l}.w_down").t()
    n = _norm(x[:, R - case["logit_rows"]:], weights["final_norm"], s.rms_eps)
    head = weights["lm_head"]
    logits = torch.cat([n @ part.double().t() for part in head.split(16384)], dim=-1)
    k_new, v_new = [torch.stack(t) for t in k_new], [torch.stack(t) for t in v_new]
    if case["branch"]:
        for j, node in enumerate(_path(case, seed)):
            for b in range(B):
                k_new[b][:, :, j + 1] = k_new[b][:, :, node].clone()
                v_new[b][..., j + 1] = v_new[b][..., node].clone()
    return {"logits": logits, "k": k_new, "v": v_new, "lens": None}
