"""The work that users of this framework have it do, as cases that can be timed
and checked: verification steps of chains, trees, batches and mask sweeps, and
prompts taken from their tokens to the first verification step.

The decoder shapes are the repository's own (the tiny fp32 decoder and the
7B, 13B and 33B LLaMA shapes) at their full widths and vocabularies, with a few
blocks instead of all of them: every kernel runs at the size it has in the
whole model, and a state is made in about a second.  Each case is a dict of

  shape, layers   decoder shape and how many of its blocks the model has
  op              "verify" (one sequence, one committed step), "batch" (several
                  sequences in one committed step), "sweep" (one draft under
                  many masks, dry runs) or "prompt" (a new request: prefill,
                  then the first step)
  ctx             context tokens in KV before the step ("prompt": the prompt;
                  "batch": the longest, the shortest is ctx_min)
  nodes           nodes of a draft, root included; tree: breadth-first tree of
                  at most four children a node instead of a chain
  seqs, masks     sequences of a batch, masks of a sweep
  skip            blocks that each sequence's mask skips
"""
import math
import random

import numpy as np
import torch

from paper_2609_26100_amd import tss
from paper_2609_26100_amd.verifier import Verifier

DEV = "cuda:0"


class Shape:
    rope_base, rms_eps = 10000.0, 1e-6

    def __init__(self, name, n_layers, d_model, n_heads, head_dim, ffn_dim, vocab, dtype):
        self.name, self.n_layers, self.d_model, self.n_heads = name, n_layers, d_model, n_heads
        self.head_dim, self.ffn_dim, self.vocab, self.dtype = head_dim, ffn_dim, vocab, dtype


SHAPES = {
    "tiny": (256, 4, 64, 704, 4096, "f32"),
    "7b": (4096, 32, 128, 11008, 32000, "bf16"),
    "13b": (5120, 40, 128, 13824, 32000, "bf16"),
    "33b": (6656, 52, 128, 17920, 32000, "bf16"),
}


def shape_of(case):
    return Shape(case["shape"], case["layers"], *SHAPES[case["shape"]])


def make(name, shape, layers, op, ctx, nodes=6, tree=False, seqs=1, masks=1, skip=0, ctx_min=0):
    c = {"shape": shape, "layers": layers, "op": op, "ctx": ctx, "ctx_min": ctx_min or ctx, "nodes": nodes,
         "tree": tree, "seqs": seqs, "masks": masks, "skip": skip}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: the fp32 decoder that examples and smoke runs use, a chain of 5 drafts;
        # launches and the host path are all there is
        make("tiny_chain6", "tiny", 4, "verify", 128, skip=1),
        # plain autoregressive decoding: the root alone
        make("7b_root", "7b", 4, "verify", 512, nodes=1),
        # the headline step: a chain of 5 drafts after 1024 tokens
        make("7b_chain6", "7b", 4, "verify", 1024),
        # tree drafts: 60 nodes and the root after 2048 tokens, under a mask
        make("7b_tree61", "7b", 4, "verify", 2048, nodes=61, tree=True, skip=1),
        # four requests of one domain served together, equal contexts
        make("7b_batch4", "7b", 4, "batch", 1024, seqs=4, skip=1),
        # eight requests, each with its own mask, contexts from 512 to 4096 tokens, 72 rows
        make("13b_batch8", "13b", 2, "batch", 4096, nodes=9, seqs=8, skip=1, ctx_min=512),
        # a large model's tree step at a long context
        make("33b_tree33", "33b", 2, "verify", 4096, nodes=33, tree=True),
        # the offline search: every non-empty skip set of four blocks on one draft, 120 rows in one step
        make("7b_sweep15", "7b", 4, "sweep", 512, nodes=8, masks=15),
        # new requests, prompt to first step: a short question ...
        make("7b_prompt117", "7b", 4, "prompt", 117),
        # ... a page of text under a domain's mask ...
        make("13b_prompt777", "13b", 2, "prompt", 777, skip=1),
        # ... the headline context ...
        make("7b_prompt1024", "7b", 4, "prompt", 1024),
        # ... and a long document
        make("7b_prompt4000", "7b", 4, "prompt", 4000),
    ]


def draw(rng):
    """One more case: the same operations over their whole ranges."""
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["verify", "verify", "batch", "sweep", "prompt", "prompt"])
    shape = rng.choice(["tiny", "7b", "7b", "13b", "33b"])
    layers = 4 if shape in ("tiny", "7b") else 2
    if shape == "tiny":
        ctx = span(17, 900)
    else:
        ctx = span(33, 4000) if op != "prompt" or shape == "7b" else span(33, 1300)
    skip = rng.randint(0, layers // 2)
    if op == "verify":
        nodes = span(1, 64)
        return make("", shape, layers, op, ctx, nodes=nodes, tree=rng.random() < 0.5 and nodes > 2, skip=skip)
    if op == "batch":
        seqs = rng.randint(2, 8)
        most = (64 if shape == "tiny" else 128) // seqs
        return make("", shape, layers, op, ctx, nodes=span(1, min(16, most)), seqs=seqs, skip=skip,
                    ctx_min=max(1, ctx // rng.randint(1, 8)))
    if op == "sweep":
        masks = rng.randint(2, 2 ** layers - 1)
        nodes = span(1, max(1, (64 if shape == "tiny" else 128) // masks))
        return make("", shape, layers, op, ctx, nodes=nodes, tree=rng.random() < 0.3 and nodes > 2, masks=masks)
    return make("", shape, layers, op, ctx, nodes=span(1, 12), skip=skip)


# --- inputs -----------------------------------------------------------------

def tree_parents(n):
    """Breadth-first parents: the first node of a level takes up to four children, the next three, then two, one."""
    parent, level = [-1], [0]
    while len(parent) < n:
        nxt = []
        for i, p in enumerate(level):
            for _ in range(max(1, 4 - i)):
                if len(parent) < n:
                    parent.append(p)
                    nxt.append(len(parent) - 1)
            if len(nxt) >= 20:
                break
        level = nxt
    return np.asarray(parent, dtype=np.int32)


def inputs(case, seed):
    """Tokens, trees and masks of the case's sequences (host values a program holds before the call)."""
    s = shape_of(case)
    rng = np.random.default_rng([seed, 1])
    n = case["nodes"]
    parent = tree_parents(n) if case["tree"] else None
    seqs = []
    for i in range(case["seqs"]):
        span = case["ctx"] - case["ctx_min"]
        ctx = case["ctx"] if i == 0 else case["ctx_min"] + int(rng.integers(0, span + 1))
        mask = np.zeros(s.n_layers, np.uint8)
        mask[rng.permutation(s.n_layers)[: case["skip"]]] = 1
        seqs.append({"ctx": rng.integers(0, s.vocab, ctx).astype(np.int32),
                     "draft": rng.integers(0, s.vocab, n).astype(np.int32), "parent": parent, "mask": mask})
    masks = None
    if case["op"] == "sweep":  # non-empty skip sets, those that run the most leading blocks first
        L = s.n_layers
        sets = [[(b >> l) & 1 for l in range(L)] for b in range(1, 2 ** L)]
        keep = rng.permutation(len(sets))[: case["masks"]]
        masks = np.asarray(sorted((sets[k] for k in keep), key=lambda m: -m.index(1)), dtype=np.uint8)
    return s, seqs, masks


def tensor_sizes(s):
    d, f, v = s.d_model, s.ffn_dim, s.vocab
    layer = [(d,), (d, d), (d, d), (d, d), (d, d), (d,), (f, d), (f, d), (d, f)]
    return [(v, d)] + layer * s.n_layers + [(d,), (v, d)]


def weights(s, seed):
    """Every tensor in load order: matrices N(0, 0.02^2), gains N(1, 0.1^2), as windows into one random pool."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    sizes = tensor_sizes(s)
    t = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    extra = 64 * 1021
    most = max(math.prod(z) for z in sizes)
    pool = (torch.randn(most + extra, generator=g, device=DEV) * 0.02).to(t)
    out = []
    for i, z in enumerate(sizes):
        at = (i * 7919 * 8) % extra // 8 * 8
        w = pool[at: at + math.prod(z)].reshape(z)
        out.append((1 + 5 * w.float()).to(t) if len(z) == 1 else w)
    return out, pool


def host(w):
    w = w.cpu()
    return w.view(torch.int16).numpy().view(np.uint16) if w.dtype == torch.bfloat16 else w.numpy()


def prepare(case, seed):
    s, seqs, masks = inputs(case, seed)
    n, longest = case["nodes"], case["ctx"]
    rows = n * max(case["seqs"], case["masks"])
    batch = max(case["seqs"], -(-rows // max(n, 16)) if masks is not None else 1)
    nodes = n if masks is None else max(n, 16)
    if case["op"] == "prompt":
        nodes = 64
    v = Verifier(s, n_seqs=len(seqs), max_tokens=longest + max(rows, nodes) + 16, max_nodes=nodes, max_batch=batch)
    w, pool = weights(s, seed)
    p = host(pool)
    base = pool.data_ptr()
    for i, t in enumerate(w):
        at = (t.data_ptr() - base) // t.element_size()
        tss.tss_load_weights(v.ctx, i, [p[at: at + t.numel()].reshape(t.shape) if t.dim() == 2 else host(t)])
    for i, q in enumerate(seqs):
        v.set_mask(i, q["mask"])
        if case["op"] != "prompt":
            v.prefill(i, q["ctx"])
    return {"op": case["op"], "v": v, "seqs": seqs, "masks": masks, "rows": rows, "ids": list(range(len(seqs)))}


def run(state):
    v, op, seqs = state["v"], state["op"], state["seqs"]
    q = seqs[0]
    if op == "verify":      # a committed step; the context is what the next call finds again
        v.verify(0, q["draft"], q["parent"], commit=True)
        v.truncate(0, len(q["ctx"]))
    elif op == "batch":
        v.verify_batch(state["ids"], [x["draft"] for x in seqs], [x["parent"] for x in seqs], commit=True)
        for i, x in enumerate(seqs):
            v.truncate(i, len(x["ctx"]))
    elif op == "sweep":
        v.verify_sweep(0, q["draft"], state["masks"], q["parent"])
    else:                   # a new request on this sequence
        v.truncate(0, 0)
        v.prefill(0, q["ctx"])
        v.verify(0, q["draft"], q["parent"])
    return v.logits_device(state["rows"])


# --- what a pass cannot do without -------------------------------------------

def work(case):
    s, seqs, masks = inputs(case, 0)
    es = 2 if s.dtype == "bf16" else 4
    d, f, v, L = s.d_model, s.ffn_dim, s.vocab, s.n_layers
    block = 4 * d * d + 3 * d * f
    n = case["nodes"]
    all_masks = masks if masks is not None else np.stack([q["mask"] for q in seqs])
    rows = n * len(all_masks)
    union = int((all_masks == 0).any(axis=0).sum())
    active = int((all_masks == 0).sum())            # (segment, block) pairs that run
    bytes_ = union * block * es + v * d * es + rows * (v * 4 + d * es)
    flops = 2.0 * n * active * block + 2.0 * rows * v * d
    for i, m in enumerate(all_masks):
        on, ctx = int((m == 0).sum()), len(seqs[i if masks is None else 0]["ctx"])
        flops += 4.0 * on * n * (ctx + n / 2) * d
        bytes_ += on * 2 * d * es * n
        if masks is None:
            bytes_ += on * 2 * d * es * ctx
    if masks is not None:                           # the context is read once for all masks
        bytes_ += union * 2 * d * es * len(seqs[0]["ctx"])
    if case["op"] == "prompt":                      # and the prompt's own pass before the step
        on, ctx = int((seqs[0]["mask"] == 0).sum()), case["ctx"]
        bytes_ += on * (block + 2 * d * ctx) * es + ctx * d * es
        flops += on * (2.0 * ctx * block + 2.0 * ctx * ctx * d)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # Relative error of the logits after a few blocks, about four times what the
    # paths show against 64 bits: 3e-7 with fp32 throughout (the tiny decoder),
    # 1.3e-3 to 2.6e-3 with fp16 operands and fp32 sums (the others).
    return {"rel": 4e-6, "max": 4e-5} if case["shape"] == "tiny" else {"rel": 8e-3, "max": 6e-2}


# --- the same in 64 bits -------------------------------------------------------

def exact(case, seed):
    """Logits of the step's rows in float64: plain torch, one sequence after the other."""
    s, seqs, masks = inputs(case, seed)
    w, _ = weights(s, seed)
    L, H, hd, d = s.n_layers, s.n_heads, s.head_dim, s.d_model
    half = hd // 2
    inv = 10000.0 ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / hd)

    def norm(x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * g.double()

    def turn(x, pos):
        a = pos.double()[:, None] * inv
        c, z = a.cos()[:, None], a.sin()[:, None]
        x = x.reshape(-1, H, hd)
        p, q = x[..., :half], x[..., half:]
        return torch.cat([p * c - q * z, q * c + p * z], -1)

    def blocks(tokens, pos, mask, kv, vis):
        """Residual after every block the mask runs; kv[l] = (K, V) of earlier rows; vis: this call's rows."""
        x = w[0][tokens].double()
        new = [None] * L
        for l in range(L):
            if mask[l]:
                continue
            an, wq, wk, wv, wo, mn, wg, wu, wd = w[1 + 9 * l: 10 + 9 * l]
            y = norm(x, an)
            q, k = turn(y @ wq.double().T, pos), turn(y @ wk.double().T, pos)
            v = (y @ wv.double().T).reshape(-1, H, hd)
            new[l] = (k, v)
            old = kv[l] if kv is not None else None
            o = torch.empty_like(q)
            for h in range(H):
                kh, vh = k[:, h], v[:, h]
                sc = (q[:, h] @ kh.T / math.sqrt(hd)).masked_fill(~vis, -math.inf)
                if old is not None:
                    sc = torch.cat([q[:, h] @ old[0][:, h].T / math.sqrt(hd), sc], 1)
                    vh = torch.cat([old[1][:, h], vh], 0)
                o[:, h] = torch.softmax(sc, 1) @ vh
            x = x + o.reshape(-1, d) @ wo.double().T
            y = norm(x, mn)
            x = x + (torch.nn.functional.silu(y @ wg.double().T) * (y @ wu.double().T)) @ wd.double().T
        return x, new

    out = []
    for q in seqs:
        n, ctx = case["nodes"], len(q["ctx"])
        tok = torch.from_numpy(q["ctx"]).long().to(DEV)
        tri = torch.ones(ctx, ctx, dtype=torch.bool, device=DEV).tril()
        _, kv = blocks(tok, torch.arange(ctx, device=DEV), q["mask"], None, tri)
        parent = q["parent"] if q["parent"] is not None else np.arange(-1, n - 1)
        vis, depth = np.eye(n, dtype=bool), np.zeros(n, np.int64)
        for i in range(1, n):
            vis[i] |= vis[parent[i]]
            depth[i] = depth[parent[i]] + 1
        pos = torch.from_numpy(ctx + depth).to(DEV)
        drafts, vis = torch.from_numpy(q["draft"]).long().to(DEV), torch.from_numpy(vis).to(DEV)
        for m in (masks if masks is not None else [q["mask"]]):
            x, _ = blocks(drafts, pos, m, kv, vis)
            out.append(norm(x, w[-2]) @ w[-1].double().T)
    return torch.cat(out)
