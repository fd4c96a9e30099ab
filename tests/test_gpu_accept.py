"""The accept scan at the row counts where its two 64-row words and its segments meet: one tree or chain of 1 to 64
nodes, segments that start before row 64 and end behind it, 128 rows, many masks of one draft.  Decision and
path must equal a plain walk over the same step's greedy tokens."""
import numpy as np
import pytest

import synth
from tests.gpu_common import gpu_verifier, log

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape("accept-d256", 106, n_layers=2, d_model=256, n_heads=2, head_dim=128, ffn_dim=352, vocab=416,
                         dtype="bf16")


def walk(tok, par, greedy):
    """(accept_len, next_token, path): the deepest node whose root path matches, lowest index among equal depths."""
    n = len(tok)
    ok, depth = [True] + [False] * (n - 1), [0] * n
    for i in range(1, n):
        depth[i] = depth[par[i]] + 1
        ok[i] = ok[par[i]] and tok[i] == greedy[par[i]]
    best = max((i for i in range(n) if ok[i]), key=lambda i: (depth[i], -i))
    path = [best]
    while path[-1]:
        path.append(int(par[path[-1]]))
    return depth[best], int(greedy[best]), path[::-1]


def fit(rng, toks, pars, greedy, p):
    """Gives each node its parent's greedy token with probability p (drawn once per node by rng)."""
    r0 = 0
    for tok, par in zip(toks, pars):
        for i in range(1, len(tok)):
            if rng[r0 + i] < p:
                tok[i] = greedy[r0 + par[i]]
        r0 += len(tok)


@pytest.fixture(scope="module")
def v():
    v = gpu_verifier(SHAPE, random_gains=True, n_seqs=8, max_tokens=300, max_nodes=64, max_batch=8)
    for i in range(8):
        v.prefill(i, synth.context_tokens(SHAPE.vocab, 20 + i, stream=i))
    yield v
    v.close()


def shapes(nodes, chain):
    return [np.arange(-1, n - 1, dtype=np.int32) if chain else synth.random_tree(n, stream=n + i, max_children=3)
            for i, n in enumerate(nodes)]


@pytest.mark.parametrize("chain,p", [(True, 1.0), (True, 0.8), (False, 1.0), (False, 0.8), (False, 0.0)])
@pytest.mark.parametrize("nodes", [[1], [64], [1, 63], [64, 64], [9] * 8, [13] * 7 + [6], [16] * 8, [1] * 8,
                                   [60, 8, 60]], ids=lambda n: "+".join(map(str, n)))
def test_decision_and_path(v, nodes, chain, p):
    pars = shapes(nodes, chain)
    toks = [synth.context_tokens(SHAPE.vocab, n, stream=50 + i) for i, n in enumerate(nodes)]
    draw = np.random.default_rng(len(nodes)).random(sum(nodes))
    seqs = list(range(len(nodes)))
    depth = max(nodes) if chain else 12
    for _ in range(depth if p else 1):   # a node's greedy token depends on its root path alone
        al, nt = v.verify_batch(seqs, toks, pars)
        g = v.greedy(sum(nodes))
        fit(draw, toks, pars, g, p)
    al, nt = v.verify_batch(seqs, toks, pars)
    g, r0, lens = v.greedy(sum(nodes)), 0, []
    for i, n in enumerate(nodes):
        want = walk(toks[i], pars[i], g[r0:r0 + n])
        assert (al[i], nt[i], list(v.path(i))) == want, i
        lens.append(want[0])
        r0 += n
    log(f"{nodes} chain {chain} p {p}: accepted {lens}")
    if p == 1.0 and chain:
        assert lens == [n - 1 for n in nodes]


def test_masks_of_one_draft(v):
    tok = synth.context_tokens(SHAPE.vocab, 8, stream=90)
    par = synth.random_tree(8, stream=91, max_children=2)
    masks = np.array([[k & 1, k >> 1 & 1] for k in range(15)], np.uint8)
    for _ in range(8):
        v.verify(0, tok, par)
        fit(np.zeros(8), [tok], [par], v.greedy(8), 0.5)
    al, nt, g = v.verify_sweep(0, tok, masks, par, want_greedy=True, reuse_prefix=False)
    for k in range(15):
        assert (al[k], nt[k], list(v.path(k))) == walk(tok, par, g[k]), k
    log(f"accepted {list(al)}")
    assert max(al) > 0
