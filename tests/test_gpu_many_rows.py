"""Steps of 2 to 8 row tiles (bf16 mode) at the edges of the tiled projections: the first and last row counts
of a row tile, column counts that no block width divides, an odd number of K chunks, K split unevenly, one
segment and several, blocks that only some segments run.  Every sequence of a batch is compared with its own
verify (at most 16 rows: another kernel) and with the oracle.

Tolerance: as for prompts, the operands' fp16 roundings give each path about 1.4e-3 of the logits' norm
against the oracle; 8e-3 allows for the growth through the blocks."""
import numpy as np
import pytest

import synth
from oracle import OracleSequence, prefill, verify
from tests.gpu_common import gpu_verifier, log, oracle_model

pytestmark = pytest.mark.gpu

REL = 8e-3
SMALL = synth.ModelShape("rows-d320", 93, n_layers=2, d_model=320, n_heads=5, head_dim=64, ffn_dim=672, vocab=416,
                         dtype="bf16")
SPLIT = synth.ModelShape("rows-d1024", 94, n_layers=2, d_model=1024, n_heads=8, head_dim=128, ffn_dim=2080, vocab=1056,
                         dtype="bf16")

# One-block models wide enough for the other blocks of steps of 6 to 8 row tiles (the two above take the narrowest):
# model, then the column tiles of its Q/K/V and gate/up blocks, which test_tile_shapes.py compares with the host's
# rule.  The gate/up columns leave a partial last block.
WIDE = {
    "d2752": (synth.ModelShape("rows-d2752", 107, n_layers=1, d_model=2752, n_heads=43, head_dim=64, ffn_dim=8224,
                               vocab=416, dtype="bf16"), 3, 6),
    "d4160": (synth.ModelShape("rows-d4160", 108, n_layers=1, d_model=4160, n_heads=65, head_dim=64, ffn_dim=12320,
                               vocab=416, dtype="bf16"), 4, 8),
    "d5504": (synth.ModelShape("rows-d5504", 109, n_layers=1, d_model=5504, n_heads=43, head_dim=128, ffn_dim=16416,
                               vocab=416, dtype="bf16"), 6, 10),
}


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module", params=[SMALL, SPLIT], ids=lambda s: s.name)
def model(request):
    shape = request.param
    order = np.random.default_rng(5).permutation(8 * 13)
    v = gpu_verifier(shape, random_gains=True, n_seqs=8, max_tokens=200, max_nodes=64, max_batch=8, page_order=order)
    m = oracle_model(shape, random_gains=True)
    masks = [synth.mask_from_layers(2, [] if i % 3 == 0 else [i % 2]) for i in range(8)]
    oseqs = []
    for i in range(8):
        ctx = synth.context_tokens(shape.vocab, 20 + 7 * i, stream=300 + i)
        v.set_mask(i, masks[i])
        v.prefill(i, ctx)
        o = OracleSequence(m, masks[i])
        prefill(m, o, ctx)
        oseqs.append(o)
    yield shape, v, m, oseqs
    v.close()


# nodes per sequence; 17, 32, 33, 48, 64, 65, 80, 81, 96, 97, 112, 113 and 128 rows
@pytest.mark.parametrize("nodes", [[9, 8], [16, 16], [16, 16, 1], [12] * 4, [8] * 8, [16] * 4 + [1], [10] * 8,
                                   [16] * 5 + [1], [16] * 6, [13] * 7 + [6], [14] * 8, [16] * 7 + [1], [16] * 8],
                         ids=lambda n: str(sum(n)))
def test_batch_rows_against_single_verifies_and_oracle(model, nodes):
    shape, v, m, oseqs = model
    seqs = list(range(len(nodes)))
    drafts = [synth.context_tokens(shape.vocab, n, stream=400 + 10 * i + n) for i, n in enumerate(nodes)]
    parents = [synth.random_tree(n, stream=500 + i, max_children=3) if i % 2 else None for i, n in enumerate(nodes)]
    v.verify_batch(seqs, drafts, parents)
    got = v.logits(sum(nodes))
    single, want = [], []
    for i in seqs:
        v.verify(i, drafts[i], parents[i])
        single.append(v.logits(nodes[i]))
        want.append(verify(m, oseqs[i], drafts[i], parents[i]).logits)
    single, want = np.concatenate(single), np.concatenate(want)
    e, e1 = _rel(got, want), _rel(single, want)
    log(f"{shape.name} {sum(nodes)} rows: rel {e:.2e} (singles {e1:.2e}, between them {_rel(got, single):.2e})")
    assert e <= REL and _rel(got, single) <= REL and e <= 2 * e1 + 1e-4
    # a repeat gives the same bits
    v.verify_batch(seqs, drafts, parents)
    np.testing.assert_array_equal(v.logits(sum(nodes)), got)


@pytest.mark.parametrize("n", [17, 33, 64])
def test_one_tree_of_many_rows(model, n):
    shape, v, m, oseqs = model
    tok = synth.context_tokens(shape.vocab, n, stream=600 + n)
    par = synth.random_tree(n, stream=600 + n, max_children=4)
    v.verify(3, tok, par)
    e = _rel(v.logits(n), verify(m, oseqs[3], tok, par).logits)
    log(f"{shape.name} tree of {n}: rel {e:.2e}")
    assert e <= REL


@pytest.mark.parametrize("ctx_len", [0, 1, 15, 16, 31, 48, 63, 64, 65, 130])
def test_tree_attention_at_page_and_step_edges(model, ctx_len):
    """Trees of 2 to 4 row tiles behind contexts that end at, before and after a page and a four-page step."""
    shape, v, m, _ = model
    s, L = 7, shape.n_layers
    ctx = synth.context_tokens(shape.vocab, ctx_len, stream=700 + ctx_len)
    v.truncate(s, 0)
    v.set_mask(s, None)
    if ctx_len:
        v.prefill(s, ctx)
    o = OracleSequence(m)
    if ctx_len:
        prefill(m, o, ctx)
    for n in (17, 33, 50, 64):
        tok = synth.context_tokens(shape.vocab, n, stream=800 + n)
        par = synth.random_tree(n, stream=800 + n, max_children=3)
        v.verify(s, tok, par)
        e = _rel(v.logits(n), verify(m, o, tok, par).logits)
        log(f"{shape.name} context {ctx_len} tree {n}: rel {e:.2e}, split {v.attn_split()}")
        assert e <= REL


def test_tree_attention_of_many_steps_per_workgroup():
    """128 heads and two items leave one workgroup per head and item, which walks 66 steps (two reads of its
    page ids) past the page ids in the arguments.  Each checked node's row against its root path verified as
    a chain of at most 16 nodes (another kernel), under both masks."""
    shape = synth.ModelShape("rows-h128", 96, n_layers=2, d_model=8192, n_heads=128, head_dim=64, ffn_dim=64, vocab=416,
                             dtype="bf16")
    pages = (4360 + 15) // 16
    v = gpu_verifier(shape, n_seqs=1, max_tokens=4360, max_nodes=64, max_batch=2,
                     page_order=np.random.default_rng(9).permutation(pages))
    ctx = synth.context_tokens(shape.vocab, 4200, stream=900)
    v.prefill(0, ctx)
    tok = synth.context_tokens(shape.vocab, 64, stream=901)
    par = synth.random_tree(64, stream=902, max_children=4)
    masks = np.array([[0, 0], [0, 1]], dtype=np.uint8)
    v.verify_sweep(0, tok, masks, par, reuse_prefix=False)
    got = v.logits(128).reshape(2, 64, -1)
    for node in (0, 1, 30, 47, 63):
        path = [node]
        while par[path[-1]] >= 0:
            path.append(int(par[path[-1]]))
        path = path[::-1]
        assert len(path) <= 16
        for k in (0, 1):
            v.verify(0, tok[path], None, masks[k])
            e = _rel(got[k, node], v.logits(len(path))[-1])
            log(f"node {node} depth {len(path) - 1} mask {k}: rel {e:.2e}")
            assert e <= REL
    v.close()


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_blocks_against_single_verifies(name):
    """81, 113 and 128 rows (6, 8 and 8 row tiles) of sequences of at most 16 rows, against each sequence's own
    verify."""
    shape = WIDE[name][0]
    v = gpu_verifier(shape, random_gains=True, n_seqs=8, max_tokens=64, max_nodes=16, max_batch=8)
    for i in range(8):
        v.prefill(i, synth.context_tokens(shape.vocab, 9 + 5 * i, stream=300 + i))
    for nodes in ([16] * 5 + [1], [16] * 7 + [1], [16] * 8):
        drafts = [synth.context_tokens(shape.vocab, n, stream=400 + i) for i, n in enumerate(nodes)]
        v.verify_batch(list(range(len(nodes))), drafts)
        got = v.logits(sum(nodes))
        single = []
        for i, n in enumerate(nodes):
            v.verify(i, drafts[i])
            single.append(v.logits(n))
        e = _rel(got, np.concatenate(single))
        log(f"{shape.name} {sum(nodes)} rows: against singles {e:.2e}")
        assert e <= REL
        v.verify_batch(list(range(len(nodes))), drafts)
        np.testing.assert_array_equal(v.logits(sum(nodes)), got)
    v.close()
