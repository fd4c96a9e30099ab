"""Prefill passes of many tokens (bf16 mode) at the sizes where their tiling can go wrong: one token past
what a small step takes, the edges of the 16- and 128-row blocks, more than one pass, a pass that starts
inside a page, both head dims, widths that no column block divides, skipped first, middle and last blocks,
permuted pages; on wider models (BLOCK_CASES) every block shape of more than 128 rows and the residual
projections' K splits, with ragged rows, columns and K chunks.  Each prompt's K/V are judged through the logits of the steps that read them,
against the oracle and against the same prompt prefilled in calls of at most 64 tokens (the small-step
path).

Tolerance: the paths share the operands' fp16 roundings except where a sum's rounding tips a stored fp16
value, so each is off the oracle by fp16's 2^-11 per operand, about sqrt(4 operands x 2 blocks) * 2^-11 =
1.4e-3 of the logits' norm; 8e-3 allows for the growth through the blocks."""
import numpy as np
import pytest

import synth
from oracle import OracleSequence, verify
from tests.gpu_common import gpu_verifier, log, oracle_model, prefill_chunked

pytestmark = pytest.mark.gpu

REL = 8e-3
HD64 = synth.ModelShape("prompt-d320", 91, n_layers=3, d_model=320, n_heads=5, head_dim=64, ffn_dim=672, vocab=416,
                        dtype="bf16")
HD128 = synth.ModelShape("prompt-d640", 92, n_layers=3, d_model=640, n_heads=5, head_dim=128, ffn_dim=1056, vocab=416,
                         dtype="bf16")

# Models wide enough for every block shape that prompts of more than 128 rows can take: column tiles that 8, 12 or
# 16 do not divide and an odd number of K chunks of the down projection (65, 131 and 33; d / 32 is always even).
WIDE = {
    "d2176": synth.ModelShape("prompt-d2176", 101, n_layers=2, d_model=2176, n_heads=17, head_dim=128, ffn_dim=2080,
                              vocab=416, dtype="bf16"),
    "d1088": synth.ModelShape("prompt-d1088", 102, n_layers=2, d_model=1088, n_heads=17, head_dim=64, ffn_dim=4192,
                              vocab=416, dtype="bf16"),
    "d4160": synth.ModelShape("prompt-d4160", 103, n_layers=2, d_model=4160, n_heads=65, head_dim=64, ffn_dim=1056,
                              vocab=416, dtype="bf16"),
}
WIDE_MAX_TOKENS = 2112
# model, prompt rows, and the blocks (row tiles, column tiles, K splits) of Q/K/V, gate/up, O and down;
# test_tile_shapes.py compares these with the host's rule.  Every row count ends inside a row tile and, but for 2045
# (13 rows in the last tile of whole blocks), inside a row block.
BLOCK_CASES = [
    ("d2176", 137, (8, 8, 1), (8, 8, 1), (8, 8, 4), (8, 4, 3)),
    ("d2176", 300, (8, 8, 1), (8, 8, 1), (8, 8, 4), (8, 8, 4)),
    ("d2176", 1030, (16, 8, 1), (16, 8, 1), (8, 8, 1), (8, 8, 1)),
    ("d2176", 1300, (16, 12, 1), (16, 8, 1), (8, 8, 1), (8, 8, 1)),
    ("d2176", 2045, (16, 16, 1), (16, 12, 1), (16, 8, 1), (16, 8, 1)),
    ("d1088", 777, (8, 8, 1), (16, 12, 1), (8, 4, 1), (8, 8, 4)),
    ("d1088", 1300, (16, 8, 1), (16, 16, 1), (8, 4, 1), (8, 8, 2)),
    ("d4160", 300, (16, 8, 1), (8, 8, 1), (8, 8, 2), (8, 4, 1)),
    ("d4160", 2045, (16, 16, 1), (16, 8, 1), (16, 16, 1), (16, 16, 1)),
]


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module", params=[HD64, HD128], ids=lambda s: s.name)
def model(request):
    shape = request.param
    max_tokens = 2300
    pages = 2 * ((max_tokens + 15) // 16)
    order = np.random.default_rng(3).permutation(pages)
    v = gpu_verifier(shape, random_gains=True, n_seqs=2, max_tokens=max_tokens, max_nodes=64, page_order=order)
    yield shape, v, oracle_model(shape, random_gains=True)
    v.close()


@pytest.mark.parametrize("lead,n,skip", [(0, 65, []), (0, 127, []), (5, 128, []), (0, 257, []), (37, 300, []),
                                         (0, 1025, []), (0, 65, [2]), (37, 300, [0]), (37, 300, [1]), (0, 129, [0, 2])])
def test_prompt_against_oracle_and_small_steps(model, lead, n, skip):
    shape, v, m = model
    mask = synth.mask_from_layers(shape.n_layers, skip)
    toks = synth.context_tokens(shape.vocab, lead + n, stream=n)
    draft = synth.context_tokens(shape.vocab, 9, stream=n + 1)
    tree = synth.random_tree(9, stream=n + 2, max_children=3)
    for s in (0, 1):
        v.truncate(s, 0)
        v.set_mask(s, mask)
        if lead:
            v.prefill(s, toks[:lead])
    v.prefill(0, toks[lead:])
    for i in range(lead, lead + n, 64):
        v.prefill(1, toks[i:i + 64][:lead + n - i])
    assert v.length(0) == v.length(1) == lead + n
    got = []
    for s in (0, 1):
        v.verify(s, draft, tree)
        got.append(v.logits(9))
    o = OracleSequence(m, mask)
    prefill_chunked(m, o, toks)
    want = verify(m, o, draft, tree).logits
    log(f"{shape.name} lead {lead} n {n} skip {skip}: rel {_rel(got[0], want):.2e} (small steps {_rel(got[1], want):.2e}, "
        f"between them {_rel(got[0], got[1]):.2e})")
    assert _rel(got[0], want) <= REL and _rel(got[0], got[1]) <= REL
    assert _rel(got[0], want) <= 2 * _rel(got[1], want) + 1e-4   # no less exact than the small steps
    v.check_kv()


def test_prompt_of_two_passes_repeats_bit_for_bit(model):
    shape, v, m = model
    toks = synth.context_tokens(shape.vocab, 2240, stream=7)
    draft = synth.context_tokens(shape.vocab, 6, stream=8)
    v.set_mask(0, None)
    out = []
    for _ in range(2):
        v.truncate(0, 0)
        v.prefill(0, toks)
        v.verify(0, draft)
        out.append(v.logits(6))
    np.testing.assert_array_equal(out[0], out[1])
    v.set_mask(1, None)
    v.truncate(1, 0)
    for i in range(0, len(toks), 64):
        v.prefill(1, toks[i:i + 64])
    v.verify(1, draft)
    assert _rel(out[0], v.logits(6)) <= REL


def test_every_block_skipped_keeps_the_length(model):
    shape, v, m = model
    v.truncate(0, 0)
    v.set_mask(0, np.ones(shape.n_layers, np.uint8))
    v.prefill(0, synth.context_tokens(shape.vocab, 200, stream=9))
    assert v.length(0) == 200
    v.set_mask(0, None)
    with pytest.raises(Exception, match="lacks K/V"):
        v.prefill(0, synth.context_tokens(shape.vocab, 100, stream=9))


def test_long_prompt_and_a_pool_without_room_for_passes():
    """4400 tokens in three passes (the last rows walk more than 64 steps of four pages) against the same
    prompt on a pool whose bytes hold the pages alone, which takes it in small steps."""
    import torch
    from paper_2609_26100_amd import tss as abi
    shape = synth.ModelShape("prompt-long", 97, n_layers=2, d_model=256, n_heads=2, head_dim=128, ffn_dim=352, vocab=416,
                             dtype="bf16")
    toks = synth.context_tokens(shape.vocab, 4400, stream=11)
    draft = synth.context_tokens(shape.vocab, 6, stream=12)
    out = []
    for small in (False, True):
        v = gpu_verifier(shape, n_seqs=1, max_tokens=4480, max_nodes=16)
        if small:
            pages = 280
            need = pages * 4 + 4480 * 64 * 8 + 2 * pages * 2 * 2 * 16 * 128 * 2 + 3 * 256
            assert need < abi.tss_kv_bytes(v.cfg, 1, 4480)
            pool = torch.zeros(need, dtype=torch.uint8, device="cuda:0")
            torch.cuda.synchronize()
            abi.tss_kv_alloc(v.ctx, 1, 4480, pool.data_ptr(), need)
        v.prefill(0, toks)
        assert v.length(0) == 4400
        v.verify(0, draft)
        out.append(v.logits(6))
        v.close()
    log(f"4400 tokens: passes against small steps {_rel(out[0], out[1]):.2e}")
    assert _rel(out[0], out[1]) <= REL


@pytest.fixture(scope="module", params=list(WIDE))
def wide(request):
    shape = WIDE[request.param]
    order = np.random.default_rng(13).permutation(2 * ((WIDE_MAX_TOKENS + 15) // 16))
    v = gpu_verifier(shape, random_gains=True, n_seqs=2, max_tokens=WIDE_MAX_TOKENS, max_nodes=64, page_order=order)
    yield request.param, shape, v
    v.close()


def test_every_block_shape_at_ragged_sizes(wide):
    """Two blocks: the first runs whole, the second ends at its K/V, so all four projections of the pass are in the
    logits.  Against the same prompt in calls of at most 64 tokens, whose kernels other tests compare with the
    oracle; a repeat gives the same bits."""
    name, shape, v = wide
    draft = synth.context_tokens(shape.vocab, 6, stream=20)
    for n in [c[1] for c in BLOCK_CASES if c[0] == name]:
        toks = synth.context_tokens(shape.vocab, n, stream=n)
        out = []
        for s, step in ((0, n), (0, n), (1, 64)):
            v.truncate(s, 0)
            for i in range(0, n, step):
                v.prefill(s, toks[i:i + step])
            v.verify(s, draft)
            out.append(v.logits(6))
        log(f"{shape.name} {n} rows: against small steps {_rel(out[0], out[2]):.2e}")
        np.testing.assert_array_equal(out[0], out[1])
        assert _rel(out[0], out[2]) <= REL


def test_split_report_of_prefill_passes(model):
    """The report describes the pass's last attention launch: one workgroup a head for each 128 rows; no items when
    the pass launches no attention (one running block, whose K/V are all that is kept, or none)."""
    shape, v, m = model
    toks = synth.context_tokens(shape.vocab, 300, stream=21)
    for skip, want in (([], [(1, 128), (1, 128), (1, 44)]), ([0, 2], []), ([], [(1, 128), (1, 128), (1, 44)]),
                       ([0, 1, 2], [])):
        v.truncate(0, 0)
        v.set_mask(0, synth.mask_from_layers(shape.n_layers, skip))
        v.prefill(0, toks)
        assert v.attn_split() == want, skip
    v.truncate(0, 0)
    v.set_mask(0, None)
    v.prefill(0, synth.context_tokens(shape.vocab, 2240, stream=22))  # two passes: 1280 and 960 rows
    assert v.attn_split() == [(1, 128)] * 7 + [(1, 64)]
