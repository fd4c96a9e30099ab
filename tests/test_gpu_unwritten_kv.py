"""KV pools that hold anything when they are bound: K/V slots that no token has filled (the rest of a context's
last page, draft slots whose segment skips the block) must not reach any row's output, as 0 * NaN would.  Every
path that reads the cache gives the same bits on a pool of NaN patterns as on a cleared one."""
import numpy as np
import pytest

import synth
from paper_2609_26100_amd import tss as abi
from tests.gpu_common import gpu_verifier, log

pytestmark = pytest.mark.gpu

BF16 = synth.ModelShape("unwritten-d256", 98, n_layers=2, d_model=256, n_heads=2, head_dim=128, ffn_dim=352, vocab=416,
                        dtype="bf16")
F32 = synth.ModelShape("unwritten-f32", 99, n_layers=2, d_model=256, n_heads=4, head_dim=64, ffn_dim=352, vocab=416,
                       dtype="f32")
MAX = 400


def _outputs(v, fill):
    """Logits of every path on a pool whose bytes are all `fill` (0xFF: a NaN in fp16 and in fp32)."""
    import torch
    v.bind_kv(2, MAX)
    v.kv_pool.fill_(fill)
    torch.cuda.synchronize()
    abi.tss_kv_alloc(v.ctx, 2, MAX, v.kv_pool.data_ptr(), v.kv_pool.numel())
    vocab, out = v.shape.vocab, {}

    def keep(name, rows):
        out[name] = v.logits(rows)

    toks = synth.context_tokens(vocab, 200, stream=1)
    draft = synth.context_tokens(vocab, 33, stream=2)
    tree = synth.random_tree(33, stream=3, max_children=3)
    v.prefill(0, toks[:5])
    v.verify(0, draft[:1])
    keep("chain behind a small step", 1)
    v.prefill(0, toks[5:135])     # a pass of many rows in the bf16 mode, ends inside a page
    v.verify(0, draft[:6])
    keep("chain behind a prompt", 6)
    v.verify(0, draft, tree)
    keep("tree", 33)
    v.prefill(1, toks[:70])
    v.verify_batch([0, 1], [draft[:17], draft[17:]], None)
    keep("batch", 33)
    masks = np.array([[0, 0], [1, 0], [0, 1]], np.uint8)
    v.verify_sweep(0, draft[:17], masks, tree[:17], reuse_prefix=False)
    keep("sweep", 51)
    return out


@pytest.mark.parametrize("shape", [BF16, F32], ids=lambda s: s.name)
def test_unwritten_slots_reach_no_output(shape):
    v = gpu_verifier(shape, n_seqs=2, max_tokens=MAX, max_nodes=64, max_batch=2)
    want, got = _outputs(v, 0), _outputs(v, 0xFF)
    v.close()
    for name in want:
        log(f"{shape.name} {name}: {int(np.isnan(got[name]).sum())} NaN of {got[name].size}")
        assert np.isfinite(want[name]).all()
    for name in want:
        np.testing.assert_array_equal(got[name], want[name], err_msg=name)
