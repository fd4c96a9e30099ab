"""Timing of single launches (tss_profile_kernel): every pass of a prefill counts, and the attention's figure is
the attention launch's own where a merge launch follows it."""
import pytest

import synth
from paper_2609_26100_amd import tss as abi
from tests.gpu_common import gpu_verifier, log

pytestmark = pytest.mark.gpu


def test_every_prefill_pass_is_counted():
    shape = synth.ModelShape("profile-d256", 104, n_layers=2, d_model=256, n_heads=2, head_dim=128, ffn_dim=352, vocab=416,
                             dtype="bf16")
    v = gpu_verifier(shape, n_seqs=1, max_tokens=4200, max_nodes=16)
    for kernel, layer in ((abi.TSS_K_QKV, 0), (abi.TSS_K_EMBED, -1)):
        abi.tss_profile_kernel(v.ctx, kernel, layer)
        v.truncate(0, 0)
        v.prefill(0, synth.context_tokens(shape.vocab, 4150, stream=1))  # three passes
        ms, n = abi.tss_profile_read(v.ctx, reset=True)
        log(f"kernel {kernel}: {n} launches, {1e3 * ms:.1f} us")
        assert n == 3 and 0 < ms < 100
    abi.tss_profile_kernel(v.ctx, -1)
    v.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_of_many_rows_is_timed_without_its_merge(dtype):
    """33 rows over 16000 tokens (8000 in fp32) of 32 heads: 262 MB of K/V, which no launch reads in less than 15 us
    (17 TB/s, more than the caches or HBM give); the merge behind it takes about 5 us."""
    shape = synth.ModelShape("profile-" + dtype, 105, n_layers=1, d_model=4096, n_heads=32, head_dim=128, ffn_dim=64,
                             vocab=416, dtype=dtype)
    n = 16000 if dtype == "bf16" else 8000
    v = gpu_verifier(shape, n_seqs=1, max_tokens=n + 64, max_nodes=64)
    v.prefill(0, synth.context_tokens(shape.vocab, n, stream=1))
    tree = synth.random_tree(33, stream=2, max_children=3)
    draft = synth.context_tokens(shape.vocab, 33, stream=3)
    v.verify(0, draft, tree)
    abi.tss_profile_kernel(v.ctx, abi.TSS_K_ATTN, 0)
    for _ in range(3):
        v.verify(0, draft, tree)
    ms, count = abi.tss_profile_read(v.ctx, reset=True)
    abi.tss_profile_kernel(v.ctx, -1)
    log(f"{dtype}: {1e3 * ms / count:.1f} us a launch")
    v.close()
    assert count == 3 and 1e3 * ms / count > 15
