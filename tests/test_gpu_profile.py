"""Timing of single launches (tss_profile_kernel): every pass of a prefill counts."""
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
