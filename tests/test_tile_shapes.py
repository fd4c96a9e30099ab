"""The host's block-shape rules, evaluated on the CPU: the sizes that test_gpu_prompt.py and test_gpu_many_rows.py
name reach the block shapes that they name, and together every shape that a prompt of more than 128 rows, or the
Q/K/V and gate/up projections of a step of 6 to 8 row tiles, can take."""
import os
import subprocess

import pytest

from tests import test_gpu_many_rows as many
from tests.test_gpu_prompt import BLOCK_CASES, WIDE, WIDE_MAX_TOKENS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
QKV, RESID, SWIGLU = 0, 1, 2  # enum Epi


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not installed")
    exe = str(tmp_path_factory.mktemp("shapes") / "shapes")
    cmd = [CLANG, "-std=c++17", "-O1", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2609_26100_amd", "csrc"),
           "-Wno-everything", os.path.join(ROOT, "tests", "host_shapes", "shapes.cpp"),
           "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def shapes(which, projections):
        args = [str(x) for p in projections for x in p]
        r = subprocess.run([exe, which, *args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        return [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
    return shapes


def prompt_shapes(rule, s, rows, max_tokens):
    """Blocks of a pass's Q/K/V, gate/up, O and down projections (partial tiles: as the KV pool has room for them)."""
    cap = min(2048, -(-max_tokens // 16) * 16)
    parts = min(16 << 20, 4 * (-(-cap // 256) * 256) * (-(-s.d_model // 256) * 256) * 4)
    rt, d, f = -(-rows // 16), s.d_model, s.ffn_dim
    return rule("prompt", [(QKV, rt, 3 * d // 16, d // 32, 0), (SWIGLU, rt, 2 * f // 16, d // 32, 0),
                           (RESID, rt, d // 16, d // 32, parts), (RESID, rt, d // 16, f // 32, parts)])


@pytest.mark.parametrize("case", BLOCK_CASES, ids=lambda c: f"{c[0]}-{c[1]}")
def test_the_sizes_reach_the_named_blocks(rule, case):
    assert tuple(prompt_shapes(rule, WIDE[case[0]], case[1], WIDE_MAX_TOKENS)) == tuple(case[2:])


def test_the_cases_cover_every_large_block():
    large, resid = {(16, 16), (16, 12), (16, 8), (8, 8)}, {(16, 16), (16, 8), (8, 8), (8, 4)}
    for i in (2, 3):
        assert {c[i][:2] for c in BLOCK_CASES} == large
    assert {c[i][:2] for c in BLOCK_CASES for i in (4, 5)} == resid
    assert {c[i][2] for c in BLOCK_CASES for i in (4, 5)} == {1, 2, 3, 4}  # K splits


def test_step_models_reach_every_block(rule):
    seen = set()
    for shape, q, g in [(many.SMALL, 2, 4), (many.SPLIT, 2, 4)] + list(many.WIDE.values()):
        d, f = shape.d_model, shape.ffn_dim
        for rt, mr in ((6, 6), (7, 8), (8, 8)):
            got = rule("step", [(QKV, rt, 3 * d // 16, d // 32, 0), (SWIGLU, rt, 2 * f // 16, d // 32, 0)])
            assert got == [(mr, q, 1), (mr, g, 1)], (shape.name, rt)
            seen |= {(QKV,) + got[0][:2], (SWIGLU,) + got[1][:2]}
    assert seen == {(QKV, m, n) for m in (6, 8) for n in (2, 3, 4, 6)} | {(SWIGLU, m, n) for m in (6, 8)
                                                                          for n in (4, 6, 8, 10)}


def test_weights_are_nontemporal_where_they_do_not_fit_the_cache(rule):
    """192 MiB of what k_tile reads in a step: O and down up to 4 row tiles, every projection from 5 on."""
    mib = 1 << 20
    models = [(4, 256, 704, 4096), (12, 512, 1408, 4096), (16, 1024, 2816, 32000), (2, 2048, 5632, 32000),
              (16, 2048, 5632, 32000), (2, 4096, 11008, 32000), (32, 4096, 11008, 32000), (60, 6656, 17920, 32000),
              (12, 2048, 2048, 32), (13, 2048, 2048, 32)]
    for L, d, f, v in models:
        resid = 2 * L * (d * d + d * f)
        every = resid + 2 * L * (3 * d * d + 2 * d * f) + 2 * v * d
        got = rule("nt", [(rt, L, d, f, v) for rt in (2, 4, 5, 8)])
        assert got == [(int(x > 192 * mib),) for x in (resid, resid, every, every)], (L, d, f, v)
