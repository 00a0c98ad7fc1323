"""The wavefront split of a step launch: its planner on the host (wave_plan_check.cpp), and its kernel
on the GPU against the oracle, where pieces, pages and slots are ragged and some slots are idle."""

import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_22950_amd", "csrc")


def test_wave_plan_host_check(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "wave_plan_check")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-I" + CSRC,
                        os.path.join(HERE, "wave_plan_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout


# (heads per KV head, KV heads, head_dim, prompts, slots a prompt, longest response, E4M3 cache)
@pytest.mark.gpu
@pytest.mark.parametrize("hpk,hkv,d,prompts,m,longest,fp8", [
    (4, 8, 128, (100, 33, 257, 64), 16, 200, False),  # 64 slots, several prompts
    (2, 8, 128, (70,), 40, 700, False),               # one prompt, pieces of several rounds
    (1, 2, 64, (31,), 64, 1500, False),               # other head size, coherence-point exchange
    (2, 8, 128, (50, 200), 20, 600, True),            # E4M3 pages
    (2, 8, 128, (0, 40, 90, 16, 1, 300, 65), 7, 400, False),  # fewer than 16 prefix rows, an empty prompt
])
def test_step_launch_wave_pieces(hpk, hkv, d, prompts, m, longest, fp8):
    from tests.gpu_harness import check_against_oracle, run_gpu_group
    from workload import get_config

    # few samples beyond the slots: every slot decodes one or two responses, and the last steps have idle slots
    cfg = get_config("tiny_f32").with_(
        name=f"waves_{hpk}_{hkv}_{d}_{len(prompts)}x{m}", layers=2, num_q_heads=hkv * hpk, num_kv_heads=hkv, head_dim=d,
        prompt_lens=prompts, slots_per_prompt=m, samples_per_prompt=m + 2, length_dist=("uniform", longest // 2, longest),
        max_suffix_len=longest, dtype="bf16", seed=31, pool_rows=1 << 14)
    every = max(1, longest // 12)
    wl, log, _, captured, tokens, _ = run_gpu_group(cfg, "fifo", entry="decode_step_layers", kv_fp8=fp8, window=128,
                                                    capture=lambda k: k % every == every - 1)
    assert np.array_equal(tokens, wl.L)
    check_against_oracle(cfg, wl, log, captured, kv_fp8=fp8)
