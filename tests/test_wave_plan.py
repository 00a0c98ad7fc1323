"""The wavefront split of a step launch: its planner on the host (wave_plan_check.cpp), and its kernels
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


# (heads per KV head, KV heads, head_dim, prompts, slots a prompt, longest response, E4M3 cache, exchange)
@pytest.mark.gpu
@pytest.mark.parametrize("hpk,hkv,d,prompts,m,longest,fp8,exchange", [
    (4, 8, 128, (100, 33, 257, 64), 16, 400, False, None),  # 64 slots, several prompts
    (2, 8, 128, (70,), 40, 700, False, None),               # one prompt, pieces of several rounds
    (1, 8, 64, (31,), 64, 400, False, 0),                   # other head size, coherence-point exchange
    (8, 8, 64, (130, 33, 64, 40), 16, 500, False, None),    # 128 prefix rows
    (2, 8, 128, (50, 200), 20, 600, True, None),            # E4M3 pages
    (1, 8, 128, (129,), 64, 500, True, 0),
    (2, 8, 128, (0, 40, 90, 16, 1, 300, 65), 7, 400, False, None),  # fewer than 16 prefix rows, an empty prompt
])
def test_step_launch_wave_pieces(hpk, hkv, d, prompts, m, longest, fp8, exchange):
    """Every compared step runs one piece per wavefront (the library's own plan says which do), with all
    slots live and with some idle; the oracle's tolerance is that of the bf16 path, 1e-2."""
    import torch

    from paper_2506_22950_amd.group import context_for
    from tests.gpu_harness import check_against_oracle, oracle_log, run_gpu_group
    from workload import Workload, get_config

    # few samples beyond the slots: every slot decodes one or two responses, and the last steps have idle slots
    cfg = get_config("tiny_f32").with_(
        name=f"waves_{hpk}_{hkv}_{d}_{len(prompts)}x{m}", layers=2, num_q_heads=hkv * hpk, num_kv_heads=hkv, head_dim=d,
        prompt_lens=prompts, slots_per_prompt=m, samples_per_prompt=m + 2, length_dist=("uniform", longest // 2, longest),
        max_suffix_len=longest, dtype="bf16", seed=31, pool_rows=1 << 14)
    wl = Workload(cfg)
    log = oracle_log(cfg, wl, "fifo")
    ctx = context_for(cfg, stream=torch.cuda.current_stream(), kv_fp8=fp8, split_tokens=128)
    nj = ctx.step_launch_workgroups // hkv
    ctx.destroy()
    ctx = context_for(cfg, dry_run=True, kv_fp8=fp8, split_tokens=128)
    for p, plen in enumerate(prompts):
        ctx.prefill_shared(p, 0, plen, None, None)
    waves = [k for k, row in enumerate(log)
             if ctx.step_launch_plan([e[2] if e is not None else 0 for e in row], nj)[0]["cut"] == 2]
    ctx.destroy()
    idle = [k for k in waves if any(e is None for e in log[k])]
    full = [k for k in waves if k not in set(idle)]
    assert idle and full, "no step took one piece per wavefront"
    steps = {x[int(i)] for x in (idle, full) for i in np.linspace(0, len(x) - 1, 4)}
    wl, ran, _, captured, tokens, _ = run_gpu_group(cfg, "fifo", wl=wl, entry="decode_step_layers", split=128, kv_fp8=fp8,
                                                    exchange=exchange, window=128, capture=steps.__contains__)
    assert ran == log and np.array_equal(tokens, wl.L) and set(captured) == steps
    check_against_oracle(cfg, wl, log, captured, kv_fp8=fp8)


@pytest.mark.gpu
def test_step_launch_long_chunks():
    """Chunks of 2048 tokens leave a response of 2290 tokens two pieces, of more pages (72) than a wavefront
    can name: the last steps fall back to the split by work-groups."""
    from tests.gpu_harness import check_against_oracle, run_gpu_group
    from workload import get_config

    cfg = get_config("tiny_f32").with_(
        name="waves_long_chunks", layers=1, num_q_heads=128, num_kv_heads=16, head_dim=128, prompt_lens=(40, 33, 64, 20),
        slots_per_prompt=16, samples_per_prompt=16, length_dist=("uniform", 2290, 2300), max_suffix_len=2300,
        dtype="bf16", seed=31, pool_rows=1 << 12)
    wl, log, _, captured, tokens, _ = run_gpu_group(cfg, "fifo", entry="decode_step_layers", split=2048, window=32,
                                                    capture=lambda k: k in (1000, 2289))
    assert np.array_equal(tokens, wl.L) and len(captured) == 2
    check_against_oracle(cfg, wl, log, captured)
