"""GPU: per-layer launches that give each short response and each merge a wavefront (work-groups that
do not fit the GPU at once, responses of at most 64 tokens), and the steps on either side of that
line, against the oracle.

Lengths reach 70, so a decode crosses the line both ways; slot counts are no multiple of the four
wavefronts, and slots fall idle at the end.  Merges take one round of loads and two.  Tolerance: the
bf16 path's 1e-2."""

import numpy as np
import pytest

from tests.gpu_harness import check_against_oracle, run_gpu_group
from workload import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hpk,prompts,m,kv_fp8,exchange", [
    (128, 2, (600,), 41, False, None), (128, 2, (600,), 41, False, 0), (128, 4, (1, 130, 257), 15, False, None),
    (64, 1, (300,), 47, False, None), (64, 8, (33, 129, 0, 64), 11, False, None), (128, 2, (257,), 50, True, None),
    (128, 4, tuple(range(10, 26)), 3, False, None), (128, 8, (260, 40, 300), 15, False, None),
    (128, 4, (1400, 130, 1000, 900), 16, False, None)])
@pytest.mark.parametrize("entry", ["decode_step", "decode_step_static"])
def test_short_responses(d, hpk, prompts, m, kv_fp8, exchange, entry):
    cfg = get_config("qwen3_1p7b_l1_g32").with_(
        name=f"short_d{d}_hpk{hpk}_m{m}", layers=2, num_q_heads=8 * hpk, num_kv_heads=8, head_dim=d, prompt_lens=prompts,
        slots_per_prompt=m, samples_per_prompt=m + 1, length_dist=("uniform", 1, 70), max_suffix_len=70, seed=31)
    wl, log, steps, captured, tokens, _ = run_gpu_group(cfg, "fifo", entry=entry, kv_fp8=kv_fp8, exchange=exchange,
                                                        capture=lambda t: t % 16 in (0, 1) or 62 <= t < 66)
    assert np.array_equal(tokens, wl.L)
    # the line itself: chunks of 128 prompt tokens and of 256 response tokens, 512 work-groups at once
    def waves(row):
        live = [e for e in row if e is not None]
        chunks = [-(-prompts[p] // (128 if m * hpk >= 16 else 256)) for p in {e[0] for e in live}]
        busy = (sum(chunks) + 2 * len(live)) * 8
        rounds = -(-(max(chunks) + 1) // (24 if hpk * d <= 256 else 8 if hpk * d <= 512 else 4))
        return max(e[2] for e in live) <= 64 and (busy > 512 if rounds == 1 else rounds <= 3 and busy > 1024)

    assert any(waves(log[t]) for t in captured) and not all(waves(log[t]) for t in captured)
    _, checked = check_against_oracle(cfg, wl, log, captured, kv_fp8=kv_fp8)
    assert checked > 0
