"""GPU: per-layer launches that give each short response and each merge a wavefront (work-groups that
do not fit the GPU at once, responses of at most 64 tokens), and the steps on either side of that
line, against the oracle.

Lengths reach 70, so a decode crosses the line both ways; slot counts are no multiple of the four
wavefronts, and slots fall idle at the end.  Tolerance: the bf16 path's 1e-2."""

import numpy as np
import pytest

from tests.gpu_harness import check_against_oracle, run_gpu_group
from workload import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hpk,prompts,m,kv_fp8,exchange", [
    (128, 2, (600,), 41, False, None), (128, 2, (600,), 41, False, 0), (128, 4, (1, 130, 257), 15, False, None),
    (64, 1, (300,), 47, False, None), (64, 8, (33, 129, 0, 64), 11, False, None), (128, 2, (257,), 50, True, None),
    (128, 4, tuple(range(10, 26)), 3, False, None)])
@pytest.mark.parametrize("entry", ["decode_step", "decode_step_static"])
def test_short_responses(d, hpk, prompts, m, kv_fp8, exchange, entry):
    cfg = get_config("qwen3_1p7b_l1_g32").with_(
        name=f"short_d{d}_hpk{hpk}_m{m}", layers=2, num_q_heads=8 * hpk, num_kv_heads=8, head_dim=d, prompt_lens=prompts,
        slots_per_prompt=m, samples_per_prompt=m + 1, length_dist=("uniform", 1, 70), max_suffix_len=70, seed=31)
    wl, log, steps, captured, tokens, _ = run_gpu_group(cfg, "fifo", entry=entry, kv_fp8=kv_fp8, exchange=exchange,
                                                        capture=lambda t: t % 16 in (0, 1) or 62 <= t < 66)
    assert np.array_equal(tokens, wl.L)
    _, checked = check_against_oracle(cfg, wl, log, captured, kv_fp8=kv_fp8)
    assert checked > 0
