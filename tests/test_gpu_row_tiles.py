"""GPU: row tiles (the prefix below 16 rows or in fp32, fp32 responses of 4 and 8 rows) at the edges
of their 16- and 32-token tiles, load rounds and chunks, through both launches, against the oracle.

Tolerances are those of the paths: fp32 1e-5 (fp32 products and sums of at most a few hundred terms),
bf16 1e-2 (the responses' probabilities are rounded to bf16)."""

import numpy as np
import pytest

from tests.gpu_harness import check_against_oracle, run_gpu_group
from workload import get_config

pytestmark = pytest.mark.gpu

PROMPTS = (1, 15, 16, 17, 33, 64, 65, 257)  # prompts of one batch: below, at and above tiles, rounds, a chunk


@pytest.mark.parametrize("entry", ["decode_step", "decode_step_layers"])
@pytest.mark.parametrize("dtype,d,hpk,m", [("f32", 128, 1, 2), ("f32", 64, 2, 8), ("f32", 128, 4, 2), ("f32", 64, 8, 1),
                                           ("bf16", 128, 4, 3), ("bf16", 64, 1, 5)])
def test_row_tiles(dtype, d, hpk, m, entry):
    cfg = get_config("tiny_f32").with_(
        name=f"rows_{dtype}_d{d}_hpk{hpk}_m{m}", layers=2, num_q_heads=2 * hpk, num_kv_heads=2, head_dim=d,
        prompt_lens=PROMPTS, slots_per_prompt=m, samples_per_prompt=m + 1, length_dist=("uniform", 1, 70),
        max_suffix_len=70, dtype=dtype, seed=29)
    wl, log, steps, captured, tokens, _ = run_gpu_group(cfg, "fifo", entry=entry)
    assert np.array_equal(tokens, wl.L)
    _, checked = check_against_oracle(cfg, wl, log, captured)
    assert checked == cfg.layers * int(wl.L.sum())
