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


@pytest.mark.parametrize("entry", ["layer", "layers"])
@pytest.mark.parametrize("dtype,d,hpk,m", [("bf16", 64, 2, 3), ("bf16", 128, 2, 3), ("f32", 128, 2, 3)])
def test_infinite_values(dtype, d, hpk, m, entry):
    """An infinite V element of the prompt makes its output element that infinity (its weight is not
    zero) and leaves the others as they are, whatever rounding the weights take on the tile."""
    import torch

    from paper_2506_22950_amd import infs

    plen, hkv, layers = 150, 2, 2
    gen = torch.Generator(device="cuda").manual_seed(d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = infs.Context(infs.make_config(
        num_layers=layers, num_q_heads=hkv * hpk, num_kv_heads=hkv, head_dim=d, num_prompts=1, slots_per_prompt=m,
        samples_per_prompt=m, max_prompt_len=plen, max_suffix_len=16, dtype=infs.F32 if dtype == "f32" else infs.BF16),
        stream=torch.cuda.current_stream())
    assert ctx.kernel_info()["mfma"] == 0

    def rows(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(dt)

    k, v = rows(layers, plen, hkv, d), rows(layers, plen, hkv, d)
    # (token, KV head, dim, value): in the first group of a wavefront, in the last, in two wavefronts
    for tok, g, dim, x in ((3, 0, 5, 1), (149, 0, 6, -1), (70, 1, d - 1, 1), (130, 1, d - 1, 1), (64, 1, 0, -1)):
        v[:, tok, g, dim] = x * float("inf")
    q, kn, vn = rows(layers, m, hkv * hpk, d), rows(layers, m, hkv, d), rows(layers, m, hkv, d)
    o = torch.empty(layers, m, hkv * hpk, d, device="cuda")
    for layer in range(layers):
        ctx.prefill_shared(0, layer, plen, k[layer], v[layer])
    for s in range(m):
        ctx.refill_slot(s, 0, s)
    if entry == "layers":
        ctx.decode_step_layers(q.data_ptr(), kn.data_ptr(), vn.data_ptr(), o.data_ptr())
    else:
        for layer in range(layers):
            ctx.decode_step(layer, q[layer].data_ptr(), kn[layer].data_ptr(), vn[layer].data_ptr(), o[layer].data_ptr())
    ctx.end_step()
    got = o.double().cpu()
    ctx.destroy()
    k, v, q, kn, vn = (x.double().cpu() for x in (k, v, q, kn, vn))
    for layer in range(layers):
        for s in range(m):
            for h in range(hkv * hpk):
                kk = torch.cat([k[layer, :, h // hpk], kn[layer, s, None, h // hpk]])
                vv = torch.cat([v[layer, :, h // hpk], vn[layer, s, None, h // hpk]])
                p = torch.softmax(kk @ q[layer, s, h] / d ** 0.5, 0)
                assert p.min() > 0
                want = (p[:, None] * vv).sum(0)
                inf = torch.isinf(want)
                assert int(inf.sum()) == 2 and torch.equal(got[layer, s, h][inf], want[inf])
                # fp32 1e-5, bf16 1e-2: the tolerances of the paths
                assert (got[layer, s, h] - want)[~inf].abs().max() <= (1e-5 if dtype == "f32" else 1e-2)
