"""GPU: the prefill kernels at the edges of their tiles (32-token blocks, rounds of 1024 16-byte
units), for every row size and odd KV head counts: the prefix store gives back the bits it was
given -- a copy, so the tolerance is zero -- and a prompt leaves its neighbours' rows alone."""

import numpy as np
import pytest

from paper_2506_22950_amd import infs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cache,d,m,hpk", [("f32", 64, 2, 2), ("f32", 128, 8, 2), ("bf16", 64, 3, 1), ("bf16", 128, 4, 1),
                                           ("bf16", 64, 8, 2), ("bf16", 128, 16, 2), ("e4m3", 128, 16, 1)])
@pytest.mark.parametrize("hkv", [1, 3, 8])
@pytest.mark.parametrize("plen", [1, 31, 32, 33, 257])
def test_prefill_round_trip(cache, d, m, hpk, hkv, plen):
    import torch

    f32, fp8 = cache == "f32", cache == "e4m3"
    gen = torch.Generator(device="cuda").manual_seed(plen * 100 + hkv)
    lens = (plen, 40)
    ctx = infs.Context(infs.make_config(
        num_layers=1, num_q_heads=hkv * hpk, num_kv_heads=hkv, head_dim=d, num_prompts=2, slots_per_prompt=m,
        samples_per_prompt=m, max_prompt_len=max(lens), max_suffix_len=16, dtype=infs.F32 if f32 else infs.BF16,
        flags=infs.FLAG_KV_FP8 if fp8 else 0), stream=torch.cuda.current_stream())
    given = []
    for p, n in enumerate(lens):
        shape = (n, hkv, d)
        if fp8:  # finite values across the E4M3 range; rounding to nearest even, saturating
            kv = [(torch.randn(shape, generator=gen, device="cuda") * 100).to(torch.bfloat16) for _ in range(2)]
            want = [x.float().clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for x in kv]
        else:  # every bit pattern, infinities and NaN among them
            dt, lo, hi = (torch.int32, -2 ** 31, 2 ** 31) if f32 else (torch.int16, -2 ** 15, 2 ** 15)
            kv = want = [torch.randint(lo, hi, shape, generator=gen, device="cuda", dtype=dt) for _ in range(2)]
        ctx.prefill_shared(p, 0, n, kv[0], kv[1])
        given.append((kv, want))
    for p, n in enumerate(lens):
        got = ctx.read_prefix(p, 0, n)
        for name, g, w in zip("KV", got, given[p][1]):
            w = w.cpu().numpy()
            assert np.array_equal(g.view(w.dtype), w), (p, name)
    ctx.destroy()
