"""Decode attention where rows at original precision weigh far more than each of very many quantized rows with small
value scales (a recent token at the centre of attention over a long diffuse context), with a single context split,
where a wavefront takes fp rows and then quantized tiles.  The quantized rows' probabilities and their products with
the value scales are fp16 operands; their precision must not depend on the weight of the fp rows.

The keys of the quantized rows are zero, so that their weights are all equal, and the value rows of the heavy fp rows
are zero, so that the output is the quantized rows' share alone: an error in those operands is an error of the output.
Bound per element: half an ulp of T, plus the noise of fp32 sums and, for bf16 caches, of one fp16 rounding of p * vs
(gpu_util.COMPUTE_NOISE), relative to the output."""
import numpy as np
import pytest

from oracle import attention
from oracle.cache import SliceCache
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# gap: log2 of a heavy row's weight over a quantized row's; wpb: wavefronts per workgroup the planner picks
CASES = [
    ("f16_g32", dict(B=64, Hq=32, Hkv=8, d=128, G=32, F=256), 16384, 14.4, 4, False),
    ("bf16_g64_d96", dict(B=16, Hq=32, Hkv=32, d=96, G=64, F=384, dtype="bf16"), 16384, 20.4, 4, False),
    ("bf16_g32_rows_apart", dict(B=64, Hq=32, Hkv=8, d=128, G=32, F=256, dtype="bf16"), 8192, 20.4, 8, True),
    ("f16_g64_twelve", dict(B=32, Hq=32, Hkv=8, d=128, G=64, F=256), 16384, 14.4, 12, False),
    ("bits4_f16_g32", dict(B=64, Hq=32, Hkv=8, d=128, G=32, F=256, bits=4), 8192, 13.4, 4, False),
]


@pytest.mark.parametrize("name,kw,L,gap,wpb,seq", CASES, ids=[c[0] for c in CASES])
def test_quantized_share_keeps_its_precision_beside_heavy_fp_rows(name, kw, L, gap, wpb, seq):
    import torch
    from paper_2503_19950_amd import binding
    wl = U.make_wl(**kw)
    dt, d, W, bits = wl["dtype"], wl["d"], wl["F"] // 2, wl.get("bits", 2)
    gh = wl["Hq"] // wl["Hkv"]
    L += W // 2 + 5
    rng = np.random.default_rng([2503_19950, L, d, bits])
    steps = (1 << bits) - 1
    step = 1.375 * 2.0 ** -9 * 3 / steps
    pos = SliceCache(W, wl["G"], d, dt, bits)            # which positions stay at original precision
    pos.append_block(np.zeros((L, d)), np.zeros((L, d)))
    K = np.zeros((L, d), np.float32)
    V = (rng.integers(0, steps + 1, (L, d)) * step).astype(np.float32)
    sign = np.where(rng.random(d) < 0.5, -1.0, 1.0)
    heavy = [p for i, p in enumerate(pos.pos_fp) if i % 32 == 5]
    K[heavy] = sign * gap * np.log(2.0) / np.sqrt(d)
    V[heavy] = 0.0
    K, V = (torch.from_numpy(x).to(binding.torch_dtype(dt)) for x in (K, V))
    oc = SliceCache(W, wl["G"], d, dt, bits)
    oc.append_block(K.float().numpy(), V.float().numpy())
    q = np.broadcast_to(sign, (wl["B"], wl["Hq"], d)).astype(np.float32)
    want = attention.decode_attention(oc, q[0, :gh])
    print("case", name, "out", np.abs(want).max(), flush=True)

    every = lambda x: x.cuda()[None, None].expand(wl["B"], wl["Hkv"], L, d).contiguous()  # noqa: E731
    cfg = binding.make_config(wl["B"], wl["Hq"], wl["Hkv"], d, wl["F"], wl["G"], dt, U.q_capacity_for(wl, L), bits)
    if seq:
        dc = binding.DeviceCacheSeq(cfg)
        dc.prefill_seq(every(K), every(V), [L] * wl["B"])
        plan = binding.logquant_decode_plan_seq(cfg, list(dc.n_fp), list(dc.n_q))
        out = dc.decode_attn_seq(U.to_dev(q, dt))
    else:
        dc = binding.DeviceCache(cfg)
        dc.prefill(every(K), every(V))
        plan = binding.logquant_decode_plan(cfg, dc.c.n_fp, dc.c.n_q)
        out = dc.decode_attn(U.to_dev(q, dt))
    assert plan.splits == 1 and plan.waves_per_block == wpb, (plan.splits, plan.waves_per_block)
    got = out.double().cpu().numpy().reshape(-1, gh, d)
    err = np.abs(got - want)
    least = {"f16": 2.0 ** -14, "bf16": 2.0 ** -126}[dt]      # smallest normal value of T
    half_ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), least))) - U.MANT_BITS[dt])
    bound = half_ulp + U.COMPUTE_NOISE[dt] * np.abs(want)
    print("  largest error: %.2e of the output, %.2f of the bound" % ((err / np.abs(want)).max(), (err / bound).max()),
          flush=True)
    assert (err <= bound).all(), (err / bound).max()
