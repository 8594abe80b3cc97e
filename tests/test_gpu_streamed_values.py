"""Launches that read the quantized values past the caches (csrc/lq_internal.h, streams_values) and the next that do not,
with 4, 8 and 12 wavefronts a workgroup, padding slots and rows of different lengths, against the oracle."""
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [  # rows, kv heads, query heads per kv head, d, G, window, tokens, dtype, wavefronts, whether it reads 64 to 160 MB
    (4, 8, 4, 128, 64, 64, 24000, "bf16", 12, False),
    (4, 8, 4, 128, 64, 64, 25000, "bf16", 12, True),
    (64, 8, 2, 96, 32, 32, 1500, "f16", 4, True),
    (16, 8, 4, 128, 32, 128, 4000, "f16", 8, True),
    (8, 8, 4, 128, 64, 42, 13000, "bf16", 12, True),     # padding
    (12, 8, 1, 64, 64, 64, 40000, "f16", 4, True),
    (64, 8, 4, 128, 32, 32, 3000, "f16", 4, False),      # above
]


@pytest.mark.parametrize("B,Hkv,gh,d,G,W,L,dt,wpb,streamed", CASES)
def test_equal_rows(B, Hkv, gh, d, G, W, L, dt, wpb, streamed):
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=gh * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt)
    dc = U.build_gpu_prefill(wl, 61, L)
    plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
    assert (64000000 <= plan.bytes_read < 160000000) == streamed and plan.waves_per_block == wpb
    ocs = {bh: U.build_oracle(wl, 61, L, *bh) for bh in ((0, 0), (B - 1, Hkv - 1))}
    for rep in range(2):
        U.check_attention(dc, ocs, wl, inputs.queries(61, rep, wl))


def test_rows_of_different_lengths():
    import torch
    from oracle import attention
    from oracle.cache import SliceCache
    from paper_2503_19950_amd import binding
    B, Hkv, gh, d, G, W = 40, 8, 4, 128, 32, 64
    wl = U.make_wl(B=B, Hq=gh * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W)
    lengths = [3300 - 23 * b for b in range(B)]
    K, V = inputs.batch_kv(63, 0, max(lengths), wl)
    cfg = binding.make_config(B, gh * Hkv, Hkv, d, 2 * W, G, "f16", U.q_capacity_for(wl, max(lengths)))
    dc = binding.DeviceCacheSeq(cfg)
    dc.prefill_seq(U.to_dev(K, "f16"), U.to_dev(V, "f16"), lengths)
    assert binding.logquant_decode_plan_seq(cfg, list(dc.n_fp), list(dc.n_q)).bytes_read >= 64000000
    q = inputs.queries(63, 0, wl)
    out = dc.decode_attn_seq(U.to_dev(q, "f16"))
    torch.cuda.synchronize()
    out = out.float().cpu().numpy()
    for b in (0, B // 2 + 1, B - 1):
        oc = SliceCache(W, G, d, "f16")
        oc.append_block(K[b, 1, :lengths[b]], V[b, 1, :lengths[b]])
        want = attention.decode_attention(oc, q[b, gh:2 * gh])
        U.assert_outputs_close(out[b, gh:2 * gh], want, "f16", "row %d" % b)
