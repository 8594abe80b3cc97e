"""Five to eight query heads per kv head, which large launches work on in one workgroup (two sets of four, the second
one short where there are fewer than eight): shapes on both sides of the rule (csrc/lq_internal.h, heads_per_group),
with one split, with splits that one wavefront merges and with more of them, with padding slots and with rows of
different lengths.  Against the oracle, the tolerance of the other attention tests."""
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [  # rows, kv heads, query heads per kv head, d, G, window, tokens, dtype, bits, workgroups per kv head and split
    (1, 2, 8, 128, 64, 64, 3000, "bf16", 2, 2),          # small: two sets, a workgroup each
    (2, 2, 5, 64, 32, 32, 500, "f16", 2, 1),             # four is no divisor
    (2, 1, 7, 96, 64, 42, 700, "bf16", 2, 1),            # padding
    (1, 1, 7, 128, 32, 64, 16384, "f16", 4, 1),          # more splits than one wavefront merges
    (1, 1, 6, 64, 32, 32, 300, "f16", 2, 2),
    (80, 8, 8, 128, 32, 64, 1000, "f16", 2, 1),          # one split
    (48, 8, 6, 128, 64, 128, 1300, "bf16", 2, 1),
    (16, 8, 8, 128, 32, 32, 4000, "f16", 4, 1),          # several splits
    (16, 8, 8, 96, 64, 85, 6000, "bf16", 2, 1),          # padding
    (4, 4, 8, 64, 128, 128, 60000, "f16", 2, 1),
]


@pytest.mark.parametrize("B,Hkv,gh,d,G,W,L,dt,bits,groups", CASES)
def test_equal_rows(B, Hkv, gh, d, G, W, L, dt, bits, groups):
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=gh * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    dc = U.build_gpu_prefill(wl, 51, L)
    plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
    assert plan.blocks == plan.splits * B * Hkv * groups
    ocs = {bh: U.build_oracle(wl, 51, L, *bh) for bh in ((0, 0), (B - 1, Hkv - 1))}
    for rep in range(2):
        U.check_attention(dc, ocs, wl, inputs.queries(51, rep, wl))


@pytest.mark.parametrize("B,Hkv,gh,d,G,W,L,step,bits", [
    (40, 4, 8, 128, 32, 64, 2200, 17, 2),
    (24, 4, 7, 96, 64, 85, 5000, 60, 2),                 # padding
    (12, 2, 5, 64, 32, 32, 900, 31, 4),
])
def test_rows_of_different_lengths(B, Hkv, gh, d, G, W, L, step, bits):
    import torch
    from oracle import attention
    from oracle.cache import SliceCache
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=gh * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, bits=bits)
    lengths = [L - step * b for b in range(B)]
    K, V = inputs.batch_kv(53, 0, L, wl)
    cfg = binding.make_config(B, gh * Hkv, Hkv, d, 2 * W, G, "f16", U.q_capacity_for(wl, L), bits)
    dc = binding.DeviceCacheSeq(cfg)
    dc.prefill_seq(U.to_dev(K, "f16"), U.to_dev(V, "f16"), lengths)
    q = inputs.queries(53, 0, wl)
    out = dc.decode_attn_seq(U.to_dev(q, "f16"))
    torch.cuda.synchronize()
    out = out.float().cpu().numpy()
    for b in (0, B // 2 + 1, B - 1):
        oc = SliceCache(W, G, d, "f16", bits)
        oc.append_block(K[b, 1, :lengths[b]], V[b, 1, :lengths[b]])
        want = attention.decode_attention(oc, q[b, gh:2 * gh])
        U.assert_outputs_close(out[b, gh:2 * gh], want, "f16", "row %d" % b)
