"""Context splits whose tiles are not drawn: shapes on both sides of the rule (csrc/lq_schedule.h, keeps_units_together)
that decides whether the wavefronts with fp rows are kept together in the first workgroups.  Against the oracle, with
equal rows, padding slots and rows of different lengths; that a shape lies on the side it is meant for is asserted."""
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [  # rows, kv heads, d, G, window, tokens, dtype, bits, where the wavefronts with fp rows are
    (32, 2, 64, 32, 32, 832, "f16", 2, "one split"),
    (32, 2, 64, 32, 32, 3936, "f16", 2, "spread"),        # 2 to 5 tiles a wavefront
    (32, 2, 128, 64, 64, 2048, "bf16", 4, "spread"),      # an eighth of the wavefronts, not more
    (32, 2, 96, 64, 42, 1700, "bf16", 2, "spread"),       # padding
    (8, 1, 128, 32, 32, 5000, "f16", 2, "spread"),        # few workgroups
    (8, 8, 128, 32, 128, 2048, "f16", 2, "together"),
    (32, 2, 64, 128, 128, 1100, "f16", 4, "together"),
    (32, 2, 96, 64, 85, 1100, "bf16", 2, "together"),     # padding
    (32, 2, 64, 64, 85, 1500, "bf16", 4, "together"),     # padding
]


def where_the_units_are(plan, n_fp, n_q, G, W):
    """Which program a launch of 8 wavefronts a workgroup takes.  n_fp, n_q: of the longest row."""
    slots = -(-W // G) * G
    tiles = n_q // slots * -(-W // 64) if G >= 64 else -(-n_q // 64)
    waves = 8 * plan.splits
    assert plan.waves_per_block == 8
    if plan.splits == 1:
        return "one split"
    for_tiles = waves - plan.fp_waves
    assert tiles < 5 * for_tiles, "the tiles are drawn"
    return "together" if plan.blocks >= 256 and tiles < 2 * for_tiles and 8 * plan.fp_waves > waves else "spread"


@pytest.mark.parametrize("B,Hkv,d,G,W,L,dt,bits,where", CASES)
def test_equal_rows(B, Hkv, d, G, W, L, dt, bits, where):
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=4 * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    dc = U.build_gpu_prefill(wl, 41, L)
    plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
    assert where_the_units_are(plan, dc.c.n_fp, dc.c.n_q, G, W) == where
    ocs = {bh: U.build_oracle(wl, 41, L, *bh) for bh in ((0, 0), (B - 1, Hkv - 1))}
    for rep in range(2):
        U.check_attention(dc, ocs, wl, inputs.queries(41, rep, wl))


@pytest.mark.parametrize("B,Hkv,d,G,W,L,step,bits,where", [
    (32, 2, 64, 32, 32, 832, 13, 2, "spread"),            # 192 workgroups
    (32, 2, 64, 32, 32, 3936, 13, 2, "spread"),
    (16, 4, 128, 32, 64, 1100, 5, 4, "together"),
    (16, 4, 64, 64, 128, 1100, 13, 2, "together"),
    (16, 4, 128, 32, 85, 1100, 5, 2, "together"),         # padding
])
def test_rows_of_different_lengths(B, Hkv, d, G, W, L, step, bits, where):
    import torch
    from oracle import attention
    from oracle.cache import SliceCache
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=4 * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, bits=bits)
    lengths = [L - step * b for b in range(B)]
    K, V = inputs.batch_kv(43, 0, L, wl)
    cfg = binding.make_config(B, 4 * Hkv, Hkv, d, 2 * W, G, "f16", U.q_capacity_for(wl, L), bits)
    dc = binding.DeviceCacheSeq(cfg)
    dc.prefill_seq(U.to_dev(K, "f16"), U.to_dev(V, "f16"), lengths)
    plan = binding.logquant_decode_plan_seq(cfg, list(dc.n_fp), list(dc.n_q))
    assert where_the_units_are(plan, max(dc.n_fp), max(dc.n_q), G, W) == where
    q = inputs.queries(43, 0, wl)
    out = dc.decode_attn_seq(U.to_dev(q, "f16"))
    torch.cuda.synchronize()
    out = out.float().cpu().numpy()
    for b in (0, B // 2 + 1, B - 1):
        oc = SliceCache(W, G, d, "f16", bits)
        oc.append_block(K[b, 1, :lengths[b]], V[b, 1, :lengths[b]])
        want = attention.decode_attention(oc, q[b, 4:8])
        U.assert_outputs_close(out[b, 4:8], want, "f16", "row %d" % b)
