"""Context splits whose tiles are not drawn, on a chip that is full: shapes on both sides of the rule that decides
whether the wavefronts with fp rows are kept together in the first workgroups.  Against the oracle, with equal rows,
padding slots and rows of different lengths."""
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [  # rows, kv heads, d, G, window, tokens, dtype, bits
    (32, 2, 64, 32, 32, 832, "f16", 2),       # 4 splits; fewer than two tiles a wavefront: together
    (32, 2, 64, 32, 32, 3936, "f16", 2),      # 2 to 5 tiles a wavefront: spread
    (32, 2, 128, 64, 64, 2048, "bf16", 4),
    (32, 2, 96, 64, 42, 1700, "bf16", 2),     # padding
    (8, 1, 128, 32, 32, 5000, "f16", 2),      # few workgroups: spread
]


@pytest.mark.parametrize("B,Hkv,d,G,W,L,dt,bits", CASES)
def test_equal_rows(B, Hkv, d, G, W, L, dt, bits):
    wl = U.make_wl(B=B, Hq=4 * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    dc = U.build_gpu_prefill(wl, 41, L)
    ocs = {bh: U.build_oracle(wl, 41, L, *bh) for bh in ((0, 0), (B - 1, Hkv - 1))}
    for rep in range(2):
        U.check_attention(dc, ocs, wl, inputs.queries(41, rep, wl))


@pytest.mark.parametrize("L", [832, 3936])
def test_rows_of_different_lengths(L):
    import torch
    from oracle import attention
    from oracle.cache import SliceCache
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=32, Hq=8, Hkv=2, d=64, G=32, F=64)
    lengths = [L - 13 * b for b in range(32)]
    K, V = inputs.batch_kv(43, 0, L, wl)
    cfg = binding.make_config(32, 8, 2, 64, 64, 32, "f16", U.q_capacity_for(wl, L))
    dc = binding.DeviceCacheSeq(cfg)
    dc.prefill_seq(U.to_dev(K, "f16"), U.to_dev(V, "f16"), lengths)
    q = inputs.queries(43, 0, wl)
    out = dc.decode_attn_seq(U.to_dev(q, "f16"))
    torch.cuda.synchronize()
    out = out.float().cpu().numpy()
    for b in (0, 17, 31):
        oc = SliceCache(32, 32, 64, "f16", 2)
        oc.append_block(K[b, 1, :lengths[b]], V[b, 1, :lengths[b]])
        want = attention.decode_attention(oc, q[b, 4:8])
        U.assert_outputs_close(out[b, 4:8], want, "f16", "row %d" % b)
