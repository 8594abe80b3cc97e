"""Launches with at most two units of fp rows or tiles to a wavefront of 8, which take one split (csrc/lq_attn.hip,
plan_decode), and the next that do not, against the oracle."""
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [  # rows, kv heads, d, G, window, tokens, dtype, bits, whether one split is planned
    (2, 8, 128, 64, 128, 300, "bf16", 2, True),       # 10 units, no tile
    (1, 4, 64, 32, 256, 767, "f16", 4, True),         # 24 units, no tile
    (1, 4, 64, 32, 256, 775, "f16", 2, False),        # 17 units and 8 tiles
    (2, 8, 128, 64, 128, 520, "bf16", 2, True),       # 9 units and 4 tiles
    (2, 8, 96, 64, 85, 500, "f16", 2, True),          # padding
    (1, 8, 128, 32, 64, 520, "f16", 2, False),        # fp16, four channel groups
]


@pytest.mark.parametrize("B,Hkv,d,G,W,L,dt,bits,one", CASES)
def test_few_items(B, Hkv, d, G, W, L, dt, bits, one):
    from paper_2503_19950_amd import binding
    wl = U.make_wl(B=B, Hq=4 * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    dc = U.build_gpu_prefill(wl, 71, L)
    plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
    assert (plan.splits == 1) == one
    ocs = {bh: U.build_oracle(wl, 71, L, *bh) for bh in ((0, 0), (B - 1, Hkv - 1))}
    for rep in range(2):
        U.check_attention(dc, ocs, wl, inputs.queries(71, rep, wl))
