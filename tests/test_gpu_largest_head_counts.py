"""Nearly as many heads as a launch can have, in one batch row: heads beyond 32768 divide by a number as large."""
import numpy as np
import pytest

from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def test_query_heads_of_one_kv_head():
    wl = U.make_wl(B=1, Hq=60001, Hkv=1, d=64, G=32, F=64)      # odd: a head to each workgroup
    dc = U.build_gpu_prefill(wl, 830, 200)
    q = inputs.queries(830, 0, wl)
    U.check_attention(dc, {(0, 0): U.build_oracle(wl, 830, 200, 0, 0)}, wl, q)


def test_kv_heads_with_counts_per_row():
    from paper_2503_19950_amd import binding as B
    heads, L = 60000, 5
    cfg = B.make_config(1, heads, heads, 64, 4, 32, "f16", 64)
    rng = np.random.default_rng(831)
    K, V = (rng.standard_normal((1, heads, L, 64)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((1, heads, 64)).astype(np.float16)
    dc = B.DeviceCacheSeq(cfg)
    dc.prefill_seq(U.to_dev(K, "f16"), U.to_dev(V, "f16"), [L])
    out = dc.decode_attn_seq(U.to_dev(q, "f16")).float().cpu().numpy()
    p = np.exp(np.einsum("hd,hld->hl", q[0], K[0], dtype=np.float64) / 8)
    want = np.einsum("hl,hld->hd", p / p.sum(axis=1, keepdims=True), V[0], dtype=np.float64)
    U.assert_outputs_close(out[0], want, "f16", "60000 kv heads")
