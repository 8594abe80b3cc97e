"""The fused append and the merge with five to eight query heads in a workgroup (two sets of four, the second one short):
decode_step and decode_step_seq against the oracle, outputs and cache, with one and with several head groups per kv head, of
which only the first may store the new row; with 4 wavefronts and 4 bits; recorded into a graph; and the merge of three heads,
which leaves wavefronts idle, by one wavefront a head and by all."""
import pytest

from oracle import attention
from oracle.cache import SliceCache
from paper_2503_19950_amd import inputs
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

STEPS = [  # rows, kv heads, query heads per kv head, d, G, window, tokens, dtype, bits, wavefronts, head groups per kv head
    (2, 2, 5, 64, 32, 32, 500, "f16", 2, 8, 1),
    (1, 2, 7, 128, 64, 64, 1500, "bf16", 2, 8, 1),
    (2, 1, 7, 96, 64, 42, 640, "bf16", 2, 8, 1),          # padding
    (36, 8, 5, 64, 32, 32, 300, "f16", 4, 4, 1),          # 4 bits, 4 wavefronts
    (40, 8, 8, 64, 32, 64, 1000, "f16", 4, 4, 1),
    (48, 4, 10, 64, 32, 32, 1700, "f16", 2, None, 2),     # two groups of five
    (12, 4, 14, 128, 64, 64, 2300, "bf16", 2, None, 2),   # two of seven
    (24, 4, 16, 64, 32, 64, 5200, "f16", 2, None, 2),     # two of eight
]


def _prompt(B, Hkv, gh, d, G, W, L, dt, bits):
    wl = U.make_wl(B=B, Hq=gh * Hkv, Hkv=Hkv, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    own = {(0, 0), (B - 1, Hkv - 1)}
    K, V = U.batch_kv_sampled(81, 0, L + 4, wl, own)
    return wl, K, V, own


def _oracle(wl, K, V, b, h, n):
    oc = SliceCache(wl["F"] // 2, wl["G"], wl["d"], wl["dtype"], wl["bits"])
    oc.append_block(K[b, h, :n], V[b, h, :n])
    return oc


@pytest.mark.parametrize("B,Hkv,gh,d,G,W,L,dt,bits,waves,groups", STEPS)
def test_decode_step(B, Hkv, gh, d, G, W, L, dt, bits, waves, groups):
    import torch
    from paper_2503_19950_amd import binding
    wl, K, V, own = _prompt(B, Hkv, gh, d, G, W, L, dt, bits)
    Kd, Vd = U.to_dev(K, dt), U.to_dev(V, dt)
    dc = U.new_cache(wl, L + 4)
    dc.prefill(Kd[:, :, :L].contiguous(), Vd[:, :, :L].contiguous())
    ocs = {bh: _oracle(wl, K, V, *bh, L) for bh in own}
    for t in range(L, L + 3):
        q = inputs.queries(81, t, wl)
        out = dc.decode_step(Kd[:, :, t:t + 1].contiguous(), Vd[:, :, t:t + 1].contiguous(), U.to_dev(q, dt))
        plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
        assert plan.blocks == plan.splits * B * Hkv * groups and waves in (None, plan.waves_per_block)
        torch.cuda.synchronize()
        out = out.float().cpu().numpy()
        for (b, h), oc in ocs.items():
            oc.append(K[b, h, t], V[b, h, t])
            want = attention.decode_attention(oc, q[b, h * gh:(h + 1) * gh])
            U.assert_outputs_close(out[b, h * gh:(h + 1) * gh], want, dt, "token %d (%d, %d)" % (t, b, h))
    for (b, h), oc in ocs.items():
        U.check_state(dc, oc, wl, b, h)


@pytest.mark.parametrize("B,Hkv,gh,d,G,W,L,step,bits", [
    (6, 2, 7, 128, 32, 64, 1500, 110, 2),
    (12, 2, 5, 64, 32, 32, 900, 31, 4),
    (20, 4, 14, 64, 32, 64, 3000, 41, 2),                 # two groups of seven
    (5, 2, 7, 96, 64, 42, 700, 90, 2),                    # padding
])
def test_decode_step_of_rows_of_different_lengths(B, Hkv, gh, d, G, W, L, step, bits):
    import torch
    wl, K, V, _ = _prompt(B, Hkv, gh, d, G, W, L, "f16", bits)
    lengths = [L - step * b for b in range(B)]
    lengths = [n - ((n + 1) % W == 0) for n in lengths]      # no window fills at the step
    Kd, Vd = U.to_dev(K, "f16"), U.to_dev(V, "f16")
    from paper_2503_19950_amd import binding
    cfg = binding.make_config(B, gh * Hkv, Hkv, d, 2 * W, G, "f16", U.q_capacity_for(wl, L + 4), bits)
    dc = binding.DeviceCacheSeq(cfg)
    dc.prefill_seq(Kd[:, :, :L].contiguous(), Vd[:, :, :L].contiguous(), lengths)
    kn, vn = (torch.stack([x[b, :, lengths[b]:lengths[b] + 1] for b in range(B)]).contiguous() for x in (Kd, Vd))
    q = inputs.queries(83, 0, wl)
    out = dc.decode_step_seq(kn, vn, U.to_dev(q, "f16"))
    torch.cuda.synchronize()
    out = out.float().cpu().numpy()
    for b in (0, B // 2, B - 1):
        for h in (0, Hkv - 1):
            oc = _oracle(wl, K, V, b, h, lengths[b] + 1)
            want = attention.decode_attention(oc, q[b, h * gh:(h + 1) * gh])
            U.assert_outputs_close(out[b, h * gh:(h + 1) * gh], want, "f16", "row %d head %d" % (b, h))
            U.check_state(dc, oc, wl, b, h, counts=dc.view(b))


def test_a_graph_of_two_sets_replays():
    import torch
    wl = U.make_wl(B=2, Hq=14, Hkv=2, d=128, G=32, F=128)
    dc = U.build_gpu_prefill(wl, 85, 3000)
    qs = [U.to_dev(inputs.queries(85, s, wl), "f16") for s in range(3)]
    eager = [dc.decode_attn(q).clone() for q in qs]
    q_in, out = qs[0].clone(), torch.empty_like(qs[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dc.decode_attn(q_in, out)
    for rep in range(3):
        for i, q in enumerate(qs):
            q_in.copy_(q)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager[i]), (rep, i)
            assert torch.equal(dc.decode_attn(qs[(i + 1) % 3]), eager[(i + 1) % 3])


@pytest.mark.parametrize("d,L,splits", [(64, 14312, 30), (128, 7400, 17), (128, 16384, 34), (64, 20000, 41)])
def test_merge_of_three_heads(d, L, splits):
    from paper_2503_19950_amd import binding
    wl = U.make_wl(Hq=3, Hkv=1, d=d, G=32, F=128)
    dc = U.build_gpu_prefill(wl, 87, L)
    plan = binding.logquant_decode_plan(dc.cfg, dc.c.n_fp, dc.c.n_q)
    assert (plan.splits, plan.blocks) == (splits, splits)
    U.check_attention(dc, {(0, 0): U.build_oracle(wl, 87, L, 0, 0)}, wl, inputs.queries(87, 0, wl))


def test_the_stream_of_a_call_is_the_current_one():
    """The handle that the calls are given against torch's public one, on the default stream and on another, for devices with
    and without an index."""
    import torch
    for device in ("cuda", "cuda:0"):
        from paper_2503_19950_amd import binding
        dc = binding.DeviceCache(binding.make_config(1, 4, 1, 128, 64, 32, "f16", 128), device=device)
        assert dc._stream() == torch.cuda.current_stream(dc.device).cuda_stream
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            assert dc._stream() == side.cuda_stream == torch.cuda.current_stream(dc.device).cuda_stream
