"""Workloads of the LogQuant cache as a serving program has them: what is timed when the library's speed is
looked at.  Each case is a plain dict; `prepare` builds what the program holds before the call (prompts, caches,
new rows, queries), `run` makes one pass through the public entry points of paper_2503_19950_amd.binding.

Kinds of pass
  decode    `steps` decode steps of a model with `layers` layers, one cache per layer: per step and layer one
            token is appended and its query attends (decode_step); at the step that fills a window the token is
            appended, the window filtered (compress) and the query attends (decode_attn).  With `ragged` the rows
            of the batch have different lengths and fill their windows at their own pace (the per-sequence calls).
  prefill   one layer's cache is built from a whole prompt (prefill, or prefill_seq with one length per row).
"""
import math
import random

import torch

from paper_2503_19950_amd import binding

DEVICE = "cuda:0"


def _case(kind, B, Hq, Hkv, d, L, dtype, G, F, bits=2, layers=1, steps=1, ragged=False, dist="normal", sinks=0):
    """B rows, Hq query and Hkv kv heads of dimension d, L tokens (the longest row's with `ragged`), G quantization
    group size, F = 2W tokens kept at original precision after a filtering event, code width `bits`."""
    return dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, d=d, L=L, dtype=dtype, G=G, F=F, bits=bits, layers=layers, steps=steps,
                ragged=ragged, dist=dist, sinks=sinks)


def listed():
    long = dict(B=1, Hq=32, Hkv=8, d=128, L=131072, dtype="bf16", G=64, sinks=4)
    batch = dict(B=64, Hq=32, Hkv=8, d=128, L=4096, dtype="f16", G=32, F=256)
    llama = dict(B=8, Hq=32, Hkv=8, d=128, dtype="f16", G=32, F=256)
    return [
        # one user, short chat: a single launch of a fraction of a megabyte, all latency
        dict(name="decode_b1_512", **_case("decode", 1, 32, 8, 128, 512, "f16", 32, 128)),
        # a small batch of ordinary prompts, Llama-3-8B head shape
        dict(name="decode_b8_8k", **_case("decode", L=8192, layers=4, **llama)),
        # the step at which every window of that batch is full: append, filter and quantize, attend
        dict(name="window_fills_b8_8k", **_case("decode", L=8191, layers=4, **llama)),
        # one very long document, the context split over the whole GPU
        dict(name="decode_b1_128k", **_case("decode", F=512, layers=4, **long)),
        # the same at the higher-precision code width
        dict(name="decode_b1_128k_4bit", **_case("decode", F=512, bits=4, layers=4, **long)),
        # the same with the window W = floor(128 / 3), which no group size divides
        dict(name="decode_b1_128k_w42", **_case("decode", F=84, layers=4, **long)),
        # a full serving batch generating 128 tokens: every window fills once on the way
        dict(name="generate_b64_4k", **_case("decode", steps=128, **batch)),
        # the same batch with rows of different ages (continuous batching): per-row counts, windows fill row by row
        dict(name="generate_ragged_b64_4k", **_case("decode", steps=16, ragged=True, **batch)),
        # multi-head attention, head dimension 96, the largest cache
        dict(name="decode_mha_b16_32k", **_case("decode", 16, 32, 32, 96, 32768, "bf16", 64, 384, dist="laplace")),
        # prompts becoming caches: one long document, a full batch, a small batch of different lengths
        dict(name="prefill_b1_128k", **_case("prefill", F=512, **long)),
        dict(name="prefill_b64_4k", **_case("prefill", **batch)),
        dict(name="prefill_ragged_b8_8k", **_case("prefill", L=8192, ragged=True, **llama)),
    ]


MOST_VALUES = 16 * 32 * 32768 * 96     # of one cache's K (or V): the largest listed case


def draw(rng):
    kind = "prefill" if rng.random() < 0.25 else "decode"
    d = rng.choice([64, 96, 128, 128])
    Hkv, gh = rng.choice([(8, 4), (8, 4), (8, 1), (32, 1), (2, 8), (4, 2), (1, 4), (8, 8)])
    G = rng.choice([32, 32, 64, 64, 128])
    if rng.random() < 0.7:
        W = G * rng.randint(1, max(1, 256 // G))
    else:                               # a third of a budget, or odd: the last key group of an event is short
        W = rng.choice([42, 85, rng.randint(20, 250)])
    B = round(2 ** rng.uniform(0, 6))
    bits = rng.choice([2, 2, 2, 4])
    L = round(2 ** rng.uniform(8, 17)) + rng.randint(0, 31)
    most = MOST_VALUES // (16 if kind == "prefill" else 4)
    while B * Hkv * L * d * bits > 2 * most and L > 300:
        L = L * 2 // 3
    while B * Hkv * L * d * bits > 2 * most:
        B = (B + 1) // 2
    values = B * Hkv * L * d
    layers = 1 if kind == "prefill" else max(1, min(4, most // values))
    # at most W steps: a window fills once in a pass, so that a pass leaves the state it began with intact
    steps = 1 if kind == "prefill" or rng.random() < 0.6 else max(1, min(rng.randint(2, 32), W, most // (values * layers)))
    return _case(kind, B, Hkv * gh, Hkv, d, L, rng.choice(["f16", "bf16"]), G, 2 * W, bits, layers, steps,
                 ragged=B > 1 and rng.random() < 0.3, dist=rng.choice(["normal", "normal", "laplace"]), sinks=rng.choice([0, 4]))


# ---- sizes ---------------------------------------------------------------------------------
def _slots_per_event(c):
    W, G = c["F"] // 2, c["G"]
    return -(-W // G) * G


def _q_capacity(c):
    W, Wq = c["F"] // 2, _slots_per_event(c)
    q = ((c["L"] + c["steps"]) // W + 4) * Wq
    while q % 64:
        q += Wq
    return q


def _lengths(c):
    """Tokens of each row: with `ragged`, spread evenly between L/2 and L in a scattered order."""
    if not c["ragged"]:
        return [c["L"]] * c["B"]
    lo = c["L"] // 2
    return [c["L"] - int((c["L"] - lo) * (b * 0.6180339887 % 1.0)) for b in range(c["B"])]


def _after(L, W):
    """(filtering events, tokens at original precision) after L tokens."""
    e = 0 if L < 3 * W else (L - 3 * W) // W + 1
    return e, L - e * W


# ---- inputs --------------------------------------------------------------------------------
def _rows(c, L, gen, outliers, sinks):
    """[B][Hkv][L][d] rows of one tensor: normal or Laplace values, four channels per kv head ten times
    larger (`outliers`: [Hkv][4]), the first rows of a long context five times larger (attention sinks)."""
    dt = binding.torch_dtype(c["dtype"])
    x = torch.empty((c["B"], c["Hkv"], L, c["d"]), dtype=dt, device=DEVICE)
    for b in range(c["B"]):
        f = torch.empty(x.shape[1:], dtype=torch.float32, device=DEVICE)
        if c["dist"] == "laplace":
            f.exponential_(generator=gen)
            f.mul_(torch.randint(0, 2, f.shape, generator=gen, device=DEVICE, dtype=torch.int8).mul_(2).sub_(1))
        else:
            f.normal_(generator=gen)
        if outliers is not None:
            f.scatter_(2, outliers, f.gather(2, outliers) * 10)
        if sinks:
            f[:, :sinks] *= 5
        x[b] = f
    return x


def _prompt(c, gen):
    pick = random.Random(gen.initial_seed())
    idx = torch.tensor([pick.sample(range(c["d"]), 4) for _ in range(c["Hkv"])], device=DEVICE)
    idx = idx[:, None, :].expand(c["Hkv"], c["L"], 4)
    return (_rows(c, c["L"], gen, idx, c["sinks"]), _rows(c, c["L"], gen, None, c["sinks"]))


def _counts(cache, ragged):
    return (list(cache.cur), list(cache.n_fp), list(cache.n_q)) if ragged else cache.counts()


def _rewind(cache, counts, ragged):
    if ragged:
        cache.cur[:], cache.n_fp[:], cache.n_q[:] = counts
    else:
        cache.set_counts(counts)


def prepare(case, seed):
    c = case
    gen = torch.Generator(DEVICE)
    gen.manual_seed(seed)
    cfg = binding.make_config(c["B"], c["Hq"], c["Hkv"], c["d"], c["F"], c["G"], c["dtype"], _q_capacity(c), c["bits"])
    kind = binding.DeviceCacheSeq if c["ragged"] else binding.DeviceCache
    lengths = _lengths(c)
    caches = []
    for _ in range(c["layers"]):
        cache = kind(cfg, DEVICE)
        K, V = _prompt(c, gen)
        if c["kind"] == "decode":
            if c["ragged"]:
                cache.prefill_seq(K, V, lengths)
            else:
                cache.prefill(K, V)
        caches.append(cache)
    state = dict(case=c, caches=caches, counts=[_counts(x, c["ragged"]) for x in caches], W=c["F"] // 2)
    if c["kind"] == "prefill":
        state.update(K=K, V=V, lengths=lengths)
        return state
    dt = binding.torch_dtype(c["dtype"])
    new = lambda *shape: torch.randn((c["steps"], c["layers"]) + shape, generator=gen, device=DEVICE).to(dt)  # noqa: E731
    k, v = new(c["B"], c["Hkv"], 1, c["d"]), new(c["B"], c["Hkv"], 1, c["d"])
    q = new(c["B"], c["Hq"], c["d"])
    state["out"] = torch.empty_like(q)
    state["calls"] = [[(caches[i], k[s, i], v[s, i], q[s, i], state["out"][s, i]) for i in range(c["layers"])]
                      for s in range(c["steps"])]
    return state


# ---- one pass ------------------------------------------------------------------------------
def _decode(state):
    full = 3 * state["W"]
    for layer_calls in state["calls"]:
        for cache, k, v, q, out in layer_calls:
            if cache.c.n_fp + 1 < full:
                cache.decode_step(k, v, q, out)
            else:
                cache.append(k, v)
                cache.compress()
                cache.decode_attn(q, out)


def _decode_ragged(state):
    full = 3 * state["W"]
    for layer_calls in state["calls"]:
        for cache, k, v, q, out in layer_calls:
            if max(cache.n_fp) + 1 < full:
                cache.decode_step_seq(k, v, q, out)
            else:
                cache.append_seq(k, v)
                cache.compress_seq()
                cache.decode_attn_seq(q, out)


QUANTIZED = ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "pos_q")


def run(state):
    """One pass.  The counts go back to where `prepare` left them first, so a pass can be repeated: the rows it
    reads are not the ones it writes (appended rows go behind the live ones, a filtering event into the other
    buffer and behind the quantized slots)."""
    c, caches = state["case"], state["caches"]
    for cache, counts in zip(caches, state["counts"]):
        _rewind(cache, counts, c["ragged"])
    if c["kind"] == "prefill":
        cache = caches[0]
        if c["ragged"]:
            cache.prefill_seq(state["K"], state["V"], state["lengths"])
        else:
            cache.prefill(state["K"], state["V"])
        return [cache.k_fp[0], cache.v_fp[0], cache.pos_fp[0]] + [getattr(cache, n) for n in QUANTIZED]
    (_decode_ragged if c["ragged"] else _decode)(state)
    result = [state["out"]]
    for cache, counts in zip(caches, state["counts"]):
        result += cache.k_fp + cache.v_fp + cache.pos_fp
        if _counts(cache, c["ragged"])[2] != counts[2]:      # a window was filtered: the quantized region grew
            result += [getattr(cache, n) for n in QUANTIZED]
    return result


# ---- what a pass cannot do without -----------------------------------------------------------
def work(case):
    c = case
    d, G, W, bits, H = c["d"], c["G"], c["F"] // 2, c["bits"], c["Hkv"]
    ngc = -(-d // G)
    token_q = d * bits // 4 + 4 * ngc                     # codes of K and V, the value groups' scales and zeros
    event = W * token_q + -(-W // G) * 4 * d              # what one filtering event adds to the quantized region
    nbytes = flops = 0
    for L in _lengths(c):
        e, n = _after(L, W)
        if c["kind"] == "prefill":
            nbytes += H * (L * 4 * d + e * event + n * 4 * d)
            continue
        for _ in range(c["steps"]):
            n += 1
            nbytes += H * 2 * 4 * d                       # the new row: read, and stored into the cache
            if n == 3 * W:
                nbytes += H * (3 * W * 4 * d + event + 2 * W * 4 * d)
                e, n = e + 1, 2 * W
            nbytes += H * (e * event + n * 4 * d) + 2 * c["Hq"] * d * 2
            flops += 4 * c["Hq"] * d * (e * W + n)
    return {"bytes": nbytes * c["layers"], "flops": flops * c["layers"]}


def tolerance(case):
    """Prefill writes codes, scales and copied rows: exact.  An attention output is rounded once to the cache
    type from sums in fp32; against the same attention in fp64 the outputs were up to 1.8e-3 (2-norm) and 3.9e-3
    (largest difference) off for bf16, 3e-4 on average and 1.3e-3 for fp16: about four times that."""
    if case["kind"] == "prefill":
        return "exact"
    return {"rel": 6e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-3, "max": 5e-3}
