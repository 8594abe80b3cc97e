"""Codes at and next to their thresholds z + (k + 1/2) s: values on integer grids (ties, zeros of both signs, thresholds
that are zero), subnormal, huge, of widely mixed exponents, and within a unit in the last place of a threshold.  Prompt
and filtering step against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle.cache import SliceCache
from oracle.quantizer import round_to_T
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def values(rng, n, dt, bits):
    """[n] values of T for one channel."""
    steps, tiny = (1 << bits) - 1, 2.0 ** (-24 if dt == "f16" else -30)
    kind = rng.integers(7)
    if kind == 0:
        x = rng.integers(-steps, steps + 1, n) * rng.choice([0.25, 1.0, 3.0, 7.0])
    elif kind == 1:                      # symmetric: the middle threshold is zero
        x = rng.choice([-1.0, -0.0, 0.0, 1.0], n) * rng.choice([1.0, 5.0, 2.0 ** -10])
    elif kind == 2:
        x = rng.integers(-40, 41, n) * tiny
    elif kind == 3:
        x = rng.choice([-65504.0, 65504.0, 60000.0, -3.0, 0.0], n) if dt == "f16" else rng.standard_normal(n) * 3e4
    elif kind == 4:
        x = rng.standard_normal(n) * 2.0 ** rng.integers(-14, 5, n)
    elif kind == 5:                      # flat, or all but one value equal
        x = np.full(n, rng.standard_normal())
        x[rng.integers(n)] += rng.choice([0.0, 2.0 ** -9, 1.0])
    else:                                # around the thresholds of the group [z, z + steps * s]
        z, s = rng.standard_normal() * 4, 2.0 ** rng.integers(-9, 3) * (1 + rng.random())
        x = z + (rng.integers(0, steps, n) + 0.5) * s * (1 + rng.integers(-2, 3, n) * 2.0 ** (-11 if dt == "f16" else -8))
        x[:2] = z, z + steps * s
    top = 65504 if dt == "f16" else 65280     # values of T within fp16's range
    return np.clip(round_to_T(x.astype(np.float32), dt), -top, top)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("d,G,W", [(128, 32, 32), (128, 128, 128), (96, 64, 42), (64, 64, 64), (96, 32, 64)])
def test_codes_at_thresholds(dt, bits, d, G, W):
    wl = U.make_wl(B=1, Hq=1, Hkv=1, d=d, G=G, F=2 * W, dtype=dt, bits=bits)
    rng = np.random.default_rng([d, G, W, bits, dt == "f16"])
    L = 3 * W + 4 * W
    # keys: a group is a channel's run of tokens; values: a token's run of channels
    K = np.stack([values(rng, L, dt, bits) for _ in range(d)], axis=1)
    V = np.stack([np.concatenate([values(rng, min(G, d - c), dt, bits) for c in range(0, d, G)]) for _ in range(L)])
    oc = SliceCache(W, G, d, dt, bits)
    oc.append_block(K, V)
    Kd, Vd = U.to_dev(K[None, None], dt), U.to_dev(V[None, None], dt)
    for bulk in (True, False):
        dc = U.new_cache(wl, L)
        if bulk:
            dc.prefill(Kd, Vd)
        else:
            dc.stream_in(Kd, Vd)
        U.check_state(dc, oc, wl, 0, 0)
    assert len({int(c) for c in np.unique(oc.K_codes)}) == 1 << bits and len({int(c) for c in np.unique(oc.V_codes)}) == 1 << bits


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("exponent", [-125, -112, -101, -99])
def test_codes_of_tiny_bf16_values(bits, exponent):
    """Scales on both sides of what the fp32 reciprocal covers."""
    wl = U.make_wl(B=1, Hq=1, Hkv=1, d=64, G=32, F=64, dtype="bf16", bits=bits)
    rng = np.random.default_rng([bits, -exponent])
    K, V = (np.ldexp(rng.integers(-100, 101, (32 * 6, 64)), exponent - 3).astype(np.float32) for _ in range(2))
    oc = SliceCache(32, 32, 64, "bf16", bits)
    oc.append_block(K, V)
    dc = U.new_cache(wl, len(K))
    dc.prefill(U.to_dev(K[None, None], "bf16"), U.to_dev(V[None, None], "bf16"))
    U.check_state(dc, oc, wl, 0, 0)
    assert len(np.unique(oc.K_codes)) == 1 << bits
