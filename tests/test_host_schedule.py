"""The static schedule of the attention kernel, restated on the host: every 64-slot tile and every unit of 32 fp rows
of a head group is taken by exactly one wavefront, whatever the counts, splits and workgroup shape."""
import random

import pytest


def first_tile(s, TQ, TF, NS, R64):
    per, rem = divmod(64 * TQ + R64 * TF, NS)
    units_before = TF // NS * s + min(s, TF % NS)
    return max(0, per * s + rem * s // NS - R64 * units_before) >> 6


def tiles_of(split, wave, TQ, TF, NS, NWB, R64):
    lo, hi = (first_tile(split, TQ, TF, NS, R64), first_tile(split + 1, TQ, TF, NS, R64)) if NS > 1 else (0, TQ)
    assert 0 <= lo <= hi <= TQ
    units = (TF - 1 - split) // NS + 1 if split < TF else 0
    nh = units % NWB
    nl = NWB - nh
    lead = nh > 0 and wave >= nh
    t = lo + (wave if nh == 0 else wave - nh if wave >= nh else 2 * nl + wave)
    while t < hi:
        yield t
        t += nl if lead else NWB
        lead = False


@pytest.mark.parametrize("NWB", [4, 8, 12])
def test_every_tile_and_unit_is_taken_once(NWB):
    rng = random.Random(NWB)
    for _ in range(1500):
        TQ = rng.choice([0, 1, 2, 3, 63, 64, 65, rng.randint(0, 400)])
        TF = rng.choice([0, 1, NWB - 1, NWB, NWB + 1, rng.randint(0, 24)])
        NS = rng.choice([1, 1, 2, 3, 4, 5, 32, rng.randint(1, 256)])
        R64 = rng.choice([60, 133, 171, 205, 240])      # bytes of a unit in 1/64 tiles, over head dimensions and group sizes
        tiles, units = [], []
        for split in range(NS):
            for wave in range(NWB):
                tiles += tiles_of(split, wave, TQ, TF, NS, NWB, R64)
                units += range(wave * NS + split, TF, NS * NWB)
        assert sorted(tiles) == list(range(TQ)) and sorted(units) == list(range(TF)), (TQ, TF, NS)
