"""The static schedule of the attention kernel, restated on the host: with a single split every 64-slot tile of
a head group is taken by exactly one wavefront, whatever the counts and the workgroup shape."""
import random

import pytest


def tiles_of(wave, TQ, TF, NWB):
    nh = TF % NWB
    nl = NWB - nh
    lead = nh > 0 and wave >= nh
    t = wave if nh == 0 else wave - nh if wave >= nh else 2 * nl + wave
    while t < TQ:
        yield t
        t += nl if lead else NWB
        lead = False


@pytest.mark.parametrize("NWB", [4, 8, 12])
def test_every_tile_is_taken_once_with_a_single_split(NWB):
    rng = random.Random(NWB)
    for _ in range(1500):
        TQ = rng.choice([0, 1, 2, 3, 63, 64, 65, rng.randint(0, 400)])
        TF = rng.choice([0, 1, NWB - 1, NWB, NWB + 1, rng.randint(0, 24)])
        tiles = [t for wave in range(NWB) for t in tiles_of(wave, TQ, TF, NWB)]
        assert sorted(tiles) == list(range(TQ)), (TQ, TF)
