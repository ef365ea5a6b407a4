"""Each wide kernel of the reduce - five and four units to four threads, ranked and sparse tiles - with
tiles that registers hold, that have more entries than that, and that go by windows, with and
without the dense copy.  Sums of dyadic values: exact in any order."""
import numpy as np
import pytest

from test_gpu_reduce_slim import regions_of, tile
from test_gpu_reduce_tiles import run_batch

pytestmark = pytest.mark.gpu
B, WIDTH = 48, 1_000_001
# tiles, P, capacity, distinct, again: the hits in the first tile of the regions at both ends
CASES = [(kernel, P, capacity, distinct, again)
         for kernel, P, capacity, room in [("wide5 ranked", 40, 150_000, 7_968), ("wide5 sparse", 40, 80_000, 7_168),
                                           ("wide4 ranked", 100, 150_000, 8_064), ("wide4 sparse", 100, 80_000, 7_168),
                                           ("wide4 sparse", 200, 20_000, 7_168)]
         for distinct, again in [(6_000, 300), (room, 0), (room + 1, 0), (5_000, 6_500), (3_000, 14_000), (16_000, 2_000),
                                 (40_000, 100)]]


@pytest.mark.parametrize("kernel,P,capacity,distinct,again", CASES)
def test_wide_tiles(kernel, P, capacity, distinct, again):
    rng = np.random.default_rng(P + capacity + distinct)
    regions = regions_of(lambda lo: tile(rng, lo, 44_000, P, distinct, again), B, P, WIDTH)
    run_batch(regions, P, WIDTH, capacity, lead=P % 4, dense=distinct % 7 == 0)


# all slots of a tile of 98,304 hit: more than 16 bits count
FULL = (12, 200, 5_000_001, 120_000)


@pytest.mark.parametrize("dense", [False, True])
def test_a_wide_tile_all_of_whose_slots_are_hit(dense):
    b, P, width, capacity = FULL
    rng = np.random.default_rng(3)
    run_batch(regions_of(lambda lo: tile(rng, lo, 98_304, P, 98_304, 500), b, P, width), P, width, capacity, lead=1, dense=dense)
