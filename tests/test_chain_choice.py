"""The choice of a uniform batch's chain mapping against measured times: us of whole
decodes on 256 CUs (1024 SIMDs) from canonical starts, p = 0.1, depolarizing noise,
under each mapping (one chain per lane, split, one per wave, the first two side by
side with the given one-lane waves per SIMD)."""

import ctypes

import pytest

from paper_1302_2669_amd import _lib

SIMDS = 1024
ONE_LANE, SPLIT, LONE, BOTH = range(4)
# L, chains, sweeps, us by (mapping, one-lane waves per SIMD)
MEASURED = [
    (3, 16384, 4, {(ONE_LANE, 0): 32, (SPLIT, 0): 44}),
    (3, 65536, 128, {(ONE_LANE, 0): 210, (SPLIT, 0): 293}),
    (3, 294912, 1, {(ONE_LANE, 0): 125, (BOTH, 3): 234, (BOTH, 4): 178}),
    (6, 49152, 4, {(ONE_LANE, 0): 58, (SPLIT, 0): 164}),
    (6, 49152, 8, {(ONE_LANE, 0): 75, (SPLIT, 0): 168}),
    (6, 65536, 1, {(ONE_LANE, 0): 51, (SPLIT, 0): 180}),
    (6, 98304, 2, {(ONE_LANE, 0): 66, (SPLIT, 0): 219, (BOTH, 1): 170}),
    (6, 159904, 2, {(ONE_LANE, 0): 91, (SPLIT, 0): 288, (BOTH, 1): 244, (BOTH, 2): 179}),
    (9, 6544, 128, {(ONE_LANE, 0): 1454, (SPLIT, 0): 193}),
    (9, 16384, 1, {(ONE_LANE, 0): 59, (SPLIT, 0): 123}),
    (9, 16384, 2, {(ONE_LANE, 0): 70, (SPLIT, 0): 123}),
    (9, 16384, 4, {(ONE_LANE, 0): 91, (SPLIT, 0): 122}),
    (9, 16384, 128, {(ONE_LANE, 0): 1420, (SPLIT, 0): 379}),
    (9, 49152, 1, {(ONE_LANE, 0): 70, (SPLIT, 0): 204}),
    (9, 49152, 4, {(ONE_LANE, 0): 101, (SPLIT, 0): 204}),
    (9, 65536, 1, {(ONE_LANE, 0): 77, (SPLIT, 0): 228}),
    (9, 65536, 8, {(ONE_LANE, 0): 149, (SPLIT, 0): 238}),
    (9, 98304, 2, {(ONE_LANE, 0): 99, (SPLIT, 0): 282, (BOTH, 1): 206}),
    (13, 1952, 128, {(ONE_LANE, 0): 2463, (SPLIT, 0): 285, (LONE, 0): 250}),
    (13, 16384, 1, {(ONE_LANE, 0): 105, (SPLIT, 0): 228}),
    (13, 16384, 2, {(ONE_LANE, 0): 123, (SPLIT, 0): 228}),
    (13, 49152, 4, {(ONE_LANE, 0): 170, (SPLIT, 0): 324}),
    (13, 49152, 8, {(ONE_LANE, 0): 243, (SPLIT, 0): 337}),
    (13, 294912, 2, {(ONE_LANE, 0): 261, (BOTH, 3): 604, (BOTH, 4): 436}),
    (17, 49152, 1, {(ONE_LANE, 0): 180, (SPLIT, 0): 432}),
    (17, 65536, 2, {(ONE_LANE, 0): 218, (SPLIT, 0): 503}),
    (17, 65536, 8, {(ONE_LANE, 0): 406, (SPLIT, 0): 554}),
    (25, 6544, 32, {(ONE_LANE, 0): 2754, (SPLIT, 0): 711}),
    (25, 65536, 4, {(ONE_LANE, 0): 641, (SPLIT, 0): 899}),
    (25, 98304, 2, {(ONE_LANE, 0): 551, (SPLIT, 0): 1082, (BOTH, 1): 738}),
]


def choice(L, chains, sweeps):
    waves = ctypes.c_int32()
    kind = _lib._lib().mcmc_chain_mapping(L, ctypes.c_int64(chains), ctypes.c_int64(sweeps), SIMDS,
                                          1, 1, ctypes.byref(waves))
    return kind, waves.value


@pytest.mark.parametrize("L,chains,sweeps,us", MEASURED,
                         ids=[f"L{m[0]}-{m[1]}x{m[2]}" for m in MEASURED])
def test_no_mapping_far_from_the_fastest_is_taken(L, chains, sweeps, us):
    # batches where the fastest wins by more than a tenth over one chain per lane, or
    # one chain per lane over every other
    assert us[choice(L, chains, sweeps)] <= 1.05 * min(us.values())


@pytest.mark.parametrize("L", [2, 9, 17, 25])
def test_without_a_sweep_the_chains_stay_on_lanes(L):
    for chains in (4, 1000, 100000, 10 ** 7):
        assert choice(L, chains, 0) == (ONE_LANE, 0)


@pytest.mark.parametrize("L,n,sweeps,splits", [(3, 1, 9, 0), (3, 2000, 9, 0), (5, 2000, 5, 0),
                                               (9, 2000, 1, 0), (3, 20000, 9, 0), (13, 1, 169, 1),
                                               (13, 20000, 169, 1), (5, 2000, 400, 1),
                                               (25, 100, 25, 1)])
def test_gated_batches_split_where_it_pays(L, n, sweeps, splits):
    assert _lib._lib().mcmc_gated_splits(L, ctypes.c_int64(n), ctypes.c_int64(16),
                                         ctypes.c_int64(sweeps), SIMDS) == splits
