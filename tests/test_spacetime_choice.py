"""The choice between the space-time kernels, against measured times: us of both on
256 CUs (1024 SIMDs), p = 0.03 on data and outcomes."""

import ctypes

import pytest

from paper_1302_2669_amd import _lib

SIMDS = 1024
# L, rounds, histories, chains, sweeps, us one lane per chain, us one lane per interval
MEASURED = [
    (2, 2, 65536, 4, 238, 4237, 5814), (2, 8, 16384, 4, 238, 7407, 14454),
    (2, 16, 4096, 4, 476, 16470, 25992), (2, 16, 65536, 4, 29, 6183, 24806),
    (3, 8, 65536, 4, 19, 5148, 6851), (3, 12, 16384, 4, 52, 6566, 9489),
    (3, 16, 65536, 4, 9, 5168, 9891), (4, 12, 65536, 4, 6, 5053, 6675),
    (4, 16, 65536, 4, 4, 4598, 6514),
    (2, 16, 1024, 4, 1907, 64735, 28952), (3, 4, 4096, 4, 635, 12204, 6060),
    (3, 16, 4096, 4, 158, 13916, 10825), (3, 16, 1024, 4, 635, 55179, 12427),
    (4, 8, 16384, 4, 39, 6282, 5617), (5, 4, 65536, 4, 11, 4644, 4239),
    (5, 8, 4096, 4, 95, 16512, 5374), (7, 7, 2048, 4, 784, 204378, 43626),
    (7, 8, 65536, 4, 2, 4234, 3880), (9, 16, 16384, 4, 3, 6792, 4647),
    (12, 12, 4096, 4, 9, 17554, 4917),
]


@pytest.mark.parametrize("L,T,n,chains,sweeps,chain_us,lanes_us", MEASURED)
def test_the_faster_kernel_is_taken(L, T, n, chains, sweeps, chain_us, lanes_us):
    lanes = _lib._lib().mcmc_spacetime_mapping(L, T, ctypes.c_int64(n * 4 * chains),
                                               ctypes.c_int64(sweeps), SIMDS)
    assert lanes == int(lanes_us < chain_us)


def test_kernels_ranges():
    mapping = _lib._lib().mcmc_spacetime_mapping
    big = ctypes.c_int64(1 << 22)
    assert mapping(13, 16, big, ctypes.c_int64(100), SIMDS) == 1   # else through memory
    assert mapping(16, 3, big, ctypes.c_int64(100), SIMDS) == 0
    assert mapping(5, 17, ctypes.c_int64(16), ctypes.c_int64(100), SIMDS) == 0
