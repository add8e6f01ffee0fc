"""Full batches of space-time histories, where one lane per chain is taken, against
the same histories in small batches, where every interval has its lane."""

import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1302_2669_amd as mc  # noqa: E402
from paper_1302_2669_amd import _lib  # noqa: E402


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")


def lanes(L, T, chains, sweeps):
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    return _lib._lib().mcmc_spacetime_mapping(L, T, ctypes.c_int64(chains), ctypes.c_int64(sweeps),
                                              simds)


@pytest.mark.parametrize("L,T,chains,sweeps", [(2, 2, 8, 20), (2, 16, 4, 6), (3, 9, 8, 6),
                                               (4, 16, 9, 4)])
def test_full_batches(L, T, chains, sweeps):
    n, part = 33001, 500
    obs = mc.sample_spacetime(L, T, 0.05, 0.08, 21, n, device="cuda")[0]
    args = dict(chains=chains, burn=1, want_sums=True)
    assert lanes(L, T, n * 4 * chains, sweeps + 1) == 0
    assert lanes(L, T, part * 4 * chains, sweeps + 1) == 1
    full = mc.decode_spacetime(obs, L, 0.05, 0.08, sweeps, 21, **args)
    for lo in (0, 16000, n - part):
        ids = torch.arange(lo, lo + part)
        few = mc.decode_spacetime(obs[lo:lo + part], L, 0.05, 0.08, sweeps, 21, syndrome_ids=ids,
                                  **args)
        torch.cuda.synchronize()
        for k in few:
            assert torch.equal(full[k][lo:lo + part], few[k]), (lo, k)
