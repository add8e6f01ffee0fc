"""Kernel variants chosen by size, at the sizes where they can go wrong, through
the C-ABI: every integer output bit-exact with the oracle or with the mapping
already pinned to it."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1302_2669_amd as mc  # noqa: E402
from oracle import decoder, geometry, sampler  # noqa: E402
from oracle import spacetime as stm  # noqa: E402

from paper_1302_2669_amd.inputs import SEED_L9  # noqa: E402

DEV = "cuda"


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")


def to_np(d):
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in d.items()}


# random scan: 32-bit rows up to L = 15 (odd rows one field up), 64-bit above;
# 65 chains span two waves, the second almost empty
@pytest.mark.parametrize("noise,p", [(0, 0.17), (1, 0.11)])
@pytest.mark.parametrize("L,n,chains,K", [(2, 5, 13, 1), (4, 17, 1, 2), (14, 2, 3, 1),
                                          (15, 3, 2, 1), (16, 3, 2, 1), (24, 2, 1, 2)])
def test_random_scan_row_widths(L, n, chains, K, noise, p):
    lat = geometry.Lattice(L)
    syn, _, _ = sampler.sample(lat, p, SEED_L9 + L, np.arange(n), noise=noise)
    s = torch.from_numpy(syn).to(DEV)
    args = dict(chains=chains, n_temps=K, noise=noise, random_scan=True, want_sums=True)
    first = mc.decode_batch(s, L, p, 1, SEED_L9, chain_state=True, **args)
    out = mc.decode_batch(s, L, p, 2, SEED_L9, resume_from=(first["chain_state"], 1), **args)
    st, w = mc.unpack_chain_state(out.pop("chain_state"), n, L, p, 2, SEED_L9, chains, K,
                                  noise=noise)
    g = to_np(out)
    o = decoder.decode(L, syn, p, 2, SEED_L9, chains_per_class=chains, n_temps=K, noise=noise,
                       scan=decoder.SCAN_RANDOM)
    for k in ("sum_n", "accepts", "chosen", "correction"):
        assert np.array_equal(g[k], o[k]), k
    assert np.array_equal(st.cpu().numpy(), o["states"])
    assert np.array_equal(w.cpu().numpy(), o["n_final"].astype(np.int32))
    np.testing.assert_allclose(g["class_prob"], o["class_prob"], rtol=1e-12, atol=0)


@pytest.mark.parametrize("L,chains,K", [(4, 17, 1), (9, 33, 2), (3, 1, 4)])
def test_estimator_lane_sums(L, chains, K):
    # replica counts around the 16 lanes a class's sums are spread over
    p, n = 0.12, 5
    lat = geometry.Lattice(L)
    syn, _, _ = sampler.sample(lat, p, SEED_L9 + L, np.arange(n))
    g = to_np(mc.decode_batch(torch.from_numpy(syn).to(DEV), L, p, 2, SEED_L9, chains=chains,
                              n_temps=K, want_sums=True))
    o = decoder.decode(L, syn, p, 2, SEED_L9, chains_per_class=chains, n_temps=K)
    for k in ("sum_n", "accepts", "chosen", "correction"):
        assert np.array_equal(g[k], o[k]), k
    np.testing.assert_allclose(g["class_prob"], o["class_prob"], rtol=1e-12, atol=0)
    np.testing.assert_allclose(g["mean_n"], o["mean_n"], rtol=1e-12, atol=0)


def test_estimator_full_batches():
    # four lanes per class from 16384 syndromes on: every syndrome as in a small batch
    L, p, n = 3, 0.12, 16385
    syn, _, _ = mc.sample_errors(L, p, 11, n)
    big = to_np(mc.decode_batch(syn, L, p, 3, 11, chains=5, n_temps=2))
    for lo in (0, 12000, n - 1000):
        ids = torch.arange(lo, lo + 1000)
        small = to_np(mc.decode_batch(syn[lo:lo + 1000], L, p, 3, 11, chains=5, n_temps=2,
                                      syndrome_ids=ids))
        for k in small:
            assert np.array_equal(big[k][lo:lo + 1000], small[k]), k


# space-time chains, one lane per interval up to L = 12 and 16 rounds: the skew
# spans two words from round 8 on, lanes are left over where T does not divide
# 64, and 17 rounds fall back to one lane per chain
@pytest.mark.parametrize("L,T,n,chains", [(2, 16, 3, 3), (3, 9, 2, 4), (5, 8, 2, 2), (6, 7, 3, 1),
                                          (7, 7, 3, 2), (8, 16, 1, 1), (9, 13, 1, 1), (10, 5, 1, 2),
                                          (12, 16, 1, 1), (4, 17, 2, 1), (9, 1, 5, 3)])
def test_spacetime_lanes(L, T, n, chains):
    p, pm, sweeps = 0.06, 0.09, 3 if L < 8 else 2
    obs, _, _, _ = stm.sample(geometry.Lattice(L), p, pm, T, SEED_L9 + L, np.arange(n))
    g = to_np(mc.decode_spacetime(torch.from_numpy(obs).to(DEV), L, p, pm, sweeps, SEED_L9,
                                  chains=chains, burn=1, want_sums=True))
    o = stm.decode(L, obs, p, pm, sweeps, SEED_L9, chains_per_class=chains, burn=1)
    for k in ("sum_n", "sum_m", "accepts", "chosen", "correction"):
        assert np.array_equal(g[k], o[k]), k
    np.testing.assert_allclose(g["class_prob"], o["class_prob"], rtol=1e-12, atol=0)
