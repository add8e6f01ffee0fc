"""Kernel variants chosen by size, at the sizes where they can go wrong, through
the C-ABI: every integer output bit-exact with the oracle or with the mapping
already pinned to it."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1302_2669_amd as mc  # noqa: E402
import test_gpu_gated  # noqa: E402
from oracle import decoder, geometry, sampler  # noqa: E402
from oracle import spacetime as stm  # noqa: E402

from paper_1302_2669_amd import gate  # noqa: E402
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


# The chain mappings of a uniform batch: a trace keeps every chain on one lane
# (pinned to the oracle elsewhere); without one the batch runs one chain per
# wave (few chains), split over lanes (up to about 1.7 waves per SIMD of 256
# CUs), or whole one-lane waves with a split rest.  All integers are equal.
def decode_pair(L, n, chains, K, noise, sweeps, burn=0, resume=False):
    p = 0.11 if noise else 0.16
    syn, _, _ = mc.sample_errors(L, p, 5 + L, n, noise=noise)
    args = dict(chains=chains, n_temps=K, burn=burn, noise=noise, want_sums=True)
    outs = []
    for trace in (False, True):
        if resume:
            first = mc.decode_batch(syn, L, p, 1, 9, chain_state=True, trace=trace, **args)
            out = mc.decode_batch(syn, L, p, sweeps, 9, trace=trace,
                                  resume_from=(first["chain_state"], burn + 1), **args)
        else:
            out = mc.decode_batch(syn, L, p, sweeps, 9, chain_state=True, trace=trace, **args)
        out.pop("trace", None)
        st, w = mc.unpack_chain_state(out.pop("chain_state"), n, L, p, sweeps, 9, chains, K, burn,
                                      noise=noise)
        outs.append({**to_np(out), "states": st.cpu().numpy(), "weights": w.cpu().numpy()})
    for k in outs[1]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("L", list(range(2, 26)))
def test_few_chains(L, noise):
    decode_pair(L, 3, 3, 1, noise, 3, burn=1)       # 36 chains: one per wave from L = 6
    decode_pair(L, 2, 5, 2, noise, 2, resume=True)


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("L", list(range(2, 26)))
def test_split_chains(L, noise):
    decode_pair(L, 231, 7, 1, noise, 2)             # 6468 chains, a ragged last tile


@pytest.mark.parametrize("L,noise,chains", [(2, 0, 65), (6, 1, 65), (9, 0, 100), (13, 0, 100),
                                            (13, 1, 65), (16, 0, 65), (17, 1, 65), (21, 0, 100),
                                            (25, 0, 80)])
def test_one_lane_waves_with_a_split_rest(L, noise, chains):
    decode_pair(L, 513, chains, 1, noise, 1)        # 2.0 to 3.1 one-lane waves per SIMD


# one-lane waves and a split rest side by side, long enough to be chosen: one to
# six waves per SIMD, the rest under and over one more wave's worth, ragged
@pytest.mark.parametrize("L,noise,chains,sweeps", [(2, 0, 83, 90), (5, 1, 78, 60), (9, 0, 105, 12),
                                                   (12, 0, 201, 8), (13, 1, 78, 8), (16, 0, 80, 6),
                                                   (17, 0, 71, 6), (25, 1, 57, 4), (25, 0, 78, 4)])
def test_both_mappings_side_by_side(L, noise, chains, sweeps):
    decode_pair(L, 513, chains, 1, noise, sweeps)
    decode_pair(L, 513, chains, 1, noise, sweeps + 1, burn=2, resume=True)


# plans whose longest groups are split and whose launches on the caller's stream
# follow each other: all groups split, a pair launch left, one-lane ranges left
@pytest.mark.parametrize("Ls,per", [((3, 5, 7, 9, 11, 13, 15), 80), ((5, 9, 13, 15, 17, 25), 120),
                                    ((8, 16, 17), 200), ((9, 11, 13, 15), 900)])
def test_plan_with_split_groups(Ls, per):
    syns = [mc.sample_errors(L, 0.1, 5, per)[0] for L in Ls]
    items = [dict(L=L, p=0.1, sweeps=L * L // 4, burn=0, chains=3, n_temps=1, syndrome_id=i)
             for L in Ls for i in range(per)]
    plan = mc.MixedPlan(items, seed=9)
    out = plan.execute(torch.cat([s.reshape(-1) for s in syns]), want_sums=True)
    g = to_np(out)
    for j, L in enumerate(Ls):
        u = to_np(mc.decode_batch(syns[j], L, 0.1, L * L // 4, 9, chains=3, want_sums=True,
                                  init=mc.MCMC_INIT_MATCHING))
        lo, hi = j * per, (j + 1) * per
        a, b = plan.chain_offsets[lo], plan.chain_offsets[hi]
        for k in ("sum_n", "accepts"):
            assert np.array_equal(g[k][a:b], u[k].reshape(-1)), (L, k)
        assert np.array_equal(g["chosen"][lo:hi], u["chosen"]), L
    plan.close()


# the gate's device-built plan: its full-budget chains all split, in whole waves
# with a split rest (ragged on both sides), and one chain per lane
@pytest.mark.parametrize("L,n,chains,full,threshold", [(5, 700, 3, 40, 0.5), (5, 9001, 4, 60, 1.0),
                                                       (13, 9001, 6, 10, 0.5), (17, 2500, 11, 5, 1.0),
                                                       (9, 8192, 2, 7, 1.0)])
def test_gated_mappings(L, n, chains, full, threshold):
    syn = mc.sample_errors(L, 0.1, 3, n)[0]
    prm = torch.from_numpy(test_gpu_gated.spread_params(L, 17)).to(DEV)
    g = gate.GatedDecoder(L, 0.1, 21, max_batch=n, sweeps_short=2, sweeps_full=full, chains=chains,
                          threshold=threshold)
    out = g.decode(prm, syn, want_correction=True)
    test_gpu_gated.check_routes(L, syn, np.full(n, 0.1), np.arange(n, dtype=np.int64), out, chains,
                                2, full, 21)
    g.close()


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


# space-time chains, one lane per interval up to L = 15 and 16 rounds: the skew
# spans two words from round 8 on, lanes are left over where T does not divide
# 64, and 17 rounds fall back to one lane per chain
@pytest.mark.parametrize("L,T,n,chains", [(2, 16, 3, 3), (3, 9, 2, 4), (5, 8, 2, 2), (6, 7, 3, 1),
                                          (7, 7, 3, 2), (8, 16, 1, 1), (9, 13, 1, 1), (10, 5, 1, 2),
                                          (12, 16, 1, 1), (4, 17, 2, 1), (9, 1, 5, 3),
                                          (13, 16, 1, 1), (14, 9, 2, 1), (15, 2, 3, 2),
                                          (15, 16, 1, 1), (16, 3, 1, 1)])
def test_spacetime_lanes(L, T, n, chains):
    p, pm, sweeps = 0.06, 0.09, 3 if L < 8 else 2
    obs, _, _, _ = stm.sample(geometry.Lattice(L), p, pm, T, SEED_L9 + L, np.arange(n))
    g = to_np(mc.decode_spacetime(torch.from_numpy(obs).to(DEV), L, p, pm, sweeps, SEED_L9,
                                  chains=chains, burn=1, want_sums=True))
    o = stm.decode(L, obs, p, pm, sweeps, SEED_L9, chains_per_class=chains, burn=1)
    for k in ("sum_n", "sum_m", "accepts", "chosen", "correction"):
        assert np.array_equal(g[k], o[k]), k
    np.testing.assert_allclose(g["class_prob"], o["class_prob"], rtol=1e-12, atol=0)


def test_matching_tiers_of_large_batches():
    # from 3072 syndromes the larger codes use capacities between the tiers: the
    # same starts as in small batches, syndromes on both sides of each capacity
    for L in (20, 25):
        n = 3072
        syn = torch.cat([mc.sample_errors(L, p, 7, n // 6, id_base=int(1000 * p))[0]
                         for p in (0.03, 0.05, 0.07, 0.10, 0.13, 0.18)])
        reps = mc.init_representatives(syn, L, mc.MCMC_INIT_MWPM)
        for lo in range(0, n, 512):
            small = mc.init_representatives(syn[lo:lo + 512], L, mc.MCMC_INIT_MWPM)
            torch.cuda.synchronize()
            assert torch.equal(reps[lo:lo + 512], small), (L, lo)


@pytest.mark.parametrize("L", [2, 5, 9, 13, 17, 21, 25])
def test_matching_problems_alone(L):
    # up to 512 syndromes (as many as the chip's LDS holds at once) every problem
    # has its own wave: the same starts as in a larger batch, lit from none to all
    n = 513
    syn = torch.cat([mc.sample_errors(L, p, 8, 128)[0] for p in (0.02, 0.08, 0.16, 0.4)])
    syn = torch.cat([syn, torch.ones_like(syn[:1])])
    syn[0] = 0
    reps = mc.init_representatives(syn, L, mc.MCMC_INIT_MWPM)
    for lo, hi in ((0, 1), (0, 256), (256, 512), (512, 513), (1, 513)):
        small = mc.init_representatives(syn[lo:hi].contiguous(), L, mc.MCMC_INIT_MWPM)
        torch.cuda.synchronize()
        assert torch.equal(reps[lo:hi], small), (lo, hi)
    assert n == len(syn)


# random scan in workgroups of four waves, and of one where those hold more
# waves (full batches from L = 19 on): one sweep against a small batch's
@pytest.mark.parametrize("L,n,chains,noise", [(13, 65, 4, 1), (18, 65, 4, 0), (19, 1200, 55, 0),
                                              (22, 1100, 60, 1)])
def test_random_scan_workgroups(L, n, chains, noise):
    syn, _, _ = mc.sample_errors(L, 0.08, 13, n, noise=noise)
    args = dict(chains=chains, noise=noise, random_scan=True, want_sums=True)
    big = to_np(mc.decode_batch(syn, L, 0.08, 1, 13, **args))
    lo = n - 20
    small = to_np(mc.decode_batch(syn[lo:].contiguous(), L, 0.08, 1, 13,
                                  syndrome_ids=torch.arange(lo, n), **args))
    for k in small:
        assert np.array_equal(big[k][lo:], small[k]), k
