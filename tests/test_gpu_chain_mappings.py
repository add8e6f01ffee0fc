"""Every chain mapping against the one-lane kernels (a trace keeps a batch there,
and the oracle pins those), at batches for which the library's own rule is asked
that it takes the mapping: a threshold that moves fails a test here instead of
leaving it to compare a kernel with itself."""

import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1302_2669_amd as mc  # noqa: E402
import test_gpu_gated  # noqa: E402
from paper_1302_2669_amd import _lib, gate  # noqa: E402

DEV = "cuda"
ONE_LANE, SPLIT, LONE, BOTH = range(4)
LONE_L_MIN = 6


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")


def mapping(L, chains, sweeps, lone=True):
    """(mapping, one-lane waves per SIMD) of `chains` chains of `sweeps` sweeps."""
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    waves = ctypes.c_int32()
    kind = _lib._lib().mcmc_chain_mapping(L, ctypes.c_int64(chains), ctypes.c_int64(sweeps), simds,
                                          1, int(lone), ctypes.byref(waves))
    return kind, waves.value


def sweeps_for(kind, L, chains, least=1, most=200):
    """The fewest sweeps from which `chains` chains run under `kind`."""
    for sweeps in range(least, most):
        if mapping(L, chains, sweeps)[0] == kind:
            return sweeps
    pytest.fail(f"L = {L}: {chains} chains never run under mapping {kind}")


def check(kind, L, n, chains, K, noise):
    """Plain and resumed, all outputs and the chain state."""
    p, seed, total = (0.11 if noise else 0.16), 9, n * 4 * chains * K
    syn = mc.sample_errors(L, p, 5 + L, n, noise=noise)[0]
    args = dict(chains=chains, n_temps=K, noise=noise, want_sums=True, chain_state=True)
    need = sweeps_for(kind, L, total, least=2)

    def outputs(sweeps, burn, trace, resume):
        if resume:
            begin = burn + 1
            first = mc.decode_batch(syn, L, p, 1, seed, burn=burn, trace=trace, **args)
            out = mc.decode_batch(syn, L, p, sweeps, seed, burn=burn, trace=trace,
                                  resume_from=(first["chain_state"], begin), **args)
        else:
            begin = 0
            out = mc.decode_batch(syn, L, p, sweeps, seed, burn=burn, trace=trace, **args)
        assert mapping(L, total, burn + sweeps - begin)[0] == kind
        out.pop("trace", None)
        st, w = mc.unpack_chain_state(out.pop("chain_state"), n, L, p, sweeps, seed, chains, K,
                                      burn, noise=noise)
        torch.cuda.synchronize()
        return {**out, "states": st, "weights": w}

    for sweeps, burn, resume in ((need - 1, 1, False), (need + 1, 1, True)):
        want = outputs(sweeps, burn, True, resume)
        got = outputs(sweeps, burn, False, resume)
        for k in want:
            assert torch.equal(got[k], want[k]), (k, resume)


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("L", list(range(2, 26)))
def test_split(L, noise):
    check(SPLIT, L, 231, 7, 1, noise)       # 6468 chains, a ragged last tile
    if L < LONE_L_MIN:
        check(SPLIT, L, 3, 3, 1, noise)     # one wave


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("L", list(range(LONE_L_MIN, 26)))
def test_one_chain_per_wave(L, noise):
    check(LONE, L, 3, 3, 1, noise)
    check(LONE, L, 2, 5, 2, noise)


@pytest.mark.parametrize("L,noise,chains", [(2, 0, 71), (3, 1, 71), (4, 0, 105), (5, 1, 78),
                                            (6, 0, 201), (8, 1, 78), (9, 0, 105), (11, 1, 78),
                                            (13, 0, 71), (14, 1, 105), (16, 0, 80), (16, 1, 105),
                                            (17, 0, 71), (20, 1, 78), (23, 0, 80), (25, 1, 57)])
def test_one_lane_waves_and_a_split_rest(L, noise, chains):
    check(BOTH, L, 513, chains, 1, noise)


def test_each_mapping_of_a_gated_decode():
    # the full budget's chains one per lane, all split, whole waves with a split rest
    seen = set()
    for L, n, chains, full in ((9, 8192, 2, 1), (9, 8192, 2, 12), (5, 700, 3, 40), (5, 9001, 4, 60),
                               (13, 9001, 6, 10), (17, 2500, 11, 30)):
        syn = mc.sample_errors(L, 0.1, 3, n)[0]
        prm = torch.from_numpy(test_gpu_gated.spread_params(L, 17)).to(DEV)
        g = gate.GatedDecoder(L, 0.1, 21, max_batch=n, sweeps_short=1, sweeps_full=full,
                              chains=chains, threshold=1.0)
        out = g.decode(prm, syn, want_correction=True)
        torch.cuda.synchronize()
        sel = torch.nonzero(out["route"] == 2).flatten()
        assert len(sel) > n // 2
        seen.add(mapping(L, len(sel) * 4 * chains, full, lone=False)[0])
        want = mc.decode_batch(syn[sel], L, 0.1, full, 21, chains=chains, syndrome_ids=sel.cpu(),
                               trace=True)
        for k in ("chosen", "correction"):
            assert torch.equal(out[k][sel], want[k]), (L, n, k)
        g.close()
    assert seen == {ONE_LANE, SPLIT, BOTH}


# all groups split, some of them, none
@pytest.mark.parametrize("Ls,per,split", [((3, 5, 7, 9, 11, 13, 15), 80, True),
                                          ((9, 11, 13, 15), 900, True), ((7, 8), 30000, False)])
def test_groups_of_a_plan(Ls, per, split):
    syns = [mc.sample_errors(L, 0.1, 5, per)[0] for L in Ls]
    items = [dict(L=L, p=0.1, sweeps=L * L // 4, burn=0, chains=3, n_temps=1,
                  syndrome_id=i) for L in Ls for i in range(per)]
    plan = mc.MixedPlan(items, seed=9)
    groups = ctypes.c_int32()
    count = _lib._lib().mcmc_plan_split_groups(plan._h, ctypes.byref(groups))
    assert groups.value == len(Ls) and (count > 0) == split
    out = plan.execute(torch.cat([s.reshape(-1) for s in syns]), want_sums=True)
    torch.cuda.synchronize()
    for j, L in enumerate(Ls):
        u = mc.decode_batch(syns[j], L, 0.1, L * L // 4, 9, chains=3, want_sums=True,
                            init=mc.MCMC_INIT_MATCHING, trace=True)
        lo, hi = j * per, (j + 1) * per
        a, b = plan.chain_offsets[lo], plan.chain_offsets[hi]
        for k in ("sum_n", "accepts"):
            assert torch.equal(out[k][a:b], u[k].reshape(-1)), (L, k)
        assert torch.equal(out["chosen"][lo:hi], u["chosen"]), L
    plan.close()
