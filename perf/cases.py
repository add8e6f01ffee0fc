"""Performance cases of the decoder: the calls its users make, from one
syndrome at a time to full batches, each through a public entry point.

A case is a plain dict.  `kind` names the entry point and the other keys its
arguments:

  decode       decode_batch: colour-phased chains, either noise model, one or
               many temperatures, optionally with the chain state kept for a
               later resume; `sweeps` 0 is the enhanced-matching decoder alone
  random_scan  decode_batch with the paper's one-random-stabilizer step
  mixed        MixedPlan.execute over codes and rates of many sizes
  spacetime    decode_spacetime over measurement histories
  gate_train   one optimizer step of the gate network
  gated        GatedDecoder.decode: network, gap route, sweep budgets

The chains' outputs are sums of keyed random draws, so they have no closed
64-bit form; the network's logits, gradients and updated weights do (exact).
"""

import numpy as np
import torch

import paper_1302_2669_amd as mc
from paper_1302_2669_amd import gate, inputs

OPS_PER_UPDATE = 40                    # integer operations of one Metropolis update
MAX_UPDATES = 65536 * 843648           # of a drawn batch: the metric launch
NETWORK_FLOPS_PER_PIXEL = 2 * 32 * (9 * 3 + 2 * 9 * 32 + 7)
# thresholds of the start-weight gap route fitted at L = 13 (rate bins 0.05 to 0.17)
GAP_BINS = [0, 0, 0, 2, 3, 3, 4, 5, 5, 5, 6, 6, 8]

INIT = {"mwpm": mc.MCMC_INIT_MWPM, "greedy": mc.MCMC_INIT_MATCHING}
NOISE = {"depolarizing": mc.MCMC_NOISE_DEPOLARIZING, "flips": mc.MCMC_NOISE_BITPHASE}


def _decode(name, L, n, p, sweeps, chains=4, temps=1, burn=0, init="mwpm", noise="depolarizing",
            state=False, kind="decode"):
    return dict(name=name, kind=kind, L=L, n=n, p=p, sweeps=sweeps, chains=chains, temps=temps,
                burn=burn, init=init, noise=noise, state=state)


def listed():
    return [
        # a live decoder: one syndrome arrives, its class is wanted at once
        _decode("one_L13", 13, 1, 0.15, 169),
        # a quick study of a small code: few lanes, long chains, greedy starts
        _decode("small_L3", 3, 1000, 0.10, 2000, chains=1, init="greedy"),
        # an ordinary batch of a medium code
        _decode("batch_L9", 9, 10000, 0.10, 81),
        # the benchmark's own launch: a full batch at L = 13, p = 0.15
        _decode("batch_L13", 13, 65536, 0.15, 169),
        # bit/phase flips with a burn-in, a ragged batch that leaves part of the chip idle
        _decode("flips_L13", 13, 4001, 0.10, 149, burn=20, noise="flips"),
        # near threshold at the largest code, eight chains per class, first checkpoint kept
        _decode("checkpoint_L25", 25, 5000, 0.16, 625, chains=8, state=True),
        # the enhanced-matching decoder alone (no sweep) at the largest code
        _decode("matching_L25", 25, 4096, 0.10, 0, chains=1),
        # a serving batch of mixed code sizes and rates
        dict(name="mixed_L5_25", kind="mixed", n=4096, chains=4),
        # repeated imperfect measurements, the benchmark's code and chain length
        dict(name="spacetime_L7", kind="spacetime", L=7, rounds=7, n=2048, p=0.02, p_m=0.02,
             sweeps=784, chains=4),
        # cross-check of a batch with the paper's own random scan
        _decode("random_scan_L13", 13, 4096, 0.15, 169, init="greedy", kind="random_scan"),
        # one step of the gate network's training
        dict(name="gate_train_L13", kind="gate_train", L=13, n=512),
        # the gated decoder over rates as they come
        dict(name="gated_L13", kind="gated", L=13, n=20000, chains=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_decode(rng):
    L = rng.randint(3, 25)
    noise = "flips" if rng.random() < 0.25 else "depolarizing"
    c = _decode("", L, 1, round(rng.uniform(0.05, 0.11 if noise == "flips" else 0.18), 4),
                max(1, round(L * L * rng.choice((0.25, 0.5, 1.0)))),
                chains=rng.choice((1, 2, 4, 8)), temps=20 if rng.random() < 0.2 else 1,
                burn=rng.choice((0, 0, L)), init="greedy" if rng.random() < 0.25 else "mwpm",
                noise=noise, state=rng.random() < 0.15)
    most = MAX_UPDATES // _updates(c)
    c["n"] = min(_log_int(rng, 1, 65536), most)
    return c


def _draw_matching(rng):
    L = rng.randint(5, 25)
    return _decode("", L, _log_int(rng, 1, min(65536, 2 * 10 ** 9 // L ** 4)),
                   round(rng.uniform(0.05, 0.16), 4), 0, chains=1)


def _draw_random_scan(rng):
    L = rng.randint(3, 17)
    c = _decode("", L, 1, round(rng.uniform(0.08, 0.16), 4), max(1, L * L // rng.choice((1, 2))),
                chains=rng.choice((1, 2, 4)), init="greedy", kind="random_scan")
    c["n"] = min(_log_int(rng, 1, 16384), 10 ** 10 // _updates(c))
    return c


def _draw_spacetime(rng):
    L = rng.randint(3, 15)
    rounds = rng.randint(2, L)
    p = round(rng.uniform(0.01, 0.03), 4)
    c = dict(kind="spacetime", L=L, rounds=rounds, n=1, p=p, p_m=p,
             sweeps=L * L * rng.choice((1, 4)), chains=rng.choice((1, 2, 4)))
    c["n"] = min(_log_int(rng, 1, 8192), 8 * 10 ** 10 // _updates(c))
    return c


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "decode", "matching", "mixed", "spacetime",
                       "random_scan", "gate_train", "gated"))
    if kind == "decode":
        c = _draw_decode(rng)
    elif kind == "matching":
        c = _draw_matching(rng)
    elif kind == "mixed":
        c = dict(kind="mixed", n=_log_int(rng, 64, 8192), chains=rng.choice((2, 4)))
    elif kind == "spacetime":
        c = _draw_spacetime(rng)
    elif kind == "random_scan":
        c = _draw_random_scan(rng)
    elif kind == "gate_train":
        c = dict(kind="gate_train", L=rng.randint(5, 13), n=_log_int(rng, 64, 1024))
    else:
        c = dict(kind="gated", L=rng.randint(7, 13), n=_log_int(rng, 500, 50000),
                 chains=rng.choice((2, 4)))
    c.pop("name", None)
    return c


def _mixed_codes(case):
    """(L, sweeps) per item of a mixed batch: the same codes for every seed."""
    L, _, sweeps = inputs.mixed_workload(case["n"], case["n"])
    return L, sweeps


def _state_pieces(case, buffer):
    """Rows and weights of a chain-state buffer (its pieces lie 256 bytes aligned)."""
    L, chains = case["L"], case["n"] * 4 * case["temps"] * case["chains"]
    rows = (2 * L - 1) * ((L + 15) // 16) * chains * 4
    at = (rows + 255) // 256 * 256
    return buffer[:rows].view(torch.int32), buffer[at:at + 4 * chains].view(torch.int32)


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    key = 0x1302266900000000 + seed
    dev = torch.device("cuda")
    if kind in ("decode", "random_scan"):
        syn, _, _ = mc.sample_errors(case["L"], case["p"], key, n, noise=NOISE[case["noise"]])
        return dict(case=case, key=key, syn=syn)
    if kind == "mixed":
        L, sweeps = _mixed_codes(case)
        p = inputs.uniform_rates(n, seed).astype(np.float64)
        plan = mc.MixedPlan.from_arrays(L, p, sweeps, key, chains=case["chains"],
                                        init=mc.MCMC_INIT_MWPM)
        syn, _ = plan.sample(key)
        return dict(case=case, plan=plan, syn=syn)
    if kind == "spacetime":
        obs, _ = mc.sample_spacetime(case["L"], case["rounds"], case["p"], case["p_m"], key, n)
        return dict(case=case, key=key, obs=obs)
    L = case["L"]
    rates = inputs.uniform_rates(n, seed)
    syn, _, ids = gate.sample_dataset(L, rates.astype(np.float64), key)
    params = torch.from_numpy(inputs.cnn_init(L, seed)).to(dev)
    if kind == "gate_train":
        target, budget = inputs.cnn_targets(n, seed)
        return dict(case=case, net=gate.GateNet(L, params), syn=syn,
                    p=torch.from_numpy(rates).to(dev), target=torch.from_numpy(target).to(dev),
                    budget=torch.from_numpy(budget).to(dev))
    table = np.full(gate.GAP_BINS, gate.GAP_NEVER, dtype=np.uint8)
    table[5:5 + len(GAP_BINS)] = GAP_BINS
    decoder = gate.GatedDecoder(L, 0.15, key, n, chains=case["chains"], init=mc.MCMC_INIT_MWPM,
                                gap_table=table)
    return dict(case=case, decoder=decoder, params=params, syn=syn,
                p=rates.astype(np.float64), ids=ids)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("decode", "random_scan"):
        out = mc.decode_batch(state["syn"], case["L"], case["p"], case["sweeps"], state["key"],
                              chains=case["chains"], n_temps=case["temps"], burn=case["burn"],
                              init=INIT[case["init"]], noise=NOISE[case["noise"]],
                              want_sums=case["state"], chain_state=case["state"] or None,
                              random_scan=kind == "random_scan")
        if case["state"]:
            out["state_rows"], out["state_n"] = _state_pieces(case, out.pop("chain_state"))
        return out
    if kind == "mixed":
        return state["plan"].execute(state["syn"])
    if kind == "spacetime":
        return mc.decode_spacetime(state["obs"], case["L"], case["p"], case["p_m"],
                                   case["sweeps"], state["key"], chains=case["chains"])
    if kind == "gate_train":
        net = state["net"]
        logits, ws = net.forward(state["syn"], state["p"])
        grads, loss = gate.backward(net.L, net.params, logits, state["target"], state["budget"],
                                    ws)
        net.step_count += 1
        gate.adam_step(net.params, grads, net.m, net.v, net.step_count)
        return dict(logits=logits, grads=grads, loss=loss, params=net.params, m=net.m, v=net.v)
    return state["decoder"].decode(state["params"], state["syn"], p=state["p"], ids=state["ids"],
                                   want_correction=True)


def _updates(case):
    """Metropolis moves per syndrome (history) of a case of one code size."""
    L = case["L"]
    if case["kind"] == "spacetime":
        T = case["rounds"]
        moves = T * 2 * L * (L - 1) + 2 * (T - 1) * (2 * L * L - 2 * L + 1)
        return 4 * case["chains"] * case["sweeps"] * moves
    return max(1, 4 * case["chains"] * case["temps"] * (case["burn"] + case["sweeps"])
               * 2 * L * (L - 1))


def _decode_bytes(L, n):
    """Syndromes in; class probabilities, means, decision and correction out."""
    return n * (2 * L * (L - 1) + 64 + 1 + 2 * L * L - 2 * L + 1)


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("decode", "random_scan"):
        L = case["L"]
        nbytes = _decode_bytes(L, n)
        if case["state"]:
            chains = n * 4 * case["chains"] * case["temps"]
            nbytes += chains * ((2 * L - 1) * ((L + 15) // 16) * 4 + 4 + 2 * 16)
        counted = case["burn"] + case["sweeps"] > 0
        return {"bytes": nbytes, "flops": n * _updates(case) * OPS_PER_UPDATE if counted else 0}
    if kind == "mixed":
        L, sweeps = _mixed_codes(case)
        L, sweeps = L.astype(np.int64), sweeps.astype(np.int64)
        updates = int((4 * case["chains"] * sweeps * 2 * L * (L - 1)).sum())
        return {"bytes": int(sum(_decode_bytes(int(v), 1) for v in L)),
                "flops": updates * OPS_PER_UPDATE}
    L = case["L"]
    if kind == "spacetime":
        return {"bytes": _decode_bytes(L, n) + n * (case["rounds"] - 1) * 2 * L * (L - 1) + 32 * n,
                "flops": n * _updates(case) * OPS_PER_UPDATE}
    weights = gate.param_count(L) * 4
    network = n * L * L * NETWORK_FLOPS_PER_PIXEL
    if kind == "gate_train":
        return {"bytes": n * (2 * L * (L - 1) + 4 + 16 + 4 + 32 + 4) + 7 * weights,
                "flops": 3 * network}
    # the gap route answers about half of these rates without a sweep
    updates = n * 4 * case["chains"] * L * L * 2 * L * (L - 1) // 2
    return {"bytes": _decode_bytes(L, n) + n * (1 + 32 + 12) + weights,
            "flops": network + updates * OPS_PER_UPDATE}


# ---- the network in 64 bits ----------------------------------------------------
def _blocks(L, flat):
    sizes = [("W1", (32, 27)), ("b1", (32,)), ("W2", (32, 288)), ("b2", (32,)),
             ("W3", (32, 288)), ("b3", (32,)), ("Wh", (7, L * L * 32)), ("bh", (7,))]
    out, at = {}, 0
    for name, shape in sizes:
        count = int(np.prod(shape))
        out[name] = flat[at:at + count].reshape(shape)
        at += count
    return out


def _conv(x, w, b):
    """3x3 convolution with zero padding of x [n, L, L, c], weights [out][tap, c]."""
    n, L, _, c = x.shape
    pad = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    taps = [pad[:, dy:dy + L, dx:dx + L, :] for dy in range(3) for dx in range(3)]
    cols = torch.cat(taps, dim=3).reshape(n * L * L, 9 * c)
    return (cols @ w.t() + b).reshape(n, L, L, -1)


def _network(L, P, syn, p):
    n, ns = syn.shape[0], L * (L - 1)
    x = torch.zeros((n, L, L, 3), dtype=torch.float64, device=syn.device)
    x[:, :L - 1, :, 0] = syn[:, :ns].reshape(n, L - 1, L).double()
    x[:, :, :L - 1, 1] = syn[:, ns:].reshape(n, L, L - 1).double()
    x[:, :, :, 2] = p.double()[:, None, None]
    for w, b in (("W1", "b1"), ("W2", "b2"), ("W3", "b3")):
        x = torch.relu(_conv(x, P[w], P[b]))
    return x.reshape(n, -1) @ P["Wh"].t() + P["bh"]


def _wide(logits):
    """Logits as the library lays them out: 8 per sample, the last one 0."""
    return torch.nn.functional.pad(logits, (0, 1))


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("gate_train", "gated"):
        return None
    state = prepare(case, seed)
    L, n = case["L"], case["n"]
    if kind == "gated":
        P = _blocks(L, state["params"].double())
        p = torch.from_numpy(state["p"]).to(state["syn"].device)
        logits = [_network(L, P, state["syn"][i:i + 1024], p[i:i + 1024])
                  for i in range(0, n, 1024)]
        return dict(chosen=None, route=None, logits=_wide(torch.cat(logits)), counts=None,
                    correction=None)
    net = state["net"]
    params = net.params.double().requires_grad_(True)
    logits = _network(L, _blocks(L, params), state["syn"], state["p"])
    log_class = torch.log_softmax(logits[:, :4], dim=1)
    log_budget = torch.log_softmax(logits[:, 4:], dim=1)
    loss = -(state["target"].double() * log_class).sum(dim=1) \
        - 0.5 * log_budget.gather(1, state["budget"].long()[:, None])[:, 0]
    grads, = torch.autograd.grad(loss.mean(), params)
    params, loss, logits = params.detach(), loss.detach(), logits.detach()
    m, v = 0.1 * grads, 0.001 * grads * grads
    params = params - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return dict(logits=_wide(logits), grads=grads, loss=loss, params=params, m=m, v=v)
