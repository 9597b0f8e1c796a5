"""Measured workloads of the multicanonical framework.

One pass of a case is one multicanonical iteration as a user's program runs
it: the sweeps of every chain, then the merge (histogram, flatness, weight
recursion, new thresholds).  The state that `prepare` hands over is a run
with a few iterations behind it, so that the weights are measured ones and
reject moves.  Sizes are those of the batched, serving, speedup and polymer
workloads of `synth` and `bench.py`, with sweeps per iteration from their
power laws where one pass stays short.

Outputs of a pass: the merged histogram, the new log weights, the
iteration's statistics and the whole configuration (a view of the run's own
workspace, where the chains live).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1312_2213_amd import muca
from synth import PAPER_POLYMER, WORKLOADS, sweeps_per_iteration

SIZES = (8, 16, 24, 32, 48, 64)
LAYOUTS = {"auto": muca.MUCA_LAYOUT_AUTO, "bit": muca.MUCA_LAYOUT_BIT, "byte": muca.MUCA_LAYOUT_BYTE}


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def lattice(name, model, L, chains, sweeps, q=2, layout="auto", beta=0.5, warm=8, em=False):
    return {"name": name, "kind": "lattice", "model": model, "L": L, "q": q, "chains": chains, "sweeps": sweeps,
            "layout": layout, "beta": beta, "warm": warm, "em": em}


def listed():
    return [
        # the smallest runs of the time-speedup study: 8 x 8, M_opt / p sweeps,
        # an iteration of a few hundred microseconds where launches and the
        # merge's round trip count
        lattice("ising8_short", "ising", 8, 64, 17, warm=30),
        # a served request of the smallest lattice (10 sweeps per iteration)
        lattice("ising16_served", "ising", 16, 1024, 10, warm=30),
        # int8 spins and a chain count that is no multiple of a wavefront
        lattice("ising32_int8_ragged", "ising", 32, 1000, 35, layout="byte"),
        # the headline configuration (Ising L = 64, bit-packed, 4096 chains)
        lattice("ising64_4096", "ising", 64, 4096, 400, layout="bit"),
        # the same lattice with the chip full of chains
        lattice("ising64_131072", "ising", 64, 131072, 50, layout="bit"),
        # multimagnetic production sweeps with the joint (E, M) histogram
        lattice("muma32_em", "muma", 32, 512, 67, layout="bit", em=True),
        # a served Potts request, ragged in chains and in rows per wavefront
        lattice("potts24_q3_ragged", "potts", 24, 700, 100, q=3),
        # the longest instance of the batched workload, at its own sweep count
        lattice("potts48_q8", "potts", 48, 2048, 362, q=8),
        # the q scan at 64 x 64: the threshold table exceeds LDS
        lattice("potts64_q10", "potts", 64, 1024, 60, q=10),
        # one round of the batched workload: four Potts and four
        # multimagnetic runs in one persistent launch, then their merges
        {"name": "batched_round", "kind": "batch", "set": "potts8_batched", "runs": 8, "seed0": 0, "chains": 0,
         "updates": 0, "warm": 1},
        # the homopolymer workload, 100 of its 1000 sweeps per iteration, and
        # the rebuild of its 2500 x 2500 threshold matrix
        {"name": "polymer40_shifts", "kind": "polymer", "beads": 40, "chains": 4096, "sweeps": 100, "therm": 0,
         "bins": 2500, "lo": -200.0, "hi": 50.0, "moves": 0, "paper": False, "warm": 1},
        # the paper's homopolymer with its full move set, two beads per lane,
        # thermalisation before the recorded sweeps
        {"name": "polymer80_paper", "kind": "polymer", "beads": 80, "chains": 512, "sweeps": 20, "therm": 5,
         "bins": 1000, "lo": -220.0, "hi": 40.0, "moves": 1, "paper": True, "warm": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lattice"] * 7 + ["batch"] + ["polymer"] * 2)
    if kind == "batch":
        return {"kind": "batch", "set": "serving", "runs": rng.randint(2, 6), "seed0": rng.randint(1, 1000),
                "chains": _log_int(rng, 64, 2048), "updates": _log_int(rng, 4096, 65536), "warm": 1}
    if kind == "polymer":
        paper = rng.random() < 0.5
        beads = _log_int(rng, 20, 100 if paper else 80)
        chains = _log_int(rng, 16, 4096)
        sweeps = max(1, min(200, int(8e6 / (chains * beads))))
        return {"kind": "polymer", "beads": beads, "chains": chains, "sweeps": rng.randint(1, sweeps),
                "therm": rng.choice([0, 2]), "bins": _log_int(rng, 50, 2500), "lo": -5.0 * beads, "hi": 60.0,
                "moves": int(paper), "paper": paper, "warm": 1}
    model = rng.choice(["ising", "ising", "muma", "potts", "potts"])
    L = rng.choice(SIZES)
    q = rng.choice([2, 3, 4, 5, 6, 8, 10]) if model == "potts" else 2
    chains = _log_int(rng, 16, 16384)
    law = sweeps_per_iteration(L, chains, model == "potts" and q >= 3)
    # at most 4e5 updates per chain (1e5 where the table is read from memory)
    # and 2e9 in all
    cap = min((1e5 if model != "ising" and L == 64 else 4e5) / (L * L), 2e9 / (chains * L * L))
    sweeps = max(1, min(law, int(cap), _log_int(rng, 5, 500)))
    layout = rng.choice(["auto", "bit", "byte"]) if model != "potts" else "auto"
    c = lattice("", model, L, chains, sweeps, q=q, layout=layout, beta=rng.choice([0.3, 0.5, 0.661]),
                warm=30 if L <= 16 else 8, em=model == "muma" and L <= 48 and rng.random() < 0.3)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# States
# ---------------------------------------------------------------------------
def _walks(beads, chains, seed, bond, min_dist):
    """Self-avoiding start conformations [chain][bead][3]: unit steps uniform
    on the sphere, re-drawn where a bead comes closer than `min_dist` to an
    earlier one that it is not bonded to."""
    rng = np.random.default_rng(seed)
    x = np.zeros((chains, beads, 3))
    for k in range(1, beads):
        left = np.arange(chains)
        for tries in range(1000):
            v = rng.normal(size=(len(left), 3))
            y = x[left, k - 1] + bond * v / np.linalg.norm(v, axis=1, keepdims=True)
            x[left, k] = y
            if k < 2:
                break
            d2 = np.sum((x[left, :k - 1] - y[:, None]) ** 2, axis=2).min(axis=1)
            left = left[d2 < min_dist * min_dist]
            if not len(left):
                break
        else:
            raise RuntimeError("could not place a bead")
    return x.astype(np.float32)


def _specs(case):
    """(config, sweeps) of every run of a batched case."""
    out = []
    if case["set"] == "potts8_batched":
        for inst in WORKLOADS["potts8_batched"]["instances"]:
            potts = inst["model"] == "potts"
            kw = {} if potts else {"beta": inst["beta"], "layout": muca.MUCA_LAYOUT_BIT}
            out.append((dict(model=inst["model"], L=inst["L"], q=inst.get("q", 2), chains=inst["chains"], **kw),
                        sweeps_per_iteration(inst["L"], inst["chains"], potts)))
        return out
    rng = np.random.default_rng(case["seed0"])
    for _ in range(case["runs"]):  # the serving mix, each run one chunk of a round
        if rng.random() < 0.5:
            m, L, q = "ising", int(rng.choice([16, 24, 32, 48, 64])), 2
        else:
            m, L, q = "potts", int(rng.choice([16, 32])), int(rng.choice([2, 4, 6, 8, 10]))
        chains = max(1, int(case["chains"] * rng.uniform(0.5, 1.0)))
        out.append((dict(model=m, L=L, q=q, chains=chains), max(1, case["updates"] // (L * L))))
    return out


def _lattice_view(run):
    """The configurations of a lattice run: [words][chain] of its workspace,
    without the padding chains."""
    cfg = run.cfg
    bits = cfg.model != muca.MUCA_POTTS and cfg.layout != muca.MUCA_LAYOUT_BYTE
    words = cfg.L * (-(-cfg.L // 32) if bits else cfg.L // 4)
    pad = -(-cfg.n_chains // 64) * 64
    off = run._ws_ptr.value - run.workspace.data_ptr()
    w = run.workspace[off:off + 4 * words * pad].view(torch.int32).view(words, pad)
    return w[:, :cfg.n_chains]


def _polymer_view(run):
    """The bead positions [chain][bead][3] of a polymer run's workspace."""
    cfg = run.cfg
    slots = 128 if cfg.n_beads > 64 else 64
    off = run._ws_ptr.value - run.workspace.data_ptr()
    w = run.workspace[off:off + 16 * slots * cfg.n_chains].view(torch.float32).view(cfg.n_chains, slots, 4)
    return w[:, :cfg.n_beads, :3]


def _warm_sweeps(sweeps):
    return max(1, min(sweeps, 40))


def prepare(case, seed):
    if case["kind"] == "polymer":
        pp = dict(PAPER_POLYMER) if case["paper"] else {}
        bond, dist = (pp["fene_r0"], pp["lj_sigma"]) if case["paper"] else (1.0, 1.0)
        cfg = muca.muca_config_default("polymer", 0, 2, case["chains"], 7000 + seed, n_beads=case["beads"],
                                       x_lo=case["lo"], x_hi=case["hi"], n_bins=case["bins"], moves=case["moves"], **pp)
        run = muca.Run(cfg, positions=_walks(case["beads"], case["chains"], seed, bond, dist))
        for _ in range(case["warm"]):
            run.run_iteration(_warm_sweeps(case["sweeps"]))
            run.merge_update()
        return {"case": case, "run": run, "view": _polymer_view(run)}
    if case["kind"] == "batch":
        stream = torch.cuda.Stream()
        specs = _specs(case)
        runs = []
        for k, (s, _) in enumerate(specs):
            kw = {n: s[n] for n in ("beta", "layout") if n in s}
            runs.append(muca.Run(muca.muca_config_default(s["model"], s["L"], s["q"], s["chains"],
                                                          1000 * seed + 30 + k, **kw), stream=stream))
        batch = muca.Batch(len(runs))
        state = {"case": case, "batch": batch, "runs": runs, "stream": stream, "views": [_lattice_view(r) for r in runs],
                 "sweeps": [sw for _, sw in specs]}
        for _ in range(case["warm"]):
            batch.run_iteration(runs, [_warm_sweeps(sw) for sw in state["sweeps"]], stream=stream)
            for r in runs:
                r.merge_update()
        return state
    kw = {"layout": LAYOUTS[case["layout"]]}
    if case["model"] == "muma":
        kw["beta"] = case["beta"]
    run = muca.Run(muca.muca_config_default(case["model"], case["L"], case["q"], case["chains"], seed, **kw))
    for _ in range(case["warm"]):
        run.run_iteration(_warm_sweeps(case["sweeps"]))
        run.merge_update()
    state = {"case": case, "run": run, "view": _lattice_view(run)}
    if case["em"]:
        ne, nm = run.em_shape()
        state["em"] = torch.zeros(ne, nm, dtype=torch.int64, device="cuda")
    return state


def _outputs(run, st, view):
    return {"hist": run.last_hist().view(np.int64), "lnw": run.lnw(), "flatness": st["flatness"],
            "accept_rate": st["accept_rate"], "samples": st["samples"], "state": view}


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        state["batch"].run_iteration(state["runs"], state["sweeps"], stream=state["stream"])
        return [_outputs(r, r.merge_update(), v) for r, v in zip(state["runs"], state["views"])]
    r = state["run"]
    if case["kind"] == "polymer":
        if case["therm"]:
            r.thermalize(case["therm"])
        r.run_iteration(case["sweeps"])
        return _outputs(r, r.merge_update(), state["view"])
    if case["em"]:
        r.run_iteration_em(case["sweeps"], state["em"])
        return {**_outputs(r, r.merge_update(), state["view"]), "em": state["em"]}
    r.run_iteration(case["sweeps"])
    return _outputs(r, r.merge_update(), state["view"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _lattice_work(model, L, q, chains, sweeps, layout):
    n = L * L
    bins = n + 1 if model != "potts" else 2 * n + 1
    cols = {"ising": 5, "potts": 9, "muma": 10}[model]
    site = 1.0 if model == "potts" or layout == "byte" else 0.125
    # spins in and out, thresholds in, histogram and new weights out; per
    # attempt 10 operations per Philox word and 13 of the Metropolis step
    return 2.0 * site * n * chains + 4.0 * bins * cols + 16.0 * bins, (33.0 if model == "potts" else 23.0) * n * chains * sweeps


def work(case):
    if case["kind"] == "batch":
        parts = [_lattice_work(s["model"], s["L"], s["q"], s["chains"], sw, "bit") for s, sw in _specs(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if case["kind"] == "polymer":
        n, c = case["beads"], case["chains"]
        moves = (2 * n + 1 if case["moves"] else n) * (case["sweeps"] + case["therm"])
        # 22 operations per new pair term, 40 per bond, 40 for the proposal
        return {"bytes": 2.0 * 12 * n * c + 4.0 * case["bins"] ** 2, "flops": (22.0 * (n - 1) + 120.0) * moves * c}
    b, f = _lattice_work(case["model"], case["L"], case["q"], case["chains"], case["sweeps"], case["layout"])
    if case["em"]:
        b += 8.0 * case["chains"] * case["sweeps"]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same numbers from plain numpy in 64 bits, for runs short enough to
# follow update by update
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, key):
    x = [np.asarray(v, np.uint64) for v in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    mask, s32 = np.uint64(0xFFFFFFFF), np.uint64(32)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * x[0], np.uint64(0xCD9E8D57) * x[2]
        x = [(p1 >> s32) ^ x[1] ^ np.uint64(k0), p1 & mask, (p0 >> s32) ^ x[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(x, axis=-1)


def exact(case, seed):
    """Ising iterations from the start in numpy; None where that is too long."""
    if case["kind"] != "lattice" or case["model"] != "ising":
        return None
    L, C = case["L"], case["chains"]
    N = L * L
    plan = [_warm_sweeps(case["sweeps"])] * case["warm"] + [case["sweeps"]]
    if sum(plan) * N > 60000 or C > 4096:
        return None
    chain = np.arange(C)
    words = _philox(chain[:, None], 0, np.arange(N // 4)[None], 1, seed).reshape(C, N)
    s = np.where(words >> np.uint64(31), 1, -1).astype(np.int64)
    g = s.reshape(C, L, L)
    E = -(g * np.roll(g, -1, 1) + g * np.roll(g, -1, 2)).sum((1, 2))
    B = N + 1
    use = np.ones(B, bool)
    use[[1, B - 2]] = False  # E = +-(2N - 4) does not occur
    idx = np.flatnonzero(use)
    lnW, lnR, P, step = np.zeros(B), np.zeros(len(idx) - 1), np.zeros(len(idx) - 1), 0
    y, x = np.divmod(np.arange(N), L)
    nb = [y * L + (x + 1) % L, y * L + (x - 1) % L, ((y + 1) % L) * L + x, ((y - 1) % L) * L + x]
    nb = np.stack(nb, axis=1)
    for sweeps in plan:
        H, acc_n = np.zeros(B, np.int64), 0
        for _ in range(sweeps):
            r = _philox(chain[:, None], step, np.arange(N // 4)[None], 0, seed).reshape(C, N)
            for i in range(N):
                dE = 2 * s[:, i] * s[:, nb[i]].sum(1)
                b, t = (E + 2 * N) // 4, (E + dE + 2 * N) // 4
                D = lnW[t] - lnW[b]
                T = np.where(D >= 0, 4294967295.0, np.minimum(np.floor(np.exp(np.minimum(D, 0.0)) * 4294967296.0),
                                                              4294967295.0))
                ok = (T == 4294967295.0) | (r[:, i] < T)
                acc_n += int(ok.sum())
                s[ok, i] *= -1
                E = E + np.where(ok, dE, 0)
            H += np.bincount((E + 2 * N) // 4, minlength=B)
            step += 1
        h = H[idx].astype(np.float64)
        h0, h1 = h[:-1], h[1:]
        both = (h0 > 0) & (h1 > 0)
        p = np.where(both, h0 * h1 / np.maximum(h0 + h1, 1.0), 0.0)
        P += p
        d = np.log(np.maximum(h0, 1.0)) - np.log(np.maximum(h1, 1.0))
        lnR += np.where(both, p / np.maximum(P, 1e-300) * d, 0.0)
        run_ = np.concatenate([[0.0], np.cumsum(lnR)])
        lnW = run_[np.searchsorted(idx, np.arange(B), side="right") - 1]
    return {"lnw": lnW, "flatness": float(h.min() / h.mean()), "accept_rate": acc_n / (plan[-1] * C * N)}
