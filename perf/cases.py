"""Timed cases of the simulator: what its users run, through the public Python calls.

A case is a dict of plain values; `kind` says which calls a pass makes:

* lattice   one lattice advanced by some Monte Carlo steps and observed
* ensemble  many lattices in one batch, advanced together and observed
* series    an ensemble measured on a list of times against a snapshot (aging)
* serve     requests queued on the server, drained and polled
* observe   the exact moments and correlations of given surfaces, no dynamics

Sizes are those of the workloads, the tests and the benchmark: lattices of
2^6 to 2^17 sites a side, device domains of 16 to 256 sites, thread cells of
8 x 8 sites (TC=1,1) and now and then 16 x 16 (TC=2,2), all three block
schemes, deposition alone (p = 1) and rates that need acceptance draws.
"""
import math
import random

import numpy as np
import torch

import paper_1705_01022_amd as okpz

SCHEMES = {"DT": okpz.BLOCK_DT, "DB": okpz.BLOCK_DB, "DTr": okpz.BLOCK_DTR}


def listed():
    return [
        # every MCS of the smallest lattice measured: one step and its roughness, latency alone
        {"name": "mcs-64", "kind": "lattice", "L": 64, "D": 16, "C": 8, "scheme": "DT", "p": 1.0, "q": 0.0,
         "warm": 20, "mcs": 1, "corr": False},
        # a short run of a small lattice by itself, as a user tries parameters out
        {"name": "run-1024-db", "kind": "lattice", "L": 1024, "D": 256, "C": 8, "scheme": "DB", "p": 0.8, "q": 0.2,
         "warm": 20, "mcs": 25, "corr": False},
        # the L=4096 workload, between two times of its logarithmic measurement grid
        {"name": "run-4096-dt", "kind": "lattice", "L": 4096, "D": 256, "C": 8, "scheme": "DT", "p": 1.0, "q": 0.0,
         "warm": 20, "mcs": 20, "corr": False},
        # a mid-size lattice, cell grid shifted every round, autocorrelation against a waiting time
        {"name": "run-16384-dtr", "kind": "lattice", "L": 16384, "D": 256, "C": 8, "scheme": "DTr", "p": 0.95,
         "q": 0.05, "warm": 10, "mcs": 3, "corr": True},
        # the paper's production size under DTrDT
        {"name": "run-65536-dt", "kind": "lattice", "L": 65536, "D": 256, "C": 8, "scheme": "DT", "p": 1.0, "q": 0.0,
         "warm": 6, "mcs": 1, "corr": True},
        # the benchmark step: the largest lattice, delayed borders, W^2 and C_h after every MCS
        {"name": "run-131072-db", "kind": "lattice", "L": 131072, "D": 256, "C": 8, "scheme": "DB", "p": 0.95,
         "q": 0.05, "warm": 4, "mcs": 1, "corr": True},
        # the batched workload: 512 realisations of four sizes, half KPZ, half equilibrium
        {"name": "batch-512-dt", "kind": "ensemble", "n": 512, "lo": 8, "hi": 11, "pick": 1, "D": 256, "C": 8,
         "scheme": "DT", "rates": "half", "warm": 10, "mcs": 15, "corr": False},
        # the 64 realisations of the L=4096 workload as one batch
        {"name": "batch-4096-dt", "kind": "ensemble", "n": 64, "lo": 12, "hi": 12, "pick": 1, "D": 256, "C": 8,
         "scheme": "DT", "rates": "kpz", "warm": 4, "mcs": 8, "corr": False},
        # a serving tick's worth of mixed requests as a batch
        {"name": "batch-mixed-db", "kind": "ensemble", "n": 24, "lo": 9, "hi": 13, "pick": 3, "D": 256, "C": 8,
         "scheme": "DB", "rates": "uniform", "warm": 4, "mcs": 16, "corr": True},
        # the aging ensemble: C_h(t, s) on a list of times
        {"name": "aging-512-db", "kind": "series", "n": 128, "lo": 9, "hi": 9, "pick": 1, "D": 256, "C": 8,
         "scheme": "DB", "rates": "kpz", "warm": 32, "times": 3, "last": 32},
        # the server from submission to result, requests of mixed sizes
        {"name": "serve-16", "kind": "serve", "n": 16, "lo": 9, "hi": 12, "pick": 2, "D": 256, "C": 8, "scheme": "DB",
         "mcs": 100},
        # both observables of a stored surface and its snapshot, no dynamics
        {"name": "observe-32768", "kind": "observe", "L": 32768, "sweeps": 12},
    ]


def draw(rng):
    kind = rng.choice(["lattice", "lattice", "lattice", "ensemble", "ensemble", "series", "serve", "observe"])
    scheme = rng.choice(["DT", "DT", "DB", "DB", "DTr"])
    C = rng.choice([8, 8, 8, 8, 16])
    if kind == "lattice":
        lg = rng.randint(6, 16)
        L = 1 << lg
        # 2 tiles at least; the design domain of 256 sites where it fits, smaller ones too
        D = rng.choice([d for d in (16, 32, 64, 128, 256, 256, 256) if 2 * d <= L and d >= C])
        p, q = rng.choice([(1.0, 0.0), (0.95, 0.05), (0.5, 0.5), (round(rng.uniform(0.5, 1.0), 4), None)])
        q = round(1.0 - p, 4) if q is None else q
        most = min(200, max(1, (1 << 33) // (L * L) // 4))
        mcs = max(1, int(round(math.exp(rng.uniform(0.0, math.log(most))))))
        return {"kind": kind, "L": L, "D": D, "C": C, "scheme": scheme, "p": p, "q": q, "warm": rng.randint(2, 20),
                "mcs": mcs, "corr": rng.random() < 0.5}
    if kind in ("ensemble", "series", "serve"):
        lo = rng.randint(8, 11)
        hi = min(12, lo + rng.randint(0, 3))
        n = int(round(math.exp(rng.uniform(math.log(4), math.log(400)))))
        n = max(3, min(n, (1 << 28) >> (2 * hi - 1)))
        case = {"kind": kind, "n": n, "lo": lo, "hi": hi, "pick": rng.randrange(1000),
                "D": rng.choice([64, 128, 256, 256, 256]), "C": C, "scheme": scheme}
        if kind == "serve":
            return dict(case, n=min(n, 40), mcs=rng.randint(20, 150))
        case["rates"] = rng.choice(["kpz", "half", "uniform"])
        case["warm"] = rng.randint(2, 12)
        if kind == "series":
            return dict(case, times=rng.randint(2, 5), last=rng.randint(5, 24))
        return dict(case, mcs=rng.randint(3, 24), corr=rng.random() < 0.5)
    return {"kind": kind, "L": 1 << rng.randint(7, 15), "sweeps": rng.randint(4, 20)}


# ---------------------------------------------------------------- members of an ensemble
def members(case):
    """(L, D, p, q) of each member: the sizes and rates belong to the case, the randomness to the seed."""
    rng = random.Random(case["pick"])
    out = []
    for _ in range(case["n"]):
        L = 1 << rng.randint(case["lo"], case["hi"])
        rates = case.get("rates", "uniform")
        if rates == "uniform":
            p = rng.uniform(0.5, 1.0)
            q = 1.0 - p
        else:
            p, q = (1.0, 0.0) if rates == "kpz" or rng.random() < 0.5 else (0.5, 0.5)
        out.append((L, min(case["D"], L // 2), p, q))
    return out


def times_of(case):
    """`times` log-spaced measurement times from 1 to `last` MCS after the snapshot."""
    k = case["times"]
    return sorted({max(1, round(case["last"] ** (i / (k - 1)))) for i in range(k)})


# ---------------------------------------------------------------- surfaces made without the library
def heights_of(L, seed, sweeps, start=None):
    """A rough periodic surface: checkerboard sweeps of random deposition on the flat one (or on `start`)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.arange(L, device="cuda", dtype=torch.int16)
    par = (x[None, :] + x[:, None]) & 1
    h = par.clone() if start is None else start.clone()
    for i in range(2 * sweeps):
        low = (par == (i & 1)) & (torch.rand(L, L, device="cuda", generator=gen) < 0.5)
        for dim in (0, 1):
            for s in (1, -1):
                low &= torch.roll(h, s, dim) > h
        h += 2 * low.to(torch.int16)
    return h


def slopes_of(h):
    """sx, sy: whether the step from the left / lower neighbour goes up."""
    return h > torch.roll(h, 1, 1), h > torch.roll(h, 1, 0)


def words_of(h):
    """The packed device layout of a surface: blocks of 32 x 4 sites, four sx words, then four sy words."""
    L = h.shape[0]
    out = torch.empty(L // 4, L // 32, 8, dtype=torch.int32, device="cuda")
    for plane, s in enumerate(slopes_of(h)):
        bits = s.view(L, L // 32, 32)
        w = torch.zeros(L, L // 32, dtype=torch.int32, device="cuda")
        for i in range(32):
            w |= bits[:, :, i].to(torch.int32) << i
        out[:, :, 4 * plane:4 * plane + 4] = w.view(L // 4, 4, L // 32).permute(0, 2, 1)
    return out.view(-1)


def surfaces(case, seed):
    hs = heights_of(case["L"], 2 * seed + 1, case["sweeps"])
    return hs, heights_of(case["L"], 2 * seed + 2, case["sweeps"], hs)


# ---------------------------------------------------------------- the passes
def on_tensor(words, L, D, C, scheme, seed, stream, hip_stream=None):
    return okpz.Lattice(L, D, D, C, C, SCHEMES[scheme], seed=seed, stream=stream, hip_stream=hip_stream,
                        device_buffer=(words.data_ptr(), 4 * words.numel()))


def prepare(case, seed):
    kind = case["kind"]
    seed &= 0xFFFFFFFF
    if kind == "lattice":
        words = torch.empty(case["L"] ** 2 // 16, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        lat = on_tensor(words, case["L"], case["D"], case["C"], case["scheme"], seed, 0)
        lat.run(case["warm"], case["p"], case["q"])
        if case["corr"]:
            lat.snapshot()
        lat.sync()
        return {"case": case, "words": words, "lat": lat}
    if kind in ("ensemble", "series"):
        mem = members(case)
        words = torch.empty(sum(L * L // 16 for L, _, _, _ in mem), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        batch, lats, at = okpz.Batch(), [], 0
        for i, (L, D, _, _) in enumerate(mem):
            lat = on_tensor(words[at:at + L * L // 16], L, D, case["C"], case["scheme"], seed, i, batch.hip_stream)
            at += L * L // 16
            batch.add(lat)
            lats.append(lat)
        p, q = [m[2] for m in mem], [m[3] for m in mem]
        # the waiting time, then the reference state
        batch.run([case["warm"]] * len(mem), p, q)
        if kind == "series" or case["corr"]:
            batch.snapshot()
        batch.sync()
        return {"case": case, "words": words, "batch": batch, "lats": lats, "p": p, "q": q,
                "times": times_of(case) if kind == "series" else None}
    if kind == "serve":
        return {"case": case, "server": okpz.Server(), "members": members(case), "seed": seed}
    hs, ht = surfaces(case, seed)
    words = torch.empty(case["L"] ** 2 // 16, dtype=torch.int32, device="cuda")
    D = min(256, case["L"] // 2)
    torch.cuda.synchronize()
    lat = on_tensor(words, case["L"], D, 8, "DB", seed, 0)
    words.copy_(words_of(hs))
    lat.snapshot()
    words.copy_(words_of(ht))
    torch.cuda.synchronize()
    return {"case": case, "words": words, "lat": lat}


def column(obs, part, key):
    return np.array([obs[r][part][key] for r in range(len(obs))])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "lattice":
        state["lat"].run(case["mcs"], case["p"], case["q"])
        mo, ac = state["lat"].observe(case["corr"])
        return {"words": state["words"], "moments": mo, "corr": ac}
    if kind == "ensemble":
        b = state["batch"]
        b.run([case["mcs"]] * case["n"], state["p"], state["q"])
        obs = b.observe(case["corr"])
        return {"words": state["words"], "w2": column(obs, 0, "w2"), "w2_sub": column(obs, 0, "w2_sub"),
                "c_h": column(obs, 1, "c_h") if case["corr"] else None,
                "c_s": column(obs, 1, "c_s") if case["corr"] else None}
    if kind == "series":
        out = state["batch"].series(state["times"], state["p"], state["q"], with_autocorr=True)
        return {"words": state["words"], "w2": [column(o, 0, "w2") for o in out],
                "c_h": [column(o, 1, "c_h") for o in out], "c_s": [column(o, 1, "c_s") for o in out]}
    if kind == "serve":
        srv = state["server"]
        for i, (L, D, p, q) in enumerate(state["members"]):
            srv.submit(L, D, D, case["C"], case["C"], SCHEMES[case["scheme"]], state["seed"], i, case["mcs"], p, q)
        srv.drain()
        got = sorted(srv.poll(len(state["members"])), key=lambda r: r["id"])
        return {k: np.array([r["moments"][k] for r in got]) for k in ("w2", "w2_sub", "s1_even", "s2_even", "s2_odd")}
    mo, ac = state["lat"].observe(True)
    return {"moments": mo, "corr": ac}


# ---------------------------------------------------------------- work and exact values
def attempts_of(case):
    """Update attempts (an MCS is L^2 of them) and the sites measured."""
    kind = case["kind"]
    if kind == "lattice":
        return case["mcs"] * case["L"] ** 2, case["L"] ** 2 * (2 if case["corr"] else 1)
    if kind in ("ensemble", "series", "serve"):
        sites = sum(m[0] ** 2 for m in members(case))
        if kind == "series":
            t = times_of(case)
            return t[-1] * sites, 2 * len(t) * sites
        return case["mcs"] * sites, (2 if case.get("corr") else 1) * sites
    return 0, 2 * case["L"] ** 2


def work(case):
    """Bytes: each MCS reads and writes every site's two bits, a measurement reads them (and the snapshot's).
    Operations: the four slopes tested and, where they allow it, turned, per attempt; one add and one
    multiply-add per height."""
    attempts, measured = attempts_of(case)
    return {"bytes": attempts / 2 + measured / 4, "flops": 8 * attempts + 3 * measured}


def exact(case, seed):
    """The observables of surfaces that this file makes itself; the dynamics' outputs are whole numbers."""
    seed &= 0xFFFFFFFF
    if case["kind"] != "observe":
        return None
    L = case["L"]
    N = L * L
    hs, ht = surfaces(case, seed)
    overlap = sum(int((a & b).sum()) for a, b in zip(slopes_of(hs), slopes_of(ht)))
    hs, ht = hs - hs[0, 0], ht - ht[0, 0]
    x = torch.arange(L, device="cuda")
    s1, s2, s1s, sts = [0, 0], [0, 0], 0, 0
    for y in range(0, L, 1024):  # a strip at a time, in 64 bits
        a, b = ht[y:y + 1024].long(), hs[y:y + 1024].long()
        odd = ((x[None, :] + torch.arange(y, y + a.shape[0], device="cuda")[:, None]) & 1).long()
        for k, m in enumerate((1 - odd, odd)):
            s1[k] += int((a * m).sum())
            s2[k] += int((a * a * m).sum())
        s1s += int(b.sum())
        sts += int((a * b).sum())
    half = N // 2
    var = [half * s2[k] - s1[k] ** 2 for k in (0, 1)]
    mo = {"mcs": 0, "n_even": half, "n_odd": half, "s1_even": s1[0], "s1_odd": s1[1], "s2_even": s2[0],
          "s2_odd": s2[1], "w2": (N * sum(s2) - sum(s1) ** 2) / N ** 2, "w2_sub": 2 * sum(var) / N ** 2}
    ac = {"t": 0, "s": 0, "s_ts": sts, "s1_t": sum(s1), "s1_s": s1s, "c_h": (N * sts - sum(s1) * s1s) / N ** 2,
          "overlap": overlap, "c_s": overlap / (2 * N) - 0.25}
    return {"moments": mo, "corr": ac}
