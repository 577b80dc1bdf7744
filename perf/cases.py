"""Timed work of this framework, through its public Python entry points.

A case is one piece of work that a program using the framework has it do:

  anneal      one population from creation to its last temperature, by the
              constant-culling step choice or on a linear schedule, any coupling
              model and layout, with its final energies and family labels
  pair        two populations of one disorder sample on a linear schedule, with
              the spin-overlap histogram after every step
  sweep       Metropolis sweeps and observables of a resident population
  overlap     spin- and link-overlap histograms of two resident populations
  batch       many instances of mixed sizes through one schedule
  serve       a request loop over runs of mixed sizes that come and go
  checkpoint  the whole state of a population to the host and back

``prepare`` holds what a program has before the call: the couplings, the seeds,
and for the resident kinds the population itself.  ``exact`` gives the FP64
scalars of the smaller cases from a plain 64-bit simulation in torch.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import pa_inputs
import paper_1711_02146_amd as pam

LATTICES = (4, 6, 8, 10, 12, 14, 16)
# a step's record: what a program plots or stores per temperature
REAL_FIELDS = ("beta", "lnQ", "beta_F", "mean_E", "rho_t", "eps_expected", "E_lowest")
COUNT_FIELDS = ("R_tilde", "n_culled", "n_at_E_min", "sum_eta2")


def listed():
    return [
        # the smallest whole run (L = 4, a thousand replicas, int8): many short
        # launches, latency everywhere
        dict(name="anneal_pm_l4_r1000", kind="anneal", model="pm", L=4, R=1000, layout="int8",
             eps=0.0, n_temps=51, beta_max=5.0, n_sweeps=10, state="all"),
        # two populations of one sample with their overlap histogram per step, int8
        dict(name="pair_pm_l8_r100k", kind="pair", L=8, R=100000, layout="int8", n_temps=201,
             beta_max=5.0, n_sweeps=10),
        # the headline run: one +-J instance at L = 10, half a million replicas
        dict(name="anneal_pm_l10_r500k", kind="anneal", model="pm", L=10, R=500000,
             layout="bitpack64", eps=0.1, n_temps=0, beta_max=5.0, n_sweeps=10, state="energies"),
        # a production-size population (the paper's reach 1.5e7), the hot part of its schedule
        dict(name="anneal_pm_l8_r3m", kind="anneal", model="pm", L=8, R=3000000, layout="auto",
             eps=0.1, n_temps=0, beta_max=0.5, n_sweeps=10, state="energies"),
        # the largest lattice: sweeps and observables of a resident population,
        # a ragged size
        dict(name="sweep_pm_l16_r100k", kind="sweep", model="pm", L=16, R=100003, layout="auto",
             beta=1.0, n_sweeps=10),
        # Gaussian couplings rounded to 1/16, the same run as the headline one
        dict(name="anneal_g16_l10_r500k", kind="anneal", model="gauss16", L=10, R=500000,
             layout="bitpack64", eps=0.1, n_temps=0, beta_max=5.0, n_sweeps=10, state="energies"),
        # real Gaussian couplings (the paper's own model), the same run
        dict(name="anneal_gauss_l10_r500k", kind="anneal", model="gauss", L=10, R=500000,
             layout="bitpack64", eps=0.1, n_temps=0, beta_max=5.0, n_sweeps=10, state="energies"),
        # real couplings at the paper's smallest lattice, an odd and modest population
        dict(name="anneal_gauss_l6_r20k", kind="anneal", model="gauss", L=6, R=20011,
             layout="auto", eps=0.1, n_temps=0, beta_max=5.0, n_sweeps=10, state="energies"),
        # q and q_l of two resident populations
        dict(name="overlap_pm_l10_r500k", kind="overlap", model="pm", L=10, R=500000,
             layout="bitpack64", beta=0.3),
        # a batch of instances of mixed sizes, two populations each
        dict(name="batch_12", kind="batch", instances=12, sizes=0xBA7C4, R_lo=20000, R_hi=100000,
             n_temps=101, beta_max=5.0, n_sweeps=10),
        # continuous batching: requests that overlap on the device
        dict(name="serve_8", kind="serve", requests=8, sizes=0x5E4E, rate=24.0, R_lo=10000,
             R_hi=200000, T_lo=51, T_hi=201, n_sweeps=10, beta_max=5.0),
        # a checkpoint out and in
        dict(name="checkpoint_pm_l8_r100k", kind="checkpoint", model="pm", L=8, R=100000,
             layout="bitpack64", beta=0.5),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("anneal", "anneal", "anneal", "anneal", "pair", "sweep", "sweep",
                       "overlap", "batch", "serve", "checkpoint"))
    L = rng.choice(LATTICES)
    N = L ** 3
    layout = rng.choice(("auto", "int8", "bitpack64"))
    model = rng.choice(("pm", "gauss16", "gauss"))
    if kind == "anneal":
        R = _log_uniform(rng, 1000, min(3e6, (1.5e8 if model == "pm" else 6e7) / N))
        linear = rng.random() < 0.4
        return dict(kind=kind, model=model, L=L, R=R, layout=layout,
                    eps=0.0 if linear else rng.choice((0.1, 0.15, 0.2)),
                    n_temps=rng.randint(20, 60) if linear else 0,
                    beta_max=round(rng.uniform(0.3, 1.0 if N > 1000 else 5.0), 3),
                    n_sweeps=rng.choice((3, 10, 10, 22)), state="energies")
    if kind == "pair":
        return dict(kind=kind, L=L, R=_log_uniform(rng, 1000, min(1e6, 5e7 / N)), layout=layout,
                    n_temps=rng.randint(20, 101), beta_max=5.0, n_sweeps=10)
    if kind == "sweep":
        return dict(kind=kind, model=model, L=L, R=_log_uniform(rng, 1000, min(3e6, 5e8 / N)),
                    layout=layout, beta=round(rng.uniform(0.05, 3.0), 3),
                    n_sweeps=rng.choice((1, 3, 10, 22)))
    if kind == "overlap":
        return dict(kind=kind, model=model, L=L, R=_log_uniform(rng, 1000, min(3e6, 5e8 / N)),
                    layout=layout, beta=round(rng.uniform(0.1, 1.0), 3))
    if kind == "batch":
        lo = _log_uniform(rng, 1000, 40000)
        return dict(kind=kind, instances=rng.randint(2, 12), sizes=rng.randrange(1 << 30),
                    R_lo=lo, R_hi=2 * lo, n_temps=rng.randint(20, 80), beta_max=5.0, n_sweeps=10)
    if kind == "serve":
        return dict(kind=kind, requests=rng.randint(3, 8), sizes=rng.randrange(1 << 30),
                    rate=rng.choice((4.0, 12.0, 24.0)), R_lo=5000, R_hi=100000, T_lo=31, T_hi=101,
                    n_sweeps=10, beta_max=5.0)
    return dict(kind=kind, model=model, L=L, R=_log_uniform(rng, 1000, min(1e6, 5e7 / N)),
                layout=layout, beta=round(rng.uniform(0.1, 2.0), 3))


# --- inputs ------------------------------------------------------------------
def _couplings(model, L, seed):
    make = {"pm": pa_inputs.couplings_pm, "gauss16": pa_inputs.couplings_gauss16,
            "gauss": pa_inputs.couplings_gauss}[model]
    return make(L, seed)


def _batch_sizes(case):
    """(L, R) of every instance, from the case alone."""
    r = random.Random(case["sizes"])
    return [(r.choice((4, 6, 8, 10)), r.randint(case["R_lo"], case["R_hi"]))
            for _ in range(case["instances"])]


def _request_sizes(case):
    """(arrival, L, R, n_temps) of every request, from the case alone."""
    r = random.Random(case["sizes"])
    t, out = 0.0, []
    for _ in range(case["requests"]):
        t += r.expovariate(case["rate"])
        out.append((t, r.choice((4, 6, 8, 10, 12)), _log_uniform(r, case["R_lo"], case["R_hi"]),
                    r.randint(case["T_lo"], case["T_hi"])))
    return out


def _population(case, J, seed, stream=None):
    return pam.Population(case["L"], case["R"], J, seed, layout=case["layout"],
                          model=case.get("model", "pm"), stream=stream)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind in ("anneal", "pair", "sweep", "overlap", "checkpoint"):
        s["J"] = _couplings(case.get("model", "pm"), case["L"], 2 * seed + 1)
        s["seeds"] = (0x5EED0000 + 2 * seed, 0x5EED0001 + 2 * seed)
    if kind == "sweep":
        s["pop"] = _population(case, s["J"], s["seeds"][0])
        s["pop"].sweep(case["beta"], 10)
    elif kind == "overlap":
        s["pops"] = [_population(case, s["J"], x) for x in s["seeds"]]
        for p in s["pops"]:
            p.sweep(case["beta"], 10)
    elif kind == "checkpoint":
        s["pop"] = _population(case, s["J"], s["seeds"][0])
        s["pop"].sweep(case["beta"], 10)
        s["obs"] = s["pop"].observables()
    elif kind == "batch":
        s["stream"] = torch.cuda.Stream()
        s["insts"] = [(L, R, pa_inputs.couplings_pm(L, 1000 * seed + i),
                       (0x5EED0000 + 2 * (1000 * seed + i), 0x5EED0001 + 2 * (1000 * seed + i)))
                      for i, (L, R) in enumerate(_batch_sizes(case))]
        s["betas"] = pam.linear_schedule(case["beta_max"], case["n_temps"])
    elif kind == "serve":
        from paper_1711_02146_amd import serve
        s["server"] = serve.Server(hbm_budget=16 << 30, max_active=32, max_L=12)
        s["requests"] = [serve.Request(rid=i, arrival=t, L=L, R=R, n_temps=n,
                                       n_sweeps=case["n_sweeps"], beta_max=case["beta_max"],
                                       J=pa_inputs.couplings_pm(L, 1000 * seed + i),
                                       seed=0x5EED0000 + 1000 * seed + i)
                         for i, (t, L, R, n) in enumerate(_request_sizes(case))]
    return s


# --- one pass ----------------------------------------------------------------
# The number of steps and the final population size follow from the run, so
# its results go to the front of arrays of a fixed length, zeros after them.
def _rows(c):
    return c["n_temps"] - 1 if c["n_temps"] else 64 + 4 * int(_steps(c))


def _slots(c):
    return c["R"] + 16 * math.isqrt(c["R"]) + 256  # the library's default capacity


def _front(values, n):
    out = np.zeros((n,) + values.shape[1:], values.dtype)
    out[:len(values)] = values
    return out


def _columns(records, rows=None):
    rows = len(records) if rows is None else rows
    out = {f: _front(np.array([o[f] for o in records], np.float64), rows) for f in REAL_FIELDS}
    out.update({f: _front(np.array([o[f] for o in records], np.int64), rows)
                for f in COUNT_FIELDS})
    return out


def _state(pop, c):
    """Final spins (all), energies and family labels on the host."""
    spins, words, fam = pop.export_state(spins=c["state"] == "all")
    n = _slots(c)
    out = {"energies": _front(words if words.dtype == np.float64 else words.view(np.int32), n),
           "families": _front(fam.view(np.int32), n)}
    if spins is not None:
        out["spins"] = _front(spins, n)
    return out


def _run_anneal(s):
    c = s["case"]
    pop = _population(c, s["J"], s["seeds"][0])
    if c["n_temps"]:
        betas = pam.linear_schedule(c["beta_max"], c["n_temps"])
        records = [pop.step_to(b, c["n_sweeps"]) for b in betas[1:]]
    else:
        records = pop.anneal_run(c["eps"], c["beta_max"], c["n_sweeps"], 100000)
    out = {**_columns(records, _rows(c)), **_state(pop, c)}
    pop.close()
    return out


def _run_pair(s):
    c = s["case"]
    pops = [_population(c, s["J"], x) for x in s["seeds"]]
    records, q = [], []
    for b in pam.linear_schedule(c["beta_max"], c["n_temps"])[1:]:
        records += [p.step_to(b, c["n_sweeps"]) for p in pops]
        q.append(pam.overlap_hist(*pops))
    for p in pops:
        p.close()
    return {**_columns(records), "q": np.stack(q).view(np.int64)}


def _run_batch(s):
    c = s["case"]
    pops = [pam.Population(L, R, J, x, stream=s["stream"]) for L, R, J, xs in s["insts"]
            for x in xs]
    b = pam.Batch(pops, s["betas"], c["n_sweeps"],
                  pairs=[(2 * i, 2 * i + 1) for i in range(len(s["insts"]))])
    b.run()
    records, q, status = b.results()
    b.close()
    for p in pops:
        p.close()
    return {**_columns([o for step in records for o in step]), "q": q.view(np.int64),
            "status": status}


def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "anneal":
        return _run_anneal(s)
    if kind == "pair":
        return _run_pair(s)
    if kind == "sweep":
        s["pop"].sweep(c["beta"], c["n_sweeps"])
        return _columns([s["pop"].observables()])
    if kind == "overlap":
        return {"q": pam.overlap_hist(*s["pops"]).view(np.int64),
                "q_l": pam.link_overlap_hist(*s["pops"]).view(np.int64)}
    if kind == "batch":
        return _run_batch(s)
    if kind == "serve":
        done = s["server"].run(s["requests"], realtime=False, tick_dt=0.002)
        return {**_columns([r.final for r in done]),
                "status": np.array([r.status for r in done], np.int64)}
    spins, words, fam = s["pop"].export_state()
    o = s["obs"]
    s["pop"].import_state(spins, fam, o["sweeps_done"], o["step"], o["beta"], o["sum_lnQ"])
    return {"spins": spins, "families": fam.view(np.int32),
            "energies": words if words.dtype == np.float64 else words.view(np.int32),
            **_columns([s["pop"].observables()])}


# --- what a pass cannot do without -------------------------------------------
# Lane operations of one spin-flip attempt: a quarter of a Philox4x32-10 call
# (ten rounds of two multiplies and two XORs, 40 / 4), the bond arithmetic of a
# site shared by 64 replicas, a compare and a select.
OPS_PER_ATTEMPT = 13.59
# steps of a constant-culling run to beta = 5 at eps = 0.1, about, for N sites:
# a step is eps sqrt(2 pi) over the spread of the energies
_STEPS = 6.0


def _steps(c):
    if c.get("n_temps"):
        return c["n_temps"] - 1
    return max(1.0, _STEPS * math.sqrt(c["L"] ** 3) * 0.1 / c["eps"] * min(1.0, c["beta_max"]))


def work(case):
    kind = case["kind"]

    def step(L, R, n_sweeps):
        """One temperature step: the spins in and out once (a bit each), 20
        bytes of source slot, energy word and family label per replica."""
        return R * (2 * L ** 3 / 8 + 20), OPS_PER_ATTEMPT * n_sweeps * L ** 3 * R

    if kind == "anneal":
        runs = [(case["L"], case["R"], _steps(case))]
    elif kind == "pair":
        runs = [(case["L"], case["R"], case["n_temps"] - 1)] * 2
    elif kind == "sweep":
        runs = [(case["L"], case["R"], 1)]
    elif kind == "batch":
        runs = [(L, R, case["n_temps"] - 1) for L, R in _batch_sizes(case)] * 2
    elif kind == "serve":
        runs = [(L, R, n - 1) for _, L, R, n in _request_sizes(case)]
    elif kind == "overlap":
        N, R = case["L"] ** 3, case["R"]
        return {"bytes": 4 * R * N / 8, "flops": R * (N + 9.0 * N)}
    else:  # checkpoint: one byte per spin to the host and back, the packed state read and written
        N, R = case["L"] ** 3, case["R"]
        return {"bytes": R * (2 * N + 2 * N / 8 + 16), "flops": 6.0 * R * N}
    total = [sum(n * step(L, R, case["n_sweeps"])[k] for L, R, n in runs) for k in (0, 1)]
    return {"bytes": float(total[0]), "flops": float(total[1])}


# --- the same scalars from a plain 64-bit simulation --------------------------
MASK = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors holding 32-bit words."""
    k0, k1 = key & MASK, key >> 32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((b >> 32) & MASK) ^ c1 ^ k0, b & MASK, ((a >> 32) & MASK) ^ c3 ^ k1,
                          a & MASK)
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1, c2, c3


class _Plain:
    """Population annealing of Sec. II with the documented random numbers: spins
    in checkerboard order (colour 0, then colour 1, each lexicographic), one
    replica per row, FP64 energies."""

    def __init__(self, case, J, seed):
        self.dev = torch.device("cuda")
        self.model = case.get("model", "pm")
        self.L, self.R, self.seed = case["L"], case["R"], seed
        L, N = self.L, self.L ** 3
        self.N = N
        z, y, x = np.meshgrid(*[np.arange(L)] * 3, indexing="ij")
        x, y, z = x.ravel(), y.ravel(), z.ravel()
        site = x + L * (y + L * z)
        colour = (x + y + z) & 1
        cm = colour * (N // 2) + (site >> 1)
        order = np.argsort(cm)

        def at(i, j, k):
            return (i % L) + L * ((j % L) + L * (k % L))

        nb = [at(x + 1, y, z), at(x - 1, y, z), at(x, y + 1, z), at(x, y - 1, z),
              at(x, y, z + 1), at(x, y, z - 1)]
        Jf = np.asarray(J, np.float64) / (16.0 if self.model == "gauss16" else 1.0)
        Js = [Jf[site], Jf[nb[1]], Jf[N + site], Jf[N + nb[3]], Jf[2 * N + site],
              Jf[2 * N + nb[5]]]
        self.nb = torch.tensor(np.stack([cm[b][order] for b in nb]), device=self.dev)
        self.Jn = torch.tensor(np.stack([j[order] for j in Js]), device=self.dev)
        r = torch.arange(self.R, device=self.dev)
        s = torch.empty(self.R, N, dtype=torch.int8, device=self.dev)
        zero = torch.zeros(1, dtype=torch.int64, device=self.dev)
        for g in range(N // 4):
            for q, w in enumerate(_philox(r, zero + g, zero, zero + 0x494E4954, seed)):
                s[:, int(cm[4 * g + q])] = (1 - 2 * (w >> 31)).to(torch.int8)
        self.s, self.fam = s, r
        self.t = self.k = 0
        self.beta = self.sum_lnQ = self.lnQ = self.eps = 0.0
        self._energies()

    def _fields(self, colour):
        """Local fields of the sites of one colour, FP64."""
        h = self.N // 2
        cols = slice(colour * h, colour * h + h)
        f = torch.zeros(self.s.shape[0], h, dtype=torch.float64, device=self.dev)
        for k in range(6):
            f += self.s[:, self.nb[k, cols]].double() * self.Jn[k, cols]
        return f

    def _energies(self):
        E = []
        for b in range(0, self.s.shape[0], 1 << 14):
            whole, self.s = self.s, self.s[b:b + (1 << 14)]
            E.append(-(self.s[:, :self.N // 2].double() * self._fields(0)).sum(1))
            self.s = whole
        self.E = torch.cat(E)

    def sweep(self, beta, n):
        h = self.N // 2
        rows = max(256, (1 << 25) // h)
        whole = self.s
        for b in range(0, whole.shape[0], rows):
            self.s = whole[b:b + rows]
            slot = torch.arange(b, b + self.s.shape[0], device=self.dev)[:, None]
            for t in range(self.t, self.t + n):
                for colour in (0, 1):
                    g = torch.arange(h // 4, device=self.dev)[None, :] + colour * (h // 4)
                    w = _philox(slot, torch.full_like(g, t), g, torch.full_like(g, 0x4D455452),
                                self.seed)
                    word = torch.stack(torch.broadcast_tensors(*w), 2).reshape(slot.shape[0], h)
                    own = self.s[:, colour * h:(colour + 1) * h]
                    dE = 2 * own.double() * self._fields(colour)
                    thr = torch.floor(torch.exp(-beta * dE.clamp(min=0)) * 2.0 ** 32)
                    own.mul_(torch.where(word.double() < thr, -1, 1).to(torch.int8))
        self.s = whole
        self.t += n
        self._energies()

    def _tau(self, db):
        w = torch.exp(-db * (self.E - self.E.min()))
        S = w.sum()
        return self.R * w / S, S

    def _eps(self, db):
        return float((1 - self._tau(db)[0]).clamp(min=0).sum()) / self.R

    def choose(self, eps, beta_max):
        lo, hi = 0.0, beta_max - self.beta
        if self._eps(hi) <= eps:
            return beta_max
        for _ in range(64):
            mid = lo + 0.5 * (hi - lo)
            if self._eps(mid) <= eps:
                lo = mid
            else:
                hi = mid
        return self.beta + lo

    def step(self, beta, n):
        db = beta - self.beta
        tau, S = self._tau(db)
        self.eps = float((1 - tau).clamp(min=0).sum()) / self.R
        self.lnQ = math.log(float(S)) - math.log(len(self.E)) - db * float(self.E.min())
        self.sum_lnQ += self.lnQ
        self.k += 1
        i = torch.arange(len(self.E), device=self.dev)
        zero = torch.zeros_like(i)
        w = _philox(i, zero + self.k, zero, zero + 0x52455341, self.seed)
        u53 = (w[0] << 21) | (w[1] >> 11)
        fl = torch.floor(tau)
        n_i = fl.long() + (u53 < torch.ceil((tau - fl) * 2.0 ** 53).long()).long()
        src = torch.repeat_interleave(i, n_i)
        self.s, self.fam, self.beta = self.s[src], self.fam[src], beta
        self.sweep(beta, n)
        return self.record()

    def record(self):
        eta = torch.bincount(self.fam).double()
        return dict(beta=self.beta, lnQ=self.lnQ,
                    beta_F=-(self.N * math.log(2.0) + self.sum_lnQ),
                    mean_E=float(self.E.mean()), rho_t=float((eta * eta).sum()) / self.R,
                    eps_expected=self.eps, E_lowest=float(self.E.min()))


def _exact_columns(records, rows=None):
    rows = len(records) if rows is None else rows
    out = {f: _front(np.array([o[f] for o in records], np.float64), rows) for f in REAL_FIELDS}
    out.update({f: None for f in COUNT_FIELDS})
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("anneal", "pair", "sweep"):
        return None  # whole numbers, or more work than a plain simulation does in seconds
    passes = 2 if kind == "pair" else 1
    steps = 2 if kind == "sweep" else _steps(case)
    if passes * steps * case["n_sweeps"] * case["L"] ** 3 * case["R"] > 1.5e10:
        return None
    J = _couplings(case.get("model", "pm"), case["L"], 2 * seed + 1)
    seeds = (0x5EED0000 + 2 * seed, 0x5EED0001 + 2 * seed)
    if kind == "sweep":
        p = _Plain(case, J, seeds[0])
        p.sweep(case["beta"], 10)
        p.sweep(case["beta"], case["n_sweeps"])
        return _exact_columns([p.record()])
    betas = pam.linear_schedule(case["beta_max"], case["n_temps"])[1:] if case["n_temps"] else None
    if kind == "pair":
        pops = [_Plain(case, J, x) for x in seeds]
        return {**_exact_columns([p.step(b, case["n_sweeps"]) for b in betas for p in pops]),
                "q": None}
    p = _Plain(case, J, seeds[0])
    records = []
    while p.beta < case["beta_max"]:
        b = betas[len(records)] if betas else p.choose(case["eps"], case["beta_max"])
        records.append(p.step(b, case["n_sweeps"]))
    out = {**_exact_columns(records, _rows(case)), "families": None, "energies": None}
    if case["model"] == "gauss":
        out["energies"] = _front(p.E.cpu().numpy(), _slots(case))
    if case["state"] == "all":
        out["spins"] = None
    return out
