"""The work that users of this framework have it do, as measurable cases.

Four kinds, all through paper_1403_4560_amd.binding.Ensemble:
  sweep   a run's steady state: sweep_pt(sweeps) with a measurement every 10
          sweeps, then the accumulators and counters read by measure();
  bin     one bin of the Table I driver (driver.run_log_binned): reset the
          accumulators, sweep, measure, disorder averages with jackknife
          errors;
  errors  disorder averages and jackknife errors of accumulators that another
          run left (finalize_jackknife alone);
  resume  continue from a checkpoint and write the next one: write_state, a
          few sweeps, read_state.
"""
import math

import numpy as np
import torch

from paper_1403_4560_amd import binding
from paper_1403_4560_amd import workload as W

EVERY = 10                    # sweeps between measurements, as in every run of this repository
BETA_TABLE1 = (0.1, 1.8)      # Table I's ladder
MIXED = (6, 8, 10, 12)        # the uneven batch's lattice sizes
# algorithmic operations of one spin-flip attempt: Gaussian couplings, four sites a word; +-1 couplings, one bit a spin
OPS = {"gauss": 28.75, "pm1": 14.83}


def _case(name, kind, L, samples, temps, sweeps, J="gauss", h=0.1, tune=False):
    c = dict(kind=kind, L=L, samples=samples, temps=temps, sweeps=sweeps, J=J, h=h, tune=tune)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest workload of workload.CONFIGS: 32 tiny chains, a run that latency decides
        _case("gauss_L4", "sweep", 4, 16, 8, 200, h=0.3),
        # workload.CONFIGS["L8_gauss"]
        _case("gauss_L8", "sweep", 8, 1024, 16, 200, h=0.2, tune=True),
        # workload.CONFIGS["L16_gauss"], the benchmark's shape, a quarter of its samples (four chains for each compute unit)
        _case("gauss_L16", "sweep", 16, 512, 24, 100, tune=True),
        # workload.CONFIGS["mixed_L6_12"], a quarter of its samples: sizes and fields of one batch differ (L = 0: MIXED in turn)
        _case("gauss_mixed", "sweep", 0, 1024, 16, 200, tune=True),
        # a size, a ladder and a sample count that nothing divides: the general code of the LDS engines
        _case("gauss_L14_odd", "sweep", 14, 37, 21, 50, h=0.25),
        # workload.CONFIGS["L32_pm1"] with one chain for each compute unit
        _case("pm1_L32", "sweep", 32, 128, 32, 100, J="pm1", h=0.4, tune=True),
        # chains that do not fit LDS: the HBM-resident tier
        _case("gauss_L24", "sweep", 24, 8, 16, 50),
        # the driver as a user starts it: 64 samples (its default) of the smallest lattice of Table I, 56 temperatures
        _case("table1_L6", "bin", 6, 64, 56, 128, J="pm1"),
        _case("table1_L8", "bin", 8, 128, 56, 128, J="pm1"),
        # the largest lattice of Table I with the sample count of the driver's own example
        _case("table1_L10", "bin", 10, 256, 56, 128, J="pm1"),
        # the errors of a finished pool of samples
        _case("errors_2048", "errors", 6, 2048, 24, 0, J="pm1"),
        # a checkpoint of the benchmark's shape
        _case("resume_L16", "resume", 16, 64, 24, 10),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: a kind, a lattice size and coupling kind that the kind is used with, a ladder length (odd ones too)
    and a sample count over its whole range, of no more attempts than the largest listed case of its kind."""
    kind = rng.choice(["sweep", "sweep", "sweep", "sweep", "bin", "bin", "errors", "resume"])
    h = round(rng.choice([-1, 1]) * rng.uniform(0.02, 0.6), 3)
    if kind == "errors":
        return _case("", kind, rng.choice([4, 6, 8]), _log_int(rng, 2, 2000), rng.randint(1, 24), 0, J="pm1", h=h)
    if kind == "bin":
        L, temps = rng.choice([6, 8, 10]), rng.choice([56, 56, rng.randint(12, 64)])
        return _case("", kind, L, _log_int(rng, 2, 256), temps, rng.choice([40, 64, 100, 128]), J="pm1", h=h)
    if kind == "resume":
        L, temps = rng.choice([8, 10, 12, 14, 16]), rng.randint(5, 24)
        cap = max(1, int(6e6 / (2 * temps * L ** 3)))
        return _case("", kind, L, _log_int(rng, 1, cap), temps, 10, J=rng.choice(["gauss", "pm1"]), h=h)
    J, L = rng.choice([("gauss", 4), ("gauss", 6), ("gauss", 8), ("gauss", 10), ("gauss", 12), ("gauss", 14), ("gauss", 16), ("gauss", 16),
                       ("gauss", 0), ("gauss", 24), ("pm1", 6), ("pm1", 12), ("pm1", 16), ("pm1", 32)])
    temps = rng.randint(5, 32 if L < 14 else 24)
    sites = L ** 3 if L else sum(x ** 3 for x in MIXED) / 4
    sweeps = rng.choice([20, 50, 100]) if L < 24 else 30
    cap = {24: 8, 32: 64}.get(L, min(1024, int(5e9 / (sites * 2 * temps * sweeps))))
    return _case("", kind, L, _log_int(rng, 1, cap), temps, sweeps, J=J, h=h, tune=L == 0)


def _sizes(case):
    n = case["samples"]
    return [MIXED[s % 4] for s in range(n)] if case["L"] == 0 else [case["L"]] * n


def _work_of(case, seed):
    """A batch as workload.make_workload draws it (couplings on the 2^-18 grid or +-1, hot start), from one stream."""
    rng = np.random.Generator(np.random.PCG64(int(seed) + 77))
    Ls = np.array(_sizes(case), dtype=np.int32)
    S, nT = len(Ls), case["temps"]
    N = Ls.astype(np.int64) ** 3
    bonds, spins = int(3 * N.sum()), int((2 * nT * N).sum())
    if case["J"] == "gauss":
        u = np.clip(np.rint(rng.standard_normal(bonds) / W.GRID), -W.JMAX_UNITS, W.JMAX_UNITS)
        J, jkind = (u * W.GRID).astype(np.float32), W.J_GAUSS
        ladder = W.geometric_betas(nT, 0.4, 1.6)
    else:
        J, jkind = _signs(rng, bonds), W.J_PM1
        ladder = W.beta_ladder(nT, *BETA_TABLE1)
    h = np.full(S, case["h"], dtype=np.float32)
    if case["L"] == 0:
        h = np.array([(0.1, 0.2, 0.3)[(s // 4) % 3] for s in range(S)], dtype=np.float32)
    return W.Workload(L=Ls, n_temps=np.full(S, nT, dtype=np.int32), h=h, sample_id=np.arange(S, dtype=np.uint32), jkind=jkind,
                      seed=int(seed) + 1, measure_every=EVERY, measure_start=0, beta=np.tile(ladder, S), J=J, spins0=_signs(rng, spins))


def _signs(rng, n):
    return (np.unpackbits(np.frombuffer(rng.bytes((n + 7) // 8), dtype=np.uint8), count=n) * np.uint8(2) - np.uint8(1)).view(np.int8)


def _accumulators(case, seed):
    """What 1000 measurements leave: sums of moments of a positive overlap and of the Fourier components, energies."""
    rng = np.random.Generator(np.random.PCG64(int(seed) + 78))
    S, nT, n = case["samples"], case["temps"], 1000.0
    cold = np.linspace(0.1, 1.0, nT)[None, :]
    q = 0.6 * cold * (1.0 + 0.2 * rng.standard_normal((S, nT)))
    v = 0.04 * cold * rng.uniform(0.8, 1.2, (S, nT))
    acc = np.empty((S, nT, binding.NACC))
    acc[:, :, 0] = n
    acc[:, :, 1] = q * n
    acc[:, :, 2] = (q * q + v) * n
    acc[:, :, 3] = (q ** 3 + 3 * q * v) * n
    acc[:, :, 4] = (q ** 4 + 6 * q * q * v + 3 * v * v) * n
    for f in range(9):
        acc[:, :, 5 + 3 * f] = 0.002 * rng.standard_normal((S, nT)) * n
        acc[:, :, 6 + 3 * f] = 0.002 * rng.standard_normal((S, nT)) * n
        acc[:, :, 7 + 3 * f] = (0.3 if f < 3 else 0.15) * v * rng.uniform(0.7, 1.3, (S, nT)) * n
    E = -1.5 * case["L"] ** 3 * cold
    for k in (32, 34):
        e = E * (1.0 + 0.05 * rng.standard_normal((S, nT)))
        acc[:, :, k], acc[:, :, k + 1] = e * n, (e * e + 3.0) * n
    return acc


def prepare(case, seed):
    torch.cuda.set_device(0)
    work = _work_of(case, seed)
    ens = binding.Ensemble(work, stream=torch.cuda.current_stream().cuda_stream)
    if case["tune"]:
        ens.autotune(trial_sweeps=4)
    state = {"kind": case["kind"], "ens": ens, "sweeps": case["sweeps"]}
    if case["kind"] == "errors":
        ens.load_accumulators(acc=list(_accumulators(case, seed)))
    if case["kind"] == "resume":
        ens.sweep_pt(5)
        state["checkpoint"] = ens.read_state()
    return state


def _whole(arrays):
    return np.concatenate([a.ravel() for a in arrays])


def run(state):
    ens, kind = state["ens"], state["kind"]
    if kind == "resume":
        at = state["checkpoint"]
        ens.write_state(at["spins"], at["sweep"], at["walker_at_slot"])
        ens.sweep_pt(state["sweeps"])
        new = ens.read_state()
        return [_whole(new["spins"]), _whole(new["walker_at_slot"]), _whole(new["E"])]
    out = []
    if kind != "errors":
        if kind == "bin":
            ens.reset_accumulators()
        ens.sweep_pt(state["sweeps"])
        m = ens.measure()
        out = [_whole(m["acc"]), _whole(m["flips"]), _whole(m["swaps"])]
    if kind != "sweep":
        obs = ens.finalize_jackknife()
        out += [np.stack([obs[k][0] for k in binding.OBS_NAMES]), np.stack([obs[k][1] for k in binding.OBS_NAMES])]
    return out


def work(case):
    nT, Ls = case["temps"], _sizes(case)
    slots = nT * len(Ls)
    sites = sum(L ** 3 for L in Ls)
    acc = 8.0 * binding.NACC * slots
    if case["kind"] == "errors":  # thermal means, leave-one-out means, observables and their spread, for each sample and slot
        return {"bytes": acc + 2 * 8 * 11 * nT, "flops": 230.0 * slots}
    attempts = 2.0 * nT * sites * case["sweeps"]
    spins = 2.0 * nT * sites
    bonds = 3.0 * sites * (4 if case["J"] == "gauss" else 1)
    counters = 2 * 2 * 8.0 * slots
    flops = attempts * OPS[case["J"]]
    if case["kind"] == "resume":
        return {"bytes": 2 * spins + bonds + 24.0 * 2 * slots, "flops": flops}
    return {"bytes": 2 * spins + bonds + 2 * acc + 2 * counters, "flops": flops + (230.0 * slots if case["kind"] == "bin" else 0.0)}


def exact(case, seed):
    """Averages and errors of given accumulators, in numpy's extended precision, rounded to 64 bits at the end.  The other
    kinds return a trajectory of accept and reject decisions and sums over it, which no higher precision defines."""
    if case["kind"] != "errors":
        return None
    acc = _accumulators(case, seed).astype(np.longdouble)
    S, L = case["samples"], case["L"]
    m = acc / acc[:, :, :1]
    total = m.sum(axis=0)
    mean = _observables(total / S, L)
    rep = _observables((total[None] - m) / (S - 1), L)
    centre = rep.mean(axis=1, keepdims=True)
    err = np.sqrt(((rep - centre) ** 2).sum(axis=1) * (np.longdouble(S - 1) / S))
    count = np.full((1, case["temps"]), float(S))
    return [np.concatenate([mean.astype(np.float64), count]), np.concatenate([err.astype(np.float64), 0.0 * count])]


def _observables(D, L):
    """Rows of binding.OBS_NAMES (the count aside) from disorder averages D [..., temps, 36]."""
    N = np.longdouble(L) ** 3
    q1, q2, q3, q4 = (D[..., k] for k in (1, 2, 3, 4))
    c2 = q2 - q1 * q1
    c4 = q4 - 4 * q1 * q3 + 6 * q1 ** 2 * q2 - 3 * q1 ** 4
    chi = [N * (D[..., 7 + 3 * f] - D[..., 5 + 3 * f] ** 2 - D[..., 6 + 3 * f] ** 2) for f in range(9)]
    chi0, k1, k2 = N * c2, sum(chi[:3]) / 3, sum(chi[3:]) / 6
    xi = np.sqrt(chi0 / k1 - 1) / (2 * np.sin(np.longdouble(math.pi) / L))
    return np.stack([q1, chi0, k1, k2, (3 - c4 / c2 ** 2) / 2, xi, k1 / k2, chi0 / k1, D[..., 32], D[..., 34]])
