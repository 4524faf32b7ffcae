"""Performance cases of the library: what its users run, through the Python
binding (one C-ABI call per method).

A case is a dict of plain values.  Its "kind" says which program it stands
for:

  run        a simulation that keeps its lattices on the device, calls sweep()
             again and again and reads energies (and overlaps, correlations or
             the whole configuration) in between;
  job        one whole job: lattices from the seed, the schedule, a logged
             run, the final configuration;
  tempering  parallel tempering of a Gaussian sample, EMCS by EMCS;
  pool       the annealing service: jobs of mixed sizes through the
             continuous-batching pool until every one is done.

Sizes, schedules and refresh periods are those of workloads.py, bench.py and
the tests, and sizes between them.  Every output is a whole number (energies,
overlap and correlation sums, spin bits, daemon levels), decided by integer
arithmetic from the seed, so two correct builds agree in every one of them.
Large lattices return what a run logs (energies, daemon energies, overlaps,
correlation sums, each one taken from every site): a program that steps them
does not copy the configuration to the host each time.  The small ones return
the whole configuration.

work() counts what a pass cannot do without: the state of every lattice (a
spin bit, two level bits per daemon, three coupling bits per site) read once
and written once, and, as operations, 16 integer operations per spin update
(six bonds compared and counted, the level added, tested and stored), 15 more
where an update draws a uniform (a quarter of a ten-round Philox call) and 15
per daemon that a refresh draws.
"""
from __future__ import annotations

import numpy as np

from paper_2506_16240_amd import micsa as M
from paper_2506_16240_amd import serve, workloads

ALGOS = {"micsa": M.ALGO_MICSA, "heatbath": M.ALGO_HEATBATH, "walkers": M.ALGO_WALKERS,
         "metropolis": M.ALGO_METROPOLIS}
LAYOUTS = {"byte": (M.LAYOUT_BYTE, M.LANES_SAMPLES), "planes": (M.LAYOUT_BITPLANE, M.LANES_SAMPLES),
           "replica_planes": (M.LAYOUT_BITPLANE, M.LANES_REPLICAS)}

# Sweeps a handle of kind "run" is set up for: longer than the quench's 1e5,
# so that one handle serves every pass.
RUN_SWEEPS = 2_000_000


def _run(name, L, S, R, sweeps, calls=1, algo="micsa", layout="byte", gamma=1, T=0.7, period=10, read="energy"):
    Lx, Ly, Lz = (L, L, L) if isinstance(L, int) else L
    case = {"kind": "run", "Lx": Lx, "Ly": Ly, "Lz": Lz, "S": S, "R": R, "sweeps": sweeps, "calls": calls,
            "algo": algo, "layout": layout, "gamma": gamma, "T": T, "period": period, "read": read}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest call there is: an interactive session steps one 8^3
        # lattice and looks at it (latency and launches)
        _run("call_8", 8, 1, 1, 10, T=1.5, read="state"),
        # the 16^3 paramagnet at full length: created, 1000 sweeps with the
        # energies logged at every sweep, final configuration read
        {"name": "paramagnet_16", "kind": "job", "Lx": 16, "Ly": 16, "Lz": 16, "S": 1, "R": 1, "algo": "micsa",
         "layout": "byte", "T0": 1.5, "T1": 1.5, "sweeps": 1000, "stride": 1, "period": 10},
        # many replicas of one 32^3 sample in the byte layout, as the service
        # and the overlap studies run them
        _run("replicas_32", 32, 1, 64, 100, read="overlap"),
        # the batched configuration: 256 samples x 2 replicas of 32^3 in bit planes
        _run("planes_32", 32, 256, 2, 200, layout="planes", T=0.8, read="overlap"),
        # the 64^3 quench: energy, overlap and the correlation function against time
        _run("quench_64", 64, 1, 2, 500, calls=2, read="c4"),
        # its heat-bath comparison run
        _run("heatbath_64", 64, 1, 2, 100, algo="heatbath", read="overlap"),
        # a ragged lattice no tuned shape fits, two samples x two replicas
        _run("ragged_104", (104, 90, 70), 2, 2, 60, T=1.1),
        # the paper's main dynamics: six walkers per site, L = 160
        _run("walkers6_160", 160, 1, 1, 60, algo="walkers", gamma=6),
        # the large anneal's sweeps (512^3, refresh every 20)
        _run("anneal_512", 512, 1, 1, 100, T=1.0, period=20),
        # the random-number-greedy baseline on a large lattice
        _run("metropolis_256", 256, 1, 1, 20, algo="metropolis", T=1.1),
        # parallel tempering: 200 runs x 2 replicas x 40 temperatures of a 10^3
        # Gaussian sample with walkers and Houdayer moves
        {"name": "tempering_10", "kind": "tempering", "Lx": 10, "Ly": 10, "Lz": 10, "runs": 200, "M": 40,
         "sweeps": 10, "emcs": 4, "algo": "walkers", "houdayer": True},
        # the service: 16 jobs of mixed size and replica count, all queued
        {"name": "pool_16", "kind": "pool", "jobs": 16, "mix": 11, "sweeps": 400, "per_step": 100},
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return lo * (hi / lo) ** rng.random()

    def side(lo, hi, step):
        return max(step, int(round(log_uniform(lo, hi) / step)) * step)

    kind = rng.choice(["run"] * 9 + ["job", "tempering", "pool"])
    if kind == "tempering":
        L = rng.choice([4, 6, 8, 10, 12])
        return {"kind": "tempering", "Lx": L, "Ly": L, "Lz": rng.choice([L, L + 2]),
                "runs": int(log_uniform(2, 120)), "M": rng.randint(6, 40), "sweeps": rng.choice([5, 10]),
                "emcs": rng.randint(1, 4), "algo": rng.choice(["walkers", "metropolis"]),
                "houdayer": rng.random() < 0.7}
    if kind == "pool":
        return {"kind": "pool", "jobs": rng.randint(2, 8), "mix": rng.randint(0, 10 ** 6),
                "sweeps": rng.choice([100, 150, 200]), "per_step": rng.choice([50, 100])}
    if kind == "job":
        return {"kind": "job", "Lx": side(8, 40, 8), "Ly": side(6, 40, 2), "Lz": side(6, 40, 2),
                "S": rng.randint(1, 4), "R": rng.randint(1, 8), "algo": rng.choice(["micsa", "micsa", "heatbath"]),
                "layout": "byte", "T0": 3.0, "T1": round(rng.uniform(0.2, 1.2), 2),
                "sweeps": rng.randint(100, 400), "stride": rng.choice([1, 5, 20]), "period": rng.choice([5, 10, 20])}
    layout = rng.choice(["byte"] * 6 + ["planes", "replica_planes"])
    T, period = round(rng.uniform(0.4, 2.0), 2), rng.choice([5, 10, 10, 20, M.REFRESH_LOG2])
    if layout != "byte":
        dims = (side(8, 64, 8), side(8, 64, 2), side(8, 64, 2))
        S, R = (rng.randint(20, 260), rng.randint(1, 2)) if layout == "planes" else (1, rng.randint(16, 64))
        algo, gamma = "micsa", 1
    else:
        dims = (side(8, 400, 8), side(8, 400, 2), side(8, 400, 2))
        S, R = (1, rng.choice([1, 1, 2, 4, 16])) if dims[0] * dims[1] * dims[2] < 1e6 else (1, rng.choice([1, 1, 2]))
        algo = rng.choice(["micsa", "micsa", "micsa", "walkers", "heatbath", "metropolis"])
        gamma = rng.choice([1, 2, 6]) if algo == "walkers" else 1
    N = dims[0] * dims[1] * dims[2]
    # about 1e8 updates where each draws a uniform or moves its walker, 3e8 where not
    budget = (3e8 if algo == "micsa" else 1e8) / (N * S * R)
    sweeps = max(4, min(int(budget), rng.randint(20, 300)))
    small = N * S * R < 20_000
    read = rng.choice((["overlap", "c4"] if R > 1 and S * R < 20 else ["energy"]) + ["energy"]
                      + (["state"] if small else []))
    return _run(None, dims, S, R, sweeps, algo=algo, layout=layout, gamma=gamma, T=T, period=period, read=read)


def _open(case, seed, n_sweeps, T0, T1, kind):
    layout, lanes = LAYOUTS[case["layout"]]
    lat = M.Lattice(case["Lx"], case["Ly"], case["Lz"], case["S"], case["R"], seed, layout=layout, lane_mode=lanes,
                    gamma=case.get("gamma", 1))
    lat.set_schedule(M.Schedule(kind, T0, T1, n_sweeps, case["period"]))
    return lat


def prepare(case, seed):
    seed = serve.splitmix64(seed)
    if case["kind"] == "run":
        return {"case": case, "lat": _open(case, seed, RUN_SWEEPS, case["T"], case["T"], M.SCHED_CONST)}
    if case["kind"] == "tempering":
        J = workloads.gaussian_couplings(case["Lx"], case["Ly"], case["Lz"], seed & 0xFFFFFFFF)
        algo = M.PT_WALKERS if case["algo"] == "walkers" else M.PT_METROPOLIS
        pt = M.PT(case["Lx"], case["Ly"], case["Lz"], case["runs"], np.linspace(0.2, 2.0, case["M"]), J, seed,
                  case["sweeps"], algo, case["houdayer"])
        return {"case": case, "pt": pt}
    if case["kind"] == "pool":
        # the mix of sizes belongs to the case, the instances to the seed
        specs = [spec for _, spec in serve.job_stream(case["jobs"], 1.0, case["mix"], case["sweeps"])]
        return {"case": case, "stream": [(0.0, serve.JobSpec(s.L, s.R, s.seed ^ seed, n_sweeps=s.n_sweeps))
                                         for s in specs]}
    return {"case": case, "seed": seed}


def _read(lat, read):
    out = {"E": lat.energy(), "D": lat.daemon_energy()}
    if read in ("overlap", "c4"):
        out["q"] = lat.overlap(0, 1)
    if read == "c4":
        out["c4"] = lat.c4_sums()
    if read == "state":
        out["spins"], out["daemons"] = lat.spins(), lat.daemons()
    return out


def run(state):
    case = state["case"]
    if case["kind"] == "run":
        lat, algo, out = state["lat"], ALGOS[case["algo"]], []
        for _ in range(case["calls"]):
            lat.sweep(algo, case["sweeps"])
            out.append(_read(lat, case["read"]))
        return out
    if case["kind"] == "tempering":
        pt = state["pt"]
        pt.step(case["emcs"])
        return pt.read()
    if case["kind"] == "pool":
        results, _ = serve.serve(state["stream"], 64 << 30, case["per_step"])
        return [r.energies for r in results]
    lat = _open(case, state["seed"], case["sweeps"], case["T0"], case["T1"], M.SCHED_LINEAR)
    E, D = lat.sweep_logged(ALGOS[case["algo"]], case["sweeps"], case["stride"])
    out = {"E": E, "D": D, "spins": lat.spins(), "daemons": lat.daemons()}
    lat.close()
    return out


def _sweep_work(N, lattices, couplings, gamma, algo, sweeps, period):
    """(bytes, operations) of `sweeps` sweeps; `couplings`: lattices' worth of coupling bits."""
    state = N * lattices * (1 + 2 * gamma) / 8
    steps = -(-sweeps // gamma)
    refreshes = steps / period if period else np.log2(steps + 1)
    drawn = gamma * N * lattices * refreshes if algo in ("micsa", "walkers") else 0
    per_update = 16 if algo in ("micsa", "walkers") else 31
    return 2 * state + 3 * N * couplings / 8, per_update * N * lattices * sweeps + 15 * drawn


def work(case):
    if case["kind"] == "tempering":
        N = case["Lx"] * case["Ly"] * case["Lz"]
        clones = case["runs"] * 2 * case["M"]
        updates = N * clones * case["sweeps"] * case["emcs"]
        draws = N * clones * case["emcs"] * (1 if case["algo"] == "walkers" else case["sweeps"])
        return {"bytes": 2 * N * clones / 8 + 12 * N, "flops": 16 * updates + 60 * draws}
    if case["kind"] == "pool":
        total = np.zeros(2)
        for _, s in serve.job_stream(case["jobs"], 1.0, case["mix"], case["sweeps"]):
            total += _sweep_work(s.L ** 3, s.R, 1, 1, "micsa", s.n_sweeps, s.period)
        return {"bytes": float(total[0]), "flops": float(total[1])}
    N = case["Lx"] * case["Ly"] * case["Lz"]
    b, f = _sweep_work(N, case["S"] * case["R"], case["S"], case.get("gamma", 1), case["algo"],
                       case["sweeps"] * case.get("calls", 1), case["period"])
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """Every output is a whole number; none has a 64-bit floating value to be compared with."""
    return None
