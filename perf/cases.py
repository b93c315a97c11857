"""The work a user of this library has it do, as measurable cases.

A case is a plain dict.  Its "kind" is how a program drives the library:

* "run": one lattice advanced by spkmc_run, then its observables (and, where the
  run recorded, its records) read and its spins left in the state buffer;
* "restart": spins set from host memory, a run, the spins read back to the host;
* "batch": lattices of a replica study advanced together by run_batch, packed
  into launches by the planner;
* "serve": requests queued on a Server and stepped until all are done.

Sizes are those of the repository's workloads, tests and benchmark, and generic
ones of the same ranges.
"""
import math
import random

import numpy as np
import torch

from paper_1005_4713_amd import spkmc, tune

T_C = 4.5115
MIX_L = (32, 48, 64, 96, 128, 192, 256)


def _run(name, L, domain, layout, cycles, obs_every=0, variant="", rates="glauber", init="random", T=T_C, H=0.0):
    return dict(name=name, kind="run", L=L, domain=domain, layout=layout, cycles=cycles, obs_every=obs_every,
                variant=variant, rates=rates, init=init, T=T, H=H)


def listed():
    return [
        # the smallest call: one cycle of a small packed lattice and its observables
        # (an interactive or coupled program that looks at every cycle)
        _run("l32_one_cycle", 32, 16, "packed", 1),
        # the small int8 configuration in full, every cycle recorded
        _run("l16_int8_every_cycle", 16, 8, "int8", 1000, obs_every=1),
        # the statistics study's step: 256 recorded cycles of the medium int8 lattice
        _run("l128_int8_statistics", 128, 8, "int8", 256, obs_every=1),
        # the bias study's finest subcells (64 sites), two colours, an odd number of
        # domains along each edge, all +1 start
        _run("l72_two_colours_fine", 72, 8, "packed", 400, obs_every=4, variant="two_colours", init="up"),
        # one configuration of the critical sweep at 512^3 (512 sites per octant)
        _run("l512_sweep", 512, 16, "packed", 500, obs_every=10, rates="metropolis", init="up"),
        # the headline benchmark: 1024^3 at T_c, a record every 10 cycles
        _run("l1024_headline", 1024, 32, "packed", 500, obs_every=10),
        # the paper's own two-colour decomposition at 1024^3
        _run("l1024_two_colours", 1024, 32, "packed", 100, variant="two_colours"),
        # the literal reading of step 2: R_max over every octant
        _run("l1024_rmax_all", 1024, 32, "packed", 100, variant="rmax_all"),
        # more domains than one resident launch holds
        _run("l2048_large", 2048, 32, "packed", 20, obs_every=10),
        # spins from another program, a short run, spins back to it; octant edge 12
        dict(name="l240_restart", kind="restart", L=240, domain=24, layout="packed", cycles=10, variant="",
             rates="glauber", T=T_C, H=0.05),
        # a replica study: temperatures around T_c, fields 0 and +-0.05, mixed sizes
        dict(name="replica_batch", kind="batch", lattices=48, mix=5, policy=16, passes=2, cycles=500),
        # the same mix as requests that arrive together: admission and short jobs
        dict(name="replica_served", kind="serve", requests=64, mix=5, domain=16, cycles=200, macro_cycles=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the ranges above."""
    kind = rng.choice(("packed", "packed", "large", "int8", "fine", "restart", "batch", "serve"))
    T, H = round(rng.uniform(4.0, 5.0), 4), rng.choice((0.0, 0.05, -0.05))
    rates, init = rng.choice(("glauber", "metropolis")), rng.choice(("random", "random", "up"))
    obs = rng.choice((0, 0, 1, 4, 10))
    if kind == "packed":  # the persistent kernels' sizes, every variant
        domain = rng.choice((16, 32))
        nd = _log_int(rng, 1 if domain == 32 else 2, 16)
        c = _run("", nd * domain, domain, "packed", _log_int(rng, 1, 600), obs,
                 rng.choice(("", "", "two_colours", "rmax_bound", "rmax_all")), rates, init, T, H)
    elif kind == "large":
        domain = rng.choice((16, 32, 32))
        nd = _log_int(rng, 17, 33 if domain == 16 else 44)
        c = _run("", nd * domain, domain, "packed", _log_int(rng, 10, 100), obs,
                 "" if domain == 16 else rng.choice(("", "", "two_colours", "rmax_bound")), rates, init, T, H)
    elif kind == "int8":  # octant edges 1 .. 16, odd ones among them
        h = rng.randint(1, 16)
        nd = max(1, _log_int(rng, 12, 130) // (2 * h))
        c = _run("", 2 * h * nd, 2 * h, "int8", _log_int(rng, 1, 300), obs, rng.choice(("", "", "two_colours")), rates,
                 init, T, H)
    elif kind == "fine":  # packed octants the row kernels do not take
        h = rng.choice((4, 4, 12, 20))
        nd = max(1, _log_int(rng, 16, 160) // (2 * h))
        c = _run("", 2 * h * nd, 2 * h, "packed", _log_int(rng, 1, 300), obs, rng.choice(("", "two_colours")), rates,
                 init, T, H)
    elif kind == "restart":
        h = rng.choice((3, 4, 5, 8, 12, 16))
        nd = max(1, _log_int(rng, 16, 240) // (2 * h))
        c = dict(kind="restart", L=2 * h * nd, domain=2 * h, layout="packed" if h % 4 == 0 and rng.random() < 0.7 else "int8",
                 cycles=_log_int(rng, 1, 20), variant="", rates=rates, T=T, H=H)
    elif kind == "batch":
        c = dict(kind="batch", lattices=_log_int(rng, 2, 56), mix=rng.randint(10, 10 ** 6), policy=rng.choice((16, 16, 32)),
                 passes=rng.choice((1, 2)), cycles=_log_int(rng, 10, 500))
    else:
        c = dict(kind="serve", requests=_log_int(rng, 2, 64), mix=rng.randint(10, 10 ** 6), domain=16,
                 cycles=_log_int(rng, 10, 200), macro_cycles=rng.choice((50, 100)))
    c.pop("name", None)
    return c


def _mix(n, mix, seed):
    """n lattices of the replica mix: sizes and parameters from `mix`, streams from `seed`."""
    g = np.random.Generator(np.random.Philox(mix))
    out = []
    for i in range(n):
        L, T, H = int(g.choice(MIX_L)), float(g.uniform(4.0, 5.0)), float(g.choice([0.0, 0.05, -0.05]))
        out.append(dict(L=L, J=1.0, H=H, T=T, seed=(seed << 16) + 1000 + i))
    return out


def _spins_in(sim):
    """The spins where the state buffer holds them (bits octant-major, or bytes), as a view."""
    info, align = sim.info(), lambda v: (v + 255) // 256 * 256
    n = info["N"] if info["layout"] == spkmc.LAYOUTS["int8"] else info["N"] // 8
    tail = align(n)
    if info["layout"] == spkmc.LAYOUTS["packed"]:
        tail += align(info["K"] * 8 * 6 * info["h"] ** 2 // 8)
    start = info["state_bytes"] - tail
    return sim.buf[start:start + n]


def _sim(case, seed):
    return spkmc.Sim(case["L"], case["domain"], layout=case["layout"], T=case["T"], H=case["H"], rates=case["rates"],
                     init=case.get("init", "up"), variant=case["variant"], seed=seed,
                     record_cap=max(case["cycles"], 1) if case.get("obs_every") else 0)


def _host_spins(case, seed):
    """Spins as another program hands them over: a partly magnetised lattice."""
    g = np.random.Generator(np.random.Philox(seed))
    return np.where(g.random(case["L"] ** 3, dtype=np.float32) < 0.55, 1, -1).astype(np.int8)


def prepare(case, seed):
    if case["kind"] == "run":
        sim = _sim(case, seed)
        return dict(case=case, sim=sim, spins=_spins_in(sim))
    if case["kind"] == "restart":
        return dict(case=case, sim=_sim(case, seed), host=_host_spins(case, seed))
    if case["kind"] == "batch":
        specs = _mix(case["lattices"], case["mix"], seed)
        plan = tune.make_plan(specs, case["policy"], {8: case["passes"], 16: case["passes"]}, tune.capacity())
        sims = tune.build(specs, plan["domains"])
        return dict(case=case, plan=plan, sims=sims, spins=[_spins_in(s) for s in sims])
    specs = _mix(case["requests"], case["mix"], seed)
    foot = sum((spkmc.state_bytes(spkmc.make_params(s["L"], case["domain"])) + 255) // 256 * 256 for s in specs)
    return dict(case=case, specs=specs, server=spkmc.Server(foot, macro_cycles=case["macro_cycles"], max_live=512))


def _states(states):
    """State or record tuples (cycle, fired, nulls, t, M, B) as integers and times."""
    a = np.array([(s[0], s[1], s[2], s[4], s[5]) for s in states], dtype=np.int64).reshape(-1, 5)
    return a, np.array([s[3] for s in states], dtype=np.float64)


def run(state):
    case = state["case"]
    if case["kind"] == "run":
        sim = state["sim"]
        sim.run(case["cycles"], case["obs_every"])
        counts, t = _states([sim.state()])
        out = dict(counts=counts, t=t, spins=state["spins"])
        if case["obs_every"]:
            out["record_counts"], out["record_t"] = _states(sim.records(case["cycles"] // case["obs_every"]))
        return out
    if case["kind"] == "restart":
        sim = state["sim"]
        sim.set_spins(state["host"])
        sim.run(case["cycles"])
        counts, t = _states([sim.state()])
        return dict(counts=counts, t=t, spins=sim.spins())
    if case["kind"] == "batch":
        tune.run_plan(state["plan"], state["sims"], case["cycles"])
        counts, t = _states([s.state() for s in state["sims"]])
        return dict(counts=counts, t=t, spins=state["spins"])
    srv, specs = state["server"], state["specs"]
    ids = [srv.submit(s["L"], case["domain"], case["cycles"], T=s["T"], H=s["H"], seed=s["seed"], record_cap=0,
                      keep=i == 0) for i, s in enumerate(specs)]
    srv.drain()
    counts, t = _states([srv.poll(r)["state_tuple"] for r in ids])
    spins = srv.lattice(ids[0], specs[0]["L"]).spins()
    for r in ids:
        srv.release(r)
    return dict(counts=counts, t=t, spins=spins)


def _line_work(L, domain, layout, lpd, cycles):
    """(bytes, operations) of the cycles of one lattice: every active octant and its
    one-site halo read once and one flip written, and the 14 products and sums of
    its frequency line."""
    lines, h = (L // domain) ** 3 * lpd, domain // 2
    sites = h ** 3 + 6 * h ** 2
    return cycles * lines * (sites / 8 + 8 if layout == "packed" else sites + 2), cycles * lines * 28


def work(case):
    if case["kind"] in ("run", "restart"):
        lpd = 4 if "two_colours" in case["variant"] else 1
        b, f = _line_work(case["L"], case["domain"], case["layout"], lpd, case["cycles"])
        if case["kind"] == "restart":
            b += case["L"] ** 3 * (2 + 2 / 8 if case["layout"] == "packed" else 4)
        elif case["obs_every"]:
            b += 48 * (case["cycles"] // case["obs_every"])
        return dict(bytes=b, flops=f)
    n = case["lattices"] if case["kind"] == "batch" else case["requests"]
    specs = _mix(n, case["mix"], 1)
    doms = [case["domain"]] * n if case["kind"] == "serve" else \
        [32 if case["policy"] == 32 and s["L"] % 32 == 0 else 16 for s in specs]
    b = f = 0.0
    for s, d in zip(specs, doms):
        x, y = _line_work(s["L"], d, "packed", 1, case["cycles"])
        b, f = b + x, f + y
        if case["kind"] == "serve":
            b += s["L"] ** 3 / 8  # the initial spins written
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------------------
# The method in plain numpy (64 bits), for the simulated times
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, key):
    m, lo = np.uint64(0xFFFFFFFF), np.uint64(32)
    c = [np.atleast_1d(np.asarray(v, dtype=np.uint64)) for v in (c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> lo) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> lo) ^ c[3] ^ np.uint64(k1), p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _times(case, seed, host=None):
    """The simulated time after every cycle."""
    L, d, h = case["L"], case["domain"], case["domain"] // 2
    nd, two = L // d, "two_colours" in case["variant"]
    if host is not None:
        up = host.reshape(L, L, L) > 0
    elif case["init"] == "up":
        up = np.ones((L, L, L), dtype=bool)
    else:
        words = np.stack(_philox(np.arange((L ** 3 + 127) // 128), 0, 0xFFFFFFFE, 0xFFFFFFFE, seed), axis=1)
        bits = (words.reshape(-1, 1) >> np.arange(32, dtype=np.uint64)) & np.uint64(1)
        up = bits.reshape(-1)[:L ** 3].astype(bool).reshape(L, L, L)
    up = up.copy()
    nup = sum(np.roll(up, s, a).astype(np.int8) for a in range(3) for s in (1, -1))
    beta, rates = 1.0 / case["T"], np.empty(14)
    for c in range(14):
        x = beta * (2.0 * (2 * (c % 7) - 6) + 2.0 * case["H"] * (1 if c >= 7 else -1))
        rates[c] = 1.0 / (1.0 + math.exp(x)) if case["rates"] == "glauber" else min(1.0, math.exp(-x))
    blocks = (nd, 2, h, nd, 2, h, nd, 2, h)
    kz, ky, kx = (v.reshape(-1) for v in np.meshgrid(*[np.arange(nd)] * 3, indexing="ij"))
    K, t, out = nd ** 3, 0.0, []

    def frequency(o):  # classes (line, site) and running sums of octant o of every domain
        sl = (slice(None), o >> 2 & 1, slice(None), slice(None), o >> 1 & 1, slice(None), slice(None), o & 1, slice(None))
        u, n = (a.reshape(blocks)[sl].transpose(0, 2, 4, 1, 3, 5).reshape(K, -1) for a in (up, nup))
        cls = np.where(u, 7 + n, 6 - n).astype(np.int64)
        cnt = np.bincount((cls + 14 * np.arange(K)[:, None]).reshape(-1), minlength=14 * K).reshape(K, 14)
        return cls, cnt, np.cumsum(cnt * rates, axis=1)

    for n in range(case["cycles"]):
        w = [int(v[0]) for v in _philox(n, 0, 0xFFFFFFFF, 0xFFFFFFFF, seed)]
        colour = w[0] >> (31 if two else 29)
        octs = [o for o in range(8) if bin(o).count("1") & 1 == colour] if two else [colour]
        lines = {o: frequency(o) for o in (range(8) if "rmax_all" in case["variant"] else octs)}
        rmax = float(h ** 3) * rates.max() if "rmax_bound" in case["variant"] else max(v[2][:, -1].max() for v in lines.values())
        for o in octs:
            cls, cnt, acc = lines[o]
            r = _philox(n, 0, np.arange(K), o, seed)
            target = ((r[0] >> np.uint64(5)).astype(float) * 67108864.0 + (r[1] >> np.uint64(6)).astype(float)) / 2.0 ** 53 * rmax
            hit = np.nonzero(target < acc[:, -1])[0]
            c = (target[hit, None] >= acc[hit]).sum(axis=1)
            j = ((r[2][hit] * cnt[hit, c].astype(np.uint64)) >> np.uint64(32)).astype(np.int64)
            rank = np.cumsum(cls[hit] == c[:, None], axis=1)
            q = (rank > j[:, None]).argmax(axis=1)
            z = kz[hit] * d + (o >> 2 & 1) * h + q // (h * h)
            y = ky[hit] * d + (o >> 1 & 1) * h + q // h % h
            x = kx[hit] * d + (o & 1) * h + q % h
            step = np.where(up[z, y, x], -1, 1).astype(np.int8)
            up[z, y, x] ^= True
            for dz, dy, dx in ((1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)):
                np.add.at(nup, ((z + dz) % L, (y + dy) % L, (x + dx) % L), step)
        ut = (((w[2] >> 6) << 26 | w[3] >> 6) + 0.5) / 2.0 ** 52
        t += -math.log(ut) / ((2.0 if two else 8.0) * rmax)
        out.append(t)
    return out


def exact(case, seed):
    if case["kind"] not in ("run", "restart"):
        return None
    lines = {"": 1, "two_colours": 4, "rmax_all": 8}.get(case["variant"], 1)
    if case["L"] ** 3 / 8 * lines * case["cycles"] > 1.5e8 or case["cycles"] * case["L"] > 1e5:
        return None  # minutes in numpy
    times = _times(case, seed, _host_spins(case, seed) if case["kind"] == "restart" else None)
    out = dict(counts=None, t=np.array(times[-1:]), spins=None)
    if case.get("obs_every"):
        out["record_counts"], out["record_t"] = None, np.array(times[case["obs_every"] - 1::case["obs_every"]])
    return out
