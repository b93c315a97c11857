"""The per-cycle engine's on-chip launch (kernels_resident.hip) against the CPU
oracle: every record, the counters, M, B and every spin bit for bit, the clock
within 1e-12 relative (the device evaluates ln(u_t) with its own libm), across
launch boundaries (1, 2 and more cycles: the slots of a launch are set up anew
after a launch of one cycle, and left ready by longer ones)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

T_REL = 1e-12
RMAX_ALL, TWO, BOUND = 1, 2, 4


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


def _same(g, o):
    assert g[:3] == o[:3] and g[4:] == o[4:], (g, o)
    assert abs(g[3] - o[3]) <= T_REL * abs(o[3]), (g, o)


def _pair(spkmc, L, d, layout, variant, **kw):
    kw = dict(dict(T=4.5115, rates="glauber", init="random", seed=31), **kw)
    gpu = spkmc.Sim(L, d, layout=layout, variant=variant, record_cap=256, **kw)
    assert gpu.info()["engine"] == spkmc.ENGINES["cycle"]
    kw["rates"], kw["init"] = spkmc.RATES[kw["rates"]], spkmc.INITS[kw["init"]]
    return gpu, oracle.Sim(L=L, d=d, colours=2 if variant & TWO else 8,
                           rmax_scope=1 if variant & RMAX_ALL else 2 if variant & BOUND else 0, **kw)


def _advance(gpu, orc, launches, obs):
    for n in launches:
        gpu.run(n, obs_every=obs)
        ro = orc.run(n, obs_every=obs)
        rg = gpu.records(len(ro)) if ro else []
        assert len(rg) == len(ro)
        for g, o in zip(rg, ro):
            _same(g, o)
        _same(gpu.state(), orc.state())
        assert np.array_equal(gpu.spins(), orc.spins())


# one workgroup: one round of lines and several; 16 and 64 lanes per line; an octant of
# one site, octants that end inside a word of four sites
ONE_WG = [(2, 2, "int8"), (6, 2, "int8"), (12, 6, "int8"), (16, 8, "int8"), (24, 8, "packed"), (40, 8, "packed"),
          (18, 18, "int8"), (20, 20, "int8"), (24, 24, "packed")]
# several workgroups: a last one partly filled, neighbours across one and several
# workgroups, two domains along an edge (both neighbours the same domain), one domain
# per workgroup
MANY_WG = [(40, 4, "int8"), (72, 8, "packed"), (90, 10, "int8"), (96, 24, "packed"), (64, 32, "int8"),
           (80, 40, "int8"), (100, 20, "int8"), (128, 8, "int8")]


@pytest.mark.parametrize("variant", [0, RMAX_ALL, TWO, BOUND, TWO | RMAX_ALL, TWO | BOUND])
@pytest.mark.parametrize("L,d,layout", ONE_WG + MANY_WG)
def test_on_chip_vs_oracle(spkmc, L, d, layout, variant):
    print("case on-chip", L, d, layout, variant, flush=True)
    gpu, orc = _pair(spkmc, L, d, layout, variant, H=0.05)
    _advance(gpu, orc, (1, 1, 2, 19, 8), 1)
    _advance(gpu, orc, (13, 7), 4)


@pytest.mark.parametrize("L,d,layout", [(16, 8, "int8"), (72, 8, "packed"), (90, 10, "int8")])
def test_on_chip_after_host_writes(spkmc, L, d, layout):
    """Spins replaced and a checkpoint restored between launches: the bytes and
    counts of the next launch come from the spins and halos in memory."""
    print("case on-chip host writes", L, d, layout, flush=True)
    gpu, orc = _pair(spkmc, L, d, layout, 0, init="up", rates="metropolis")
    _advance(gpu, orc, (11,), 5)
    blob = gpu.save()
    want = gpu.spins()
    gpu.run(9)
    gpu.load(blob)
    assert np.array_equal(gpu.spins(), want)
    _advance(gpu, orc, (6, 5), 1)
    spins = orc.spins()
    gpu.set_spins(-spins)
    assert gpu.state()[4] == -orc.state()[4] and gpu.state()[5] == orc.state()[5]
    gpu.set_spins(spins)
    _advance(gpu, orc, (7, 3), 1)


@pytest.mark.parametrize("variant", [0, TWO])
def test_octants_too_large_for_a_workgroup(spkmc, variant):
    """Octant edge 28 (a domain of 175 616 sites): the three per-cycle kernels."""
    print("case per-cycle kernels", variant, flush=True)
    gpu, orc = _pair(spkmc, 112, 56, "int8", variant, H=-0.05)
    _advance(gpu, orc, (3, 4), 1)


@pytest.mark.parametrize("L,d,layout", [(16, 8, "int8"), (24, 24, "int8"), (64, 8, "int8"), (40, 40, "packed")])
def test_short_and_long_runs(spkmc, L, d, layout):
    """Runs too short to repay the on-chip set-up take the per-cycle kernels: lengths on
    both sides of the line in turn, each continuing where the other stopped."""
    print("case short and long runs", L, d, layout, flush=True)
    gpu, orc = _pair(spkmc, L, d, layout, 0, H=0.05)
    _advance(gpu, orc, (1, 12, 2, 3, 20, 1, 8, 4), 3)
