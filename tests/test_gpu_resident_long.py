"""The on-chip launch (kernels_resident.hip) of several workgroups over runs long enough
to take it (its shortest run goes up to about 40 cycles, by the shape).  Launches that follow one another without a new set-up, over both parities of
every bank of slots, counters and records; launches after spins were set and states
restored.  Against the CPU oracle, every spin, counter and
record; the clock within 1e-12 relative (the device has its own logarithm)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

T_REL = 1e-12
RMAX_ALL, TWO, BOUND = 1, 2, 4
SHAPES = [(40, 4, "int8"), (64, 8, "int8"), (72, 8, "packed"), (90, 10, "int8"), (96, 24, "packed"), (64, 32, "int8"),
          (80, 40, "int8"), (100, 20, "int8"), (128, 8, "int8")]
# few lines: one workgroup up to 128 of 16 lanes or 32 of 64 (half as many with the
# all-octant maximum), else several; with two colours there are four times as many
FEW = [(8, 2, "int8"), (12, 4, "int8"), (16, 4, "int8"), (24, 4, "int8"), (24, 8, "int8"), (32, 8, "int8"),
       (40, 8, "packed"), (36, 12, "int8"), (48, 16, "int8"), (40, 20, "int8"), (60, 20, "int8"), (48, 24, "packed")]


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


def _pair(spkmc, L, d, layout, variant=0, **kw):
    kw = dict(dict(T=4.5115, H=0.05, rates="glauber", init="random", seed=77), **kw)
    gpu = spkmc.Sim(L, d, layout=layout, variant=variant, engine="cycle", record_cap=128, **kw)
    kw["rates"], kw["init"] = spkmc.RATES[kw["rates"]], spkmc.INITS[kw["init"]]
    return gpu, oracle.Sim(L=L, d=d, colours=2 if variant & TWO else 8,
                           rmax_scope=1 if variant & RMAX_ALL else 2 if variant & BOUND else 0, **kw)


def _same(g, o):
    assert g[:3] == o[:3] and g[4:] == o[4:], (g, o)
    assert abs(g[3] - o[3]) <= T_REL * abs(o[3]), (g, o)


def _compare(gpu, orc, want):
    got = gpu.records(len(want)) if want else []
    assert len(got) == len(want)
    for g, o in zip(got, want):
        _same(g, o)
    _same(gpu.state(), orc.state())
    assert np.array_equal(gpu.spins(), orc.spins())


def _advance(gpu, orc, lengths, obs):
    """Each run checked, then all of them without a read in between."""
    for n in lengths:
        gpu.run(n, obs_every=obs)
        _compare(gpu, orc, orc.run(n, obs_every=obs))
    want = []
    for n in lengths:
        gpu.run(n, obs_every=obs)
        want += orc.run(n, obs_every=obs)
    _compare(gpu, orc, want)


@pytest.mark.parametrize("variant", [0, RMAX_ALL, BOUND, TWO])
@pytest.mark.parametrize("L,d,layout", SHAPES + FEW)
def test_launch_after_launch(spkmc, L, d, layout, variant):
    print("case launch after launch", L, d, layout, variant, flush=True)
    gpu, orc = _pair(spkmc, L, d, layout, variant)
    _advance(gpu, orc, (49, 42, 41, 20), 3)


@pytest.mark.parametrize("L,d,layout", [(64, 8, "int8"), (72, 8, "packed"), (90, 10, "int8"), (96, 24, "packed")])
def test_after_host_writes(spkmc, L, d, layout):
    print("case long after host writes", L, d, layout, flush=True)
    gpu, orc = _pair(spkmc, L, d, layout, init="up", rates="metropolis")
    _advance(gpu, orc, (24, 33), 5)
    blob, want = gpu.save(), gpu.spins()
    gpu.run(29)
    gpu.load(blob)
    assert np.array_equal(gpu.spins(), want)
    _advance(gpu, orc, (24, 31), 4)
    spins = np.random.default_rng(L).choice(np.array([-1, 1], dtype=np.int8), L ** 3)
    gpu.set_spins(spins)
    orc.set_state(spins, *orc.state()[:4])
    _advance(gpu, orc, (32, 25), 4)
