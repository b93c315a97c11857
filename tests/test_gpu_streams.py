"""Contexts on streams of their own: a launch of one workgroup, a plain dispatch, beside
cooperative launches that need every compute unit (their waits end after 2 s)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ONE_WG = [(16, 8, "int8", "cycle"), (32, 32, "packed", "persistent"), (32, 32, "packed", "slab")]


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


@pytest.mark.parametrize("L,d,layout,engine", ONE_WG)
def test_long_run_of_one_workgroup(spkmc, L, d, layout, engine):
    """More cycles than one launch of a single workgroup takes, against the oracle."""
    print("case long run", L, d, layout, engine, flush=True)
    gpu = spkmc.Sim(L, d, layout=layout, engine=engine, rates="glauber", init="random", T=4.5115, seed=12, record_cap=64)
    orc = oracle.Sim(L=L, d=d, rates=spkmc.RATES["glauber"], init=spkmc.INITS["random"], T=4.5115, seed=12)
    for n in (4096, 4097, 8195):
        gpu.run(n, obs_every=1000)
        want = orc.run(n, obs_every=1000) + [orc.state()]
        got = gpu.records(len(want) - 1) + [gpu.state()]
        assert len(got) == len(want)
        for g, o in zip(got, want):
            assert g[:3] == o[:3] and g[4:] == o[4:]
            assert abs(g[3] - o[3]) <= 1e-12 * abs(o[3])
        assert np.array_equal(gpu.spins(), orc.spins())


@pytest.mark.parametrize("L,d,layout,engine", ONE_WG)
def test_beside_a_launch_of_the_whole_chip(spkmc, L, d, layout, engine):
    """A run of one workgroup of more than 2 s, and runs of 1024^3 on another stream
    meanwhile: these end while the long one goes on, with the results they have alone."""
    import torch
    print("case beside", L, d, layout, engine, flush=True)
    alone = spkmc.Sim(1024, 32, layout="packed", T=4.5115, seed=8)
    for _ in range(3):
        alone.run(20)
    want = alone.state()
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(one):
        a = spkmc.Sim(L, d, layout=layout, engine=engine, T=4.5115, seed=8)
    with torch.cuda.stream(other):
        b = spkmc.Sim(1024, 32, layout="packed", T=4.5115, seed=8)
    b.state()
    n = 1000000 if layout == "int8" else 600000
    a.run(n)
    for _ in range(3):
        b.run(20)
        other.synchronize()
    running = not one.query()
    assert b.state() == want
    assert running
    assert a.state()[0] == n
