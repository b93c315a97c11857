"""The set-up kernels (random start, halo copies, M and B) and the spins' way in and
out against the oracle and plain numpy, over the octant edges with kernels of their
own (8, 16) and others, edges that are no multiple of the 128 sites of one draw, and
rows that end inside a byte of packed spins."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(16, 16, "packed"), (48, 16, "packed"), (96, 16, "packed"), (144, 16, "packed"), (32, 32, "packed"),
          (96, 32, "packed"), (160, 32, "packed"), (256, 32, "packed"), (8, 8, "packed"), (24, 8, "packed"),
          (72, 24, "packed"), (80, 40, "packed"), (72, 72, "packed"), (2, 2, "int8"), (30, 10, "int8"),
          (66, 22, "int8"), (200, 8, "int8")]


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


def _observables(spins, L):
    s = spins.reshape(L, L, L).astype(np.int64)
    return int(s.sum()), int(sum((s * np.roll(s, -1, a)).sum() for a in range(3)))


@pytest.mark.parametrize("init", ["random", "up", "down"])
@pytest.mark.parametrize("L,d,layout", SHAPES)
def test_start(spkmc, L, d, layout, init):
    print("case start", L, d, layout, init, flush=True)
    sim = spkmc.Sim(L, d, layout=layout, init=init, seed=(1 << 40) + 7)
    want = oracle.Sim(L=L, d=d, init=spkmc.INITS[init], seed=(1 << 40) + 7).spins()
    assert np.array_equal(sim.spins(), want)
    assert sim.state() == (0, 0, 0, 0.0) + _observables(want, L)


@pytest.mark.parametrize("L,d,layout", SHAPES)
def test_spins_set_and_read(spkmc, L, d, layout):
    """Any spins come back as they were set, with their M and B; what is not +1 or -1
    is refused, wherever it is, and changes nothing."""
    print("case set spins", L, d, layout, flush=True)
    sim = spkmc.Sim(L, d, layout=layout, seed=3)
    want = np.random.default_rng(L * d).choice(np.array([-1, 1], dtype=np.int8), L ** 3)
    sim.set_spins(want)
    assert np.array_equal(sim.spins(), want)
    assert sim.state()[4:] == _observables(want, L)
    for bad in (0, 2, -2, 127, -128, -127):
        spins = np.ones(L ** 3, dtype=np.int8)
        spins[(bad * 37) % L ** 3] = bad
        with pytest.raises(spkmc.SpkmcError):
            sim.set_spins(spins)
    assert np.array_equal(sim.spins(), want)
    assert sim.state()[4:] == _observables(want, L)
    # the halo copies: a cycle from these spins ends with the M and B of its spins
    sim.run(3)
    assert sim.state()[4:] == _observables(sim.spins(), L)
