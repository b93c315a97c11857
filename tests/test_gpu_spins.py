"""Spins of lattices that several host threads convert (2^21 sites and more), with
octant edges of 4 modulo 8: they come back as they were set, call after call, with
their M and B."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


@pytest.mark.parametrize("L,d", [(128, 8), (144, 24), (160, 40)])
def test_set_and_read(spkmc, L, d):
    print("case set and read", L, d, flush=True)
    sim = spkmc.Sim(L, d, layout="packed", init="up", seed=5)
    rng = np.random.default_rng(L + d)
    for _ in range(20):
        want = rng.choice(np.array([-1, 1], dtype=np.int8), L ** 3)
        sim.set_spins(want)
        assert np.array_equal(sim.spins(), want)
        s = want.reshape(L, L, L).astype(np.int64)
        assert sim.state()[4:] == (int(s.sum()), int(sum((s * np.roll(s, -1, a)).sum() for a in range(3))))
