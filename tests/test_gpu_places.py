"""The per-cycle kernels' sums over workgroups: in the state header for few workgroups, in
up to 64 places for many.  Lattices on both sides of each line, against the persistent
engine (packed) and the oracle (bytes, a cycle a call: longer runs go on chip)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spkmc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1005_4713_amd import spkmc as mod
    return mod


# octant edge 8: 256 lines to a workgroup, 13 824 lines one place, 17 576 eight; edge 16: 64
# (two colours 128), 3375 lines one and 4096 eight, 6912 one and 8788 eight
@pytest.mark.parametrize("L,d,variant", [(384, 16, 0), (416, 16, 0), (416, 16, 4), (240, 16, 2), (272, 16, 2),
                                         (480, 32, 0), (512, 32, 0), (480, 32, 4), (384, 32, 2), (416, 32, 2)])
def test_packed(spkmc, L, d, variant):
    print("case places", L, d, variant, flush=True)
    kw = dict(layout="packed", variant=variant, seed=21, T=4.5115, H=0.05, record_cap=32)
    a, b = spkmc.Sim(L, d, engine="cycle", **kw), spkmc.Sim(L, d, engine="persistent", **kw)
    for n in (5, 8):
        a.run(n, obs_every=1)
        b.run(n, obs_every=1)
        assert a.records() == b.records()
        assert a.state() == b.state()
    assert np.array_equal(a.spins(), b.spins())


# 1 to 4 lines to a workgroup: up to 127 lines one place, 64 domains with two colours four,
# 216 domains eight; the all-octant maximum of packed lattices
@pytest.mark.parametrize("L,d,layout,variant", [(40, 8, "int8", 0), (32, 8, "int8", 2), (40, 8, "int8", 2), (48, 8, "int8", 0), (48, 8, "int8", 2), (48, 8, "int8", 1),
                                                (80, 16, "packed", 1), (96, 16, "packed", 1), (128, 8, "int8", 0)])
def test_generic(spkmc, L, d, layout, variant):
    print("case places generic", L, d, layout, variant, flush=True)
    gpu = spkmc.Sim(L, d, layout=layout, engine="cycle", variant=variant, seed=21, T=4.5115, H=0.05)
    orc = oracle.Sim(L=L, d=d, seed=21, T=4.5115, H=0.05, colours=2 if variant & 2 else 8, rmax_scope=variant & 1)
    for _ in range(12):
        gpu.run(1)
        orc.run(1)
        g, o = gpu.state(), orc.state()
        assert g[:3] == o[:3] and g[4:] == o[4:]
        assert abs(g[3] - o[3]) <= 1e-12 * abs(o[3])
    assert np.array_equal(gpu.spins(), orc.spins())
