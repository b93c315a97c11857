"""On-chip launches of several contexts in turn: the launch limits belong to the kernel,
not to the context that set them last."""
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


# (large, small) of one kernel instance: 64 lanes per line and 16
@pytest.mark.parametrize("large,small", [((48, 48), (20, 20)), ((96, 48), (40, 20)), ((128, 8), (8, 4)), ((40, 10), (6, 2))])
def test_contexts_of_different_sizes(spkmc, large, small):
    print("case sizes", large, small, flush=True)
    pairs = []
    for L, d in (large, small):  # the smaller one made last
        pairs.append((spkmc.Sim(L, d, layout="int8", engine="cycle", T=4.5115, seed=4),
                      oracle.Sim(L=L, d=d, T=4.5115, seed=4)))
    for _ in range(3):
        for gpu, orc in (pairs[1], pairs[0]):
            gpu.run(64)
            orc.run(64)
            g, o = gpu.state(), orc.state()
            assert g[:3] == o[:3] and g[4:] == o[4:]
            assert abs(g[3] - o[3]) <= 1e-12 * abs(o[3])
            assert np.array_equal(gpu.spins(), orc.spins())
