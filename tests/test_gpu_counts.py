"""Counts that stay with the lattice between runs (the slab kernels bin them
only when something else changed the spins), and the per-cycle engine under stream
capture: against a twin on the re-binning engine, bit for bit, with everything that
changes spins between the runs."""
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


def _equal(a, b):
    assert a.state() == b.state()
    assert np.array_equal(a.spins(), b.spins())


@pytest.mark.parametrize("engine,L,variant", [
    ("cycle", 96, 0), ("cycle", 160, 0), ("cycle", 160, 4), ("cycle", 224, 0),  # 27, 125 and 343 lines
    ("slab", 96, 0), ("slab", 160, 0), ("slab", 96, 1), ("slab", 192, 1),       # 1 and 2 workgroups
])
def test_counts_follow_every_change(spkmc, engine, L, variant):
    print("case counts", engine, L, variant, flush=True)
    kw = dict(layout="packed", variant=variant, seed=17, T=4.5115, H=0.05, record_cap=64)
    twin = "incremental" if variant == 1 else "persistent"
    a, b = spkmc.Sim(L, 32, engine=engine, **kw), spkmc.Sim(L, 32, engine=twin, **kw)

    def both(n):
        a.run(n, obs_every=2)
        b.run(n, obs_every=2)
        _equal(a, b)
        assert a.records() == b.records()

    both(5)
    both(7)
    blob, other = a.save(), b.save()
    if variant != 1:  # a batch does not take the all-octant R_max
        spkmc.run_batch([a], 4)
        b.run(4)
        both(6)
    a.load(blob)
    b.load(other)
    both(3)
    for s in (a, b):
        s.set_spins(-s.spins())
    both(4)
    if variant != 1:
        g = spkmc.BatchGraph([a], 3)
        g.launch(2)
        b.run(6)
        _equal(a, b)
        g.close()
    both(2)


@pytest.mark.parametrize("L,d,layout", [(96, 32, "packed"), (48, 8, "int8"), (72, 8, "packed")])
def test_capture(spkmc, L, d, layout):
    """A captured run replays its own cycles and leaves the runs around it right."""
    import torch
    print("case capture", L, d, layout, flush=True)
    kw = dict(layout=layout, engine="cycle", seed=9, T=4.5115)
    b = spkmc.Sim(L, d, **kw)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = spkmc.Sim(L, d, **kw)
    for s in (a, b):
        s.run(3)
        s.run(4)
    _equal(a, b)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.run(5)
    with torch.cuda.stream(stream):
        graph.replay()
    b.run(5)
    _equal(a, b)
    for n in (1, 6):
        a.run(n)
        b.run(n)
        _equal(a, b)
