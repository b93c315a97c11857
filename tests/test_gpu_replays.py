"""Captured calls replayed between other runs of the context: a replay changes the
lattice without a call of the library, so no launch may take its set-up or the slab
counts as the last one left them.  Against a twin that never captures; on the on-chip
launch (several workgroups, runs above and below its shortest) the twin stays on the
per-cycle kernels, a cycle a call."""
import struct

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


def _at_cycle(spkmc, blob, n):
    """The checkpoint with the context's cycle number set to n."""
    at = 8 + len(bytes(spkmc.Params()))
    out = bytearray(blob)
    out[at:at + 8] = struct.pack("<Q", n)
    return bytes(out)


@pytest.mark.parametrize("L,d,layout", [(64, 8, "int8"), (72, 8, "packed"), (96, 24, "packed"), (96, 32, "packed")])
def test_captured_run(spkmc, L, d, layout):
    import torch
    print("case captured run", L, d, layout, flush=True)
    kw = dict(layout=layout, engine="cycle", seed=9, T=4.5115)
    b = spkmc.Sim(L, d, **kw)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = spkmc.Sim(L, d, **kw)

    def both(*lengths):
        for n in lengths:
            a.run(n)
            for _ in range(n):
                b.run(1)
            _equal(a, b)

    both(20, 21)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.run(16)
    with torch.cuda.stream(stream):
        graph.replay()
    for _ in range(16):
        b.run(1)
    _equal(a, b)
    both(20, 21)
    for again in range(2):  # cycles 41 .. 56 once more, on the spins of now
        with torch.cuda.stream(stream):
            graph.replay()
        b.load(_at_cycle(spkmc, b.save(), 41))
        for _ in range(16):
            b.run(1)
        b.load(_at_cycle(spkmc, b.save(), 98 + 62 * again))
        _equal(a, b)
        both(22, 3, 37)


@pytest.mark.parametrize("engine,L,d,layout", [("cycle", 64, 8, "int8"), ("cycle", 96, 32, "packed"),
                                               ("cycle", 64, 16, "packed"), ("persistent", 160, 32, "packed"),
                                               ("incremental", 160, 32, "packed"), ("slab", 192, 32, "packed")])
def test_captured_init(spkmc, engine, L, d, layout):
    """Every replay starts the lattice anew; the context's cycle number goes on."""
    import torch
    print("case captured init", engine, L, d, layout, flush=True)
    kw = dict(layout=layout, engine=engine, seed=9, T=4.5115)
    b = spkmc.Sim(L, d, **kw)
    start = b.save()
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a = spkmc.Sim(L, d, **kw)
    done = 0
    for lengths in ((20, 21), (22, 20), (30,)):
        with torch.cuda.stream(stream):
            graph.replay()
        b.load(_at_cycle(spkmc, start, done))
        for n in lengths:
            a.run(n)
            b.run(n)
            done += n
            _equal(a, b)
