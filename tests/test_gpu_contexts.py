"""Creating and destroying contexts beside other work."""
import gc

import numpy as np
import pytest
import torch

from paper_2303_02346_amd import _lib, scenes

pytestmark = pytest.mark.gpu


def particles():
    from paper_2303_02346_amd.sim import Simulator
    return Simulator(scenes.tiny(n_particles=100, steps=4))


def gas():
    from paper_2303_02346_amd.gas import GasSim
    return GasSim(scenes.gas_room(n=(8, 8, 8), steps=4))


@pytest.mark.parametrize("make", [particles, gas])
@pytest.mark.parametrize("collect", [False, True])
def test_contexts_can_be_destroyed_during_a_graph_capture(make, collect):
    """A program's own graph capture goes on when a simulator of its is closed
    or collected in between, as garbage collection may do at any time."""
    sim = make()
    sim.step(1)
    x = torch.ones(1000, device="cuda")
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y.copy_(x * 2)
        if collect:
            del sim
            gc.collect()
        else:
            sim.close()
    for v in (3.0, 5.0):
        x.fill_(v)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full_like(y, 2 * v))
    again = make()
    again.step(1)


def test_many_contexts_report_their_own_errors():
    """More contexts than one page of error words serves, destroyed and
    created again in between: each reports its own invalid state and no
    other's."""
    sims = [particles() for _ in range(70)]
    for k in range(0, 70, 3):
        sims[k].close()
        sims[k] = particles()
    bad = {5, 63, 64, 69}
    for k in bad:
        sims[k].x[0, 0] = float("nan")
    for k, s in enumerate(sims):
        if k in bad:
            with pytest.raises(_lib.MpmError) as e:
                s.step(2)
            assert e.value.status == _lib.MPM_EDOMAIN and e.value.bits & 1
        else:
            s.step(2)
            assert np.isfinite(s.positions()).all()
    for s in sims:
        s.reset()
        s.step(4)
