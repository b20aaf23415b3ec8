"""What a simulator holds beside its buffers."""
import numpy as np
import pytest

from paper_2303_02346_amd import scenes

pytestmark = pytest.mark.gpu


def test_a_simulator_keeps_no_host_copy_of_the_particles():
    """The initial state is on the device (100 bytes a particle); the arrays
    it was made from are the scenes'."""
    from paper_2303_02346_amd.sim import Simulator, STATE_ROWS
    sim = Simulator([scenes.tiny(n_particles=300, seed=s) for s in range(3)])

    def arrays(o):
        if isinstance(o, np.ndarray):
            yield o
        elif isinstance(o, dict):
            for v in o.values():
                yield from arrays(v)
        elif isinstance(o, (list, tuple)):
            for v in o:
                yield from arrays(v)

    own = {k: v for k, v in vars(sim).items() if k != "scenes"}
    assert max((a.size for a in arrays(own)), default=0) < sim.N
    assert sim._buf0.shape == (STATE_ROWS, sim.N) and sim._buf0.is_cuda
