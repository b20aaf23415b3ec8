"""Calls that hand over device memory keep their order with torch's streams.

On the CPU the library and the streams are stand-ins that write down what is
called; on the GPU the same calls are made from two streams."""
import types

import pytest
import torch

from paper_2303_02346_amd import _lib, gas as gas_mod, scenes, sim as sim_mod


class Recorder:
    """A library that notes every call on it."""

    def __init__(self, log):
        self._log = log

    def __getattr__(self, what):
        def call(*a, **k):
            self._log.append(what)
            return 0
        return call


class Stream:
    """A stream that notes what it waits for and when the host waits for it."""

    def __init__(self, log, name, stream_id=33, cuda_stream=0x1000):
        self._log, self._name, self.stream_id, self.cuda_stream = log, name, stream_id, cuda_stream

    def wait_stream(self, other):
        self._log.append(f"{self._name} waits for {other._name}")

    def synchronize(self):
        self._log.append(f"host waits for {self._name}")


def simulator_stub(monkeypatch, rigid=False):
    """A simulator on stand-ins, its log, and a function that makes a stream
    current."""
    log = []
    sim = object.__new__(sim_mod.Simulator)
    sim.ctx, sim.device = types.SimpleNamespace(value=0), torch.device("cpu")
    sim.mat, sim.buf = torch.zeros(4, dtype=torch.uint8), torch.zeros(sim_mod.STATE_ROWS, 4)
    sim.stream, sim._written, sim._rigid = Stream(log, "library"), [], rigid
    current = [Stream(log, "a")]
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: current[0])
    monkeypatch.setattr(_lib, "lib", lambda: Recorder(log))

    def use(stream):
        current[0] = stream
    return sim, log, use


def test_state_set_under_another_stream_is_waited_for(monkeypatch):
    """The state may have been written on the stream that is current at
    set_state, and the step that reads it follow under another one."""
    sim, log, use = simulator_stub(monkeypatch)
    sim.set_state()
    use(Stream(log, "b"))
    sim.set_state()
    use(Stream(log, "c"))
    sim.step(1)
    assert log[:2] == ["mpm_set_state"] * 2 and log[-1] == "mpm_step"
    assert sorted(log[2:-1]) == [f"library waits for {s}" for s in "abc"]
    del log[:]
    sim.step(1)                  # (once)
    assert log == ["library waits for c", "mpm_step"]


def test_state_set_under_the_stream_of_the_step_is_waited_for_once(monkeypatch):
    sim, log, use = simulator_stub(monkeypatch)
    sim.set_state()
    sim.step(1)
    assert log == ["mpm_set_state", "library waits for a", "mpm_step"]


@pytest.mark.parametrize("rigid,stream", [(True, {}), (False, {"stream_id": 0x1000})])
def test_state_is_waited_for_at_once(monkeypatch, rigid, stream):
    """Rest shapes are taken from the state by set_state itself; a stream of
    the caller's own may be destroyed before the step."""
    sim, log, use = simulator_stub(monkeypatch, rigid)
    use(Stream(log, "own", **stream))
    sim.set_state()
    assert log == ["library waits for own", "mpm_set_state"]


def test_load_waits_for_its_copy(monkeypatch):
    """The initial state is kept on the device, and a copy within the device
    returns before it is done."""
    sim, log, _ = simulator_stub(monkeypatch)
    sim._buf0 = torch.ones(sim_mod.STATE_ROWS, 4)
    sim.load()
    assert torch.equal(sim.buf, sim._buf0) and log == ["host waits for a"]


@pytest.mark.parametrize("function,restore", [(sim_mod.MpmRollout, "load"), (gas_mod.GasRollout, "reset")])
def test_rollouts_restore_their_state_through_load_and_reset(function, restore):
    """(a program that starts its rollouts elsewhere overrides these)  Their
    wait is left out there, and only there: the step waits."""
    log = []
    state = types.SimpleNamespace(requires_grad=True, x=torch.zeros(3, 4), v=torch.zeros(3, 4), buf=torch.zeros(25, 4),
                                  _buf0=torch.zeros(25, 4), _step_follows=False)

    def note(name, fail=False):
        def call(*a):
            log.append((name, state._step_follows))
            if fail:
                raise RuntimeError(name)
        return call

    for name in ("load", "reset", "set_state", "set_actions", "step"):
        setattr(state, name, note(name))
    function.forward(types.SimpleNamespace(), torch.zeros(2, 1, 6), state)
    assert log[0] == (restore, True) and log[-2:] == [("set_actions", False), ("step", False)]
    setattr(state, restore, note(restore, fail=True))
    with pytest.raises(RuntimeError):
        function.forward(types.SimpleNamespace(), torch.zeros(2, 1, 6), state)
    assert not state._step_follows


def test_gas_reset_waits_for_its_transfers(monkeypatch):
    """The initial fields go through staging memory, in transfers that return
    before they are done."""
    log = []
    sim = object.__new__(gas_mod.GasSim)
    sim.ctx, sim.device = types.SimpleNamespace(value=0), torch.device("cpu")
    sim.buf, sim.actions = torch.zeros(4), torch.zeros(2, 6)
    sim.stream = Stream(log, "library")
    for name in ("load", "set_actions"):
        monkeypatch.setattr(sim, name, lambda *a, n=name: log.append(n), raising=False)
    monkeypatch.setattr(sim, "struct", lambda buf: _lib.GasState(), raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(log, "a"))
    monkeypatch.setattr(_lib, "lib", lambda: Recorder(log))
    sim.reset()
    assert log.index("host waits for a") > log.index("load")


def delayed(stream):
    """About 0.1 s of work on the stream, for what follows on it to be late."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(200_000_000)


@pytest.mark.gpu
def test_state_written_on_another_stream_is_the_one_stepped():
    sc = scenes.tiny(n_particles=300, steps=4, seed=3)
    sim = sim_mod.Simulator(sc)
    start = sim.buf.clone()
    sim.step(4)
    ref = sim.buf.clone()
    sim.reset()
    sim.buf.zero_()
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    delayed(other)
    with torch.cuda.stream(other):
        sim.buf.copy_(start)
        sim.set_state()
    sim.step(4)
    # (the sums' order differs from run to run)
    assert torch.allclose(sim.buf, ref, rtol=0, atol=1e-5 * float(ref.abs().max()))


@pytest.mark.gpu
def test_loaded_state_is_there_for_every_stream():
    sim = sim_mod.Simulator(scenes.tiny(n_particles=300, steps=4, seed=3))
    start = sim.buf.clone()
    for call in (sim.load, sim.reset):
        sim.buf.zero_()
        torch.cuda.synchronize()
        other = torch.cuda.Stream()
        delayed(other)
        with torch.cuda.stream(other):
            call()
        assert torch.equal(sim.buf, start)


@pytest.mark.gpu
def test_gas_state_is_there_for_every_stream_after_a_reset():
    sim = gas_mod.GasSim(scenes.gas_room(n=(16, 24, 32), steps=2))
    start = sim.buf.clone()
    sim.buf.zero_()
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    delayed(other)
    with torch.cuda.stream(other):
        sim.reset()
    assert torch.equal(sim.buf, start)
