"""What the closure's training keeps between its calls."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2303_02346_amd import _lib
from test_gpu_closure import synthetic_records

P = 4803
BLOCK = (4 * P + 255) // 256 * 64        # floats of a parameter block of the state: params, m, v


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["workspace", "static"])
def test_a_gradient_call_clears_the_adam_step_count(entry):
    """A training step after a gradient call takes the bias correction of a
    first step (beta 0.9 and 0.999) on the moments that are there.  The update
    is known to FP32 rounding; the correction of a step after 5 differs by
    more than a half."""
    from paper_2303_02346_amd.closure import MLP
    rec = torch.from_numpy(synthetic_records(700, seed=4)).cuda()
    lr = 1e-3
    net = MLP()
    net.init(rec, seed=1)
    net.train(rec, epochs=5, batch=700, lr=lr, seed=2)
    if entry == "workspace":
        _, g = net.grad(rec, batch=700)
    else:
        g = torch.zeros(P, device="cuda")
        loss = ctypes.c_double(0)
        assert _lib.lib().mpm_mlp_grad_noalloc(
            ctypes.c_void_p(net.state.data_ptr()), ctypes.c_void_p(rec.data_ptr()), 700, 700,
            ctypes.c_void_p(g.data_ptr()), ctypes.byref(loss),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == _lib.MPM_OK
    p, m, v = (net.state[k * BLOCK:k * BLOCK + P].double().cpu().numpy() for k in range(3))
    g = g.double().cpu().numpy()
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    net.train(rec, epochs=1, batch=700, lr=lr, seed=3)
    step = net.state[:P].double().cpu().numpy() - p

    def update(t):
        return -lr * (m / (1 - 0.9 ** t)) / (np.sqrt(v / (1 - 0.999 ** t)) + 1e-8)

    rel = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))
    print(f"  update against a first step's {rel(step, update(1)):.2e}, a sixth's {rel(step, update(6)):.2e}", flush=True)
    assert rel(step, update(1)) <= 1e-2 and rel(step, update(6)) >= 0.2


def test_scratch_leaves_room_to_align_it():
    """816 bytes a record and 8 per 16 of them, and 15 to reach the next
    multiple of 16 (host arithmetic: no GPU)."""
    size = _lib.lib().mpm_mlp_scratch_bytes
    for batch in list(range(1, 2049)) + [4096, 16385, 1 << 20]:
        assert size(batch) >= 816 * batch + 8 * ((batch + 15) // 16) + 15


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [1, 17, 700])
def test_scratch_of_any_alignment(batch):
    """The gradient does not depend on where the scratch starts, and what
    follows it stays as it was."""
    from paper_2303_02346_amd.closure import MLP
    rec = torch.from_numpy(synthetic_records(700, seed=4)).cuda()
    net = MLP()
    net.init(rec, seed=1)
    loss0, ref = net.grad(rec, batch=batch)
    n = _lib.lib().mpm_mlp_scratch_bytes(batch)
    for shift in (0, 4, 8, 12):
        buf = torch.full((n + 64,), 123, dtype=torch.uint8, device="cuda")
        g = torch.zeros(P, device="cuda")
        loss = ctypes.c_double(0)
        assert _lib.lib().mpm_mlp_grad(
            ctypes.c_void_p(net.state.data_ptr()), ctypes.c_void_p(rec.data_ptr()), 700, batch,
            ctypes.c_void_p(buf.data_ptr() + shift), ctypes.c_void_p(g.data_ptr()), ctypes.byref(loss),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == _lib.MPM_OK
        assert loss.value == loss0 and torch.equal(g, ref)
        assert bool((buf[:shift] == 123).all()) and bool((buf[n + shift:] == 123).all())
