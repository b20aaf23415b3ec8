"""GPU parity: the HIP step (through the C ABI) against the FP64 oracle on
identical seeded inputs.

Tolerance (positions after 100 steps): ||X_gpu - X_ref||_F / ||X_ref||_F
<= 1e-4, the relative tolerance the build targets for the FP32 step with
FP64 SVD/polar.  Gradients: ||g_gpu - g_ref|| / ||g_ref||.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import mpm_oracle as O
from paper_2303_02346_amd import scenes
from paper_2303_02346_amd import _lib

pytestmark = pytest.mark.gpu


from parity import compare_states, liquid_mask, rel, say, state_errors


def sim_of(sc, **kw):
    from paper_2303_02346_amd.sim import Simulator
    return Simulator(sc, **kw)


def oracle_state(sc, steps):
    st = O.rollout(sc, steps=steps)
    return {k: v.detach().numpy() for k, v in st.items()}


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_tiny_one_step_all_materials(seed):
    sc = scenes.tiny(n_particles=300, n_grid=24, steps=1, seed=seed)
    say(f"tiny one step seed {seed}")
    sim = sim_of(sc)
    sim.step(1)
    compare_states(sim.state_numpy(), oracle_state(sc, 1), liquid_mask(sc), tol_x=1e-6, tol=1e-4)


def test_tiny_many_steps_with_contact():
    sc = scenes.tiny(n_particles=600, n_grid=32, steps=60, seed=4, dt=1e-4)
    say("tiny 60 steps")
    sim = sim_of(sc)
    sim.step(60)
    compare_states(sim.state_numpy(), oracle_state(sc, 60), liquid_mask(sc), tol_x=1e-5, tol=2e-3)


def test_config1_free_fall_100_steps():
    sc = scenes.config1()
    say("config 1, 100 steps")
    sim = sim_of(sc)
    sim.step(100)
    g = sim.state_numpy()
    x0 = sc.x
    dy = -9.8 * sc.dt ** 2 * 100 * 101 / 2
    assert np.abs(g["x"][:, 1] - x0[:, 1] - dy).max() < 2e-6
    ref = oracle_state(sc, 100)
    compare_states(g, ref, liquid_mask(sc), tol_x=1e-6, tol=1e-4, tol_x_max=1e-5, tol_max=1e-3, tol_FJ=1e-5,
                   n_grid=sc.n_grid)


def test_config1b_affine_100_steps():
    sc = scenes.config1(affine=True)
    say("config 1b (affine velocity), 100 steps")
    sim = sim_of(sc)
    sim.step(100)
    g = sim.state_numpy()
    ref = oracle_state(sc, 100)
    # the stiff elastic body's velocities carry the FP32 rounding of 100
    # steps of its stress (1.3e-4 measured): their gates are 5e-4 / 2e-3
    compare_states(g, ref, liquid_mask(sc), tol_x=1e-6, tol=5e-4, tol_x_max=1e-5, tol_max=2e-3, tol_FJ=1e-5)


def test_config2_full_size_first_steps():
    """Config 2 at its full size (250k particles, 128^3) in the launch
    configuration the benchmark times, 3 steps against the oracle."""
    sc = scenes.config2()
    say("config 2 full size, 3 steps")
    sim = sim_of(sc)
    sim.step(3)
    g = sim.state_numpy()
    ref = oracle_state(sc, 3)
    compare_states(g, ref, liquid_mask(sc), tol_x=1e-6, tol=1e-3)


@pytest.mark.timeout(900)
def test_config2_full_size_100_steps_vs_oracle():
    """Config 2 at its full size (250k particles, 128^3) in the launch the
    benchmark times (autotuned shape), 100 steps against the oracle: the
    stated bar of 1e-4 relative error on positions after 100 steps, here
    asserted per particle as well.  The window holds particles inside the
    cylinder's contact band."""
    from parity import oracle_rollout_coverage
    sc = scenes.config2(steps=100)
    say("config 2 full size, 100 steps (autotuned launch)")
    sim = sim_of(sc)
    tune = sim.autotune(n_steps=10)
    say(f"  launch {tune}")
    sim.reset()
    sim.step(100)
    g = sim.state_numpy()
    ref, cases, band = oracle_rollout_coverage(O, sc, 100)
    say(f"  oracle window: sand cases inside/apex/cone {cases.tolist()}, particle-steps in the contact band {band}")
    assert band > 1000
    compare_states(g, ref, liquid_mask(sc), tol_x=1e-5, tol=1e-3, tol_x_max=1e-4, tol_max=1e-2, tol_FJ=1e-4,
                   tol_FJ_max=1e-3)


@pytest.mark.timeout(900)
def test_config2_stirred_sand_100_steps_vs_oracle():
    """Config 2 at full size with the sand box stirred (a seeded smooth
    velocity field of 1 m/s), so that the window holds all three
    Drucker-Prager cases (inside, apex, cone) and the contact band; 100
    steps against the oracle, Frobenius and per-particle."""
    from parity import oracle_rollout_coverage
    sc = scenes.config2(steps=100, sand_stir=1.0)
    say("config 2 full size with stirred sand, 100 steps")
    sim = sim_of(sc)
    sim.step(100)
    g = sim.state_numpy()
    ref, cases, band = oracle_rollout_coverage(O, sc, 100)
    say(f"  oracle window: sand cases inside/apex/cone {cases.tolist()}, particle-steps in the contact band {band}")
    assert (cases > 100).all() and band > 1000
    compare_states(g, ref, liquid_mask(sc), tol_x=1e-5, tol=1e-3, tol_x_max=1e-4, tol_max=1e-2, tol_FJ=1e-4,
                   tol_FJ_max=1e-2)


def test_config2_full_horizon_invariants():
    """200 steps of config 2: finite state inside the domain; the sand box,
    which neither the cylinder nor the walls reach in 10 ms, keeps its
    momentum balance: its mean displacement is the free-fall value
    g dt^2 n(n+1)/2 (stresses carry no net force through APIC)."""
    sc = scenes.config2()
    say("config 2 full size, 200 steps")
    sim = sim_of(sc)
    sim.step(200)
    g = sim.state_numpy()
    assert np.isfinite(g["x"]).all() and np.isfinite(g["v"]).all()
    assert (g["x"] > 0).all() and (g["x"] < 1).all()
    sand = ~liquid_mask(sc)
    dy = (g["x"][sand, 1] - sc.x[sand, 1]).mean()
    ref = -9.8 * sc.dt ** 2 * 200 * 201 / 2
    say(f"  sand mean dy {dy:.6e} free fall {ref:.6e}")
    assert abs(dy - ref) <= 2e-3 * abs(ref)


def test_domain_error_is_reported():
    sc = scenes.tiny(n_particles=50, n_grid=16, steps=2)
    sc.x[3] = [0.01, 0.5, 0.5]          # stencil leaves the grid
    say("domain error")
    sim = sim_of(sc)
    with pytest.raises(_lib.MpmError) as e:
        sim.step(1)
    assert e.value.status == _lib.MPM_EDOMAIN and e.value.bits & 1


def test_nonfinite_error_is_reported():
    sc = scenes.tiny(n_particles=50, n_grid=16, steps=2)
    sc.v[5] = [np.nan, 0.0, 0.0]
    say("non-finite error")
    sim = sim_of(sc)
    with pytest.raises(_lib.MpmError) as e:
        sim.step(2)
    assert e.value.status == _lib.MPM_EDOMAIN


def test_sand_sigma_error_is_reported():
    """A sand particle whose deformation gradient has det F <= 0 (here
    diag(1, 1, -1)) is an invalid state: the call reports MPM_ERR_SAND_SIGMA
    and does not clamp it."""
    sc = scenes.tiny(n_particles=60, n_grid=16, steps=2, kinds=(scenes.SAND,), with_cylinder=False)
    sc.F[7] = np.diag([1.0, 1.0, -1.0])
    say("sand sigma error")
    sim = sim_of(sc)
    with pytest.raises(_lib.MpmError) as e:
        sim.step(1)
    assert e.value.status == _lib.MPM_EDOMAIN and e.value.bits & 4


def test_tile_reach_error_is_reported():
    """A particle that moves more than one cell in a step leaves the reach of
    the transfer tiles (the CFL > 1 condition): MPM_ERR_TILE."""
    sc = scenes.tiny(n_particles=60, n_grid=32, steps=3, kinds=(scenes.ELASTIC,), with_cylinder=False)
    dx = 1.0 / sc.n_grid
    # one particle far from the others, moving 8 cells per step along x (a
    # particle's stencil may drift at most one cell per step from its block)
    sc.x[11] = [0.4, 0.8, 0.5]
    sc.v[11] = [8.0 * dx / sc.dt, 0.0, 0.0]
    say("tile reach error")
    sim = sim_of(sc)
    with pytest.raises(_lib.MpmError) as e:
        sim.step(3)
    assert e.value.status == _lib.MPM_EDOMAIN and e.value.bits & 8


@pytest.mark.timeout(600)
@pytest.mark.parametrize("threads", [512, 0])
def test_paper_operating_point_vs_oracle(threads):
    """The paper's operating point (section 4.2, App. B.1: about 1e5
    particles of Table 4 water, viscous liquid and elastic solid on 64^3, dt
    1e-4) in the 512-thread launch the autotuner picks for it (and, threads
    = 0, whatever it picks), 20 steps against the oracle."""
    sc = scenes.paper_point(steps=20)
    say(f"paper operating point, {sc.n} particles, 20 steps, threads {threads or 'autotuned'}")
    sim = sim_of(sc)
    tune = sim.autotune(n_steps=10)
    if threads:
        sim.set_option(_lib.MPM_OPT_PART_THREADS, threads)
    say(f"  launch {tune}, particle threads {sim.get_option(_lib.MPM_OPT_PART_THREADS)}")
    sim.reset()
    sim.step(20)
    compare_states(sim.state_numpy(), oracle_state(sc, 20), liquid_mask(sc), tol_x=1e-6, tol=1e-3, tol_FJ=1e-5)


# ---------------------------------------------------------------------------
# gradients
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("adjoint", ["tiled", "plain"])
@pytest.mark.parametrize("seed,ckpt", [(0, 3), (1, 3), (0, 1), (1, 8)])
def test_gradient_tiny_vs_oracle(seed, ckpt, adjoint):
    """Segments of 3, 3 and 2 steps, of one step each (no fused recompute
    step), and one segment of all 8 steps."""
    sc = scenes.tiny(n_particles=90, n_grid=16, steps=8, seed=seed)
    say(f"gradient tiny seed {seed}, checkpoint every {ckpt}, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=ckpt, adjoint=adjoint)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga = sim.backward(g[0:3], torch.zeros_like(g[0:3]))[:, 0].double().cpu().numpy()
    L, gref = O.loss_and_action_grad(sc)
    gref = gref.numpy()
    e = rel(ga, gref)
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; grad rel err {e:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert e <= 1e-4


@pytest.mark.parametrize("adjoint", ["tiled", "plain"])
def test_gradient_state0_vs_oracle(adjoint):
    """dL/dx_0 and dL/dv_0 through the full adjoint (P2G/G2P weights,
    stresses, contact) against oracle autograd."""
    sc = scenes.tiny(n_particles=90, n_grid=16, steps=5, seed=2)
    say(f"gradient wrt initial state, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=2, adjoint=adjoint)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    p = O.params_from_scene(sc)
    st0 = O.state_from_scene(sc, requires_grad=True)
    st = O.rollout(sc, state=st0, params=p)
    L = O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma)
    L.backward()
    gx = g0[0:3].T.double().cpu().numpy()
    gv = g0[3:6].T.double().cpu().numpy()
    ex = rel(gx, st0["x"].grad.numpy())
    ev = rel(gv, st0["v"].grad.numpy())
    say(f"  dL/dx0 rel {ex:.2e} dL/dv0 rel {ev:.2e}")
    assert ex <= 1e-4 and ev <= 1e-4


# ---------------------------------------------------------------------------
# von Mises ice cream (section 3.2's non-Newtonian liquid)
# ---------------------------------------------------------------------------
def _ice_cream_scene(steps, n=600, seed=5):
    return scenes.tiny(n_particles=n, n_grid=24, steps=steps, seed=seed,
                       kinds=(scenes.VONMISES, scenes.LIQUID), velocity=3.0, dt=1e-4)


@pytest.mark.parametrize("adjoint", ["tiled", "plain"])
def test_gradient_ill_conditioned_solids_vs_oracle(adjoint):
    """Half of the solids (elastic, sand, von Mises, box-yield; a liquid box
    carries the loss) start with
    s2 < s0/4, so that the forward's FP64 redo of the return map and of the
    stress, and the adjoint's FP64 passes (plastic-return adjoint, stress
    adjoint), all run; forward state, action gradient and dL/d(x0, v0, F0)
    against the oracle."""
    from parity import ill_conditioned_solids
    sc = scenes.tiny(n_particles=160, n_grid=16, steps=6, seed=5,
                     kinds=(scenes.ELASTIC, scenes.LIQUID, scenes.SAND, scenes.VONMISES, scenes.BOX))
    n_ill = ill_conditioned_solids(sc, 0)
    say(f"ill-conditioned solids: {n_ill} of {sc.n} particles, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=4, adjoint=adjoint)
    sim.step(sc.horizon)
    compare_states(sim.state_numpy(), oracle_state(sc, sc.horizon), liquid_mask(sc), tol_x=1e-6, tol=1e-4,
                   tol_FJ=1e-5, n_grid=sc.n_grid)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    ga = ga[:, 0].double().cpu().numpy()
    p = O.params_from_scene(sc)
    st0 = O.state_from_scene(sc, requires_grad=True)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st = O.rollout(sc, state=st0, params=p, actions=acts)
    L = O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma)
    L.backward()
    ea = rel(ga, acts.grad.numpy())
    ex = rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy())
    ev = rel(g0[3:6].T.double().cpu().numpy(), st0["v"].grad.numpy())
    solid = ~liquid_mask(sc)
    gF = g0[15:24].T.double().cpu().numpy().reshape(-1, 3, 3)[solid]
    eF = rel(gF, st0["F"].grad.numpy()[solid])
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; actions {ea:.2e} dL/dx0 {ex:.2e} dL/dv0 {ev:.2e} "
        f"dL/dF0 {eF:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert ea <= 1e-4 and ex <= 1e-4 and ev <= 1e-4 and eF <= 1e-4


def test_von_mises_forward_vs_oracle():
    """The ice cream yields under a random velocity field (most particles
    return to the yield surface); 20 steps against the oracle."""
    sc = _ice_cream_scene(20)
    say("von Mises ice cream, 20 steps")
    sim = sim_of(sc)
    sim.step(20)
    compare_states(sim.state_numpy(), oracle_state(sc, 20), liquid_mask(sc), tol_x=1e-5, tol=2e-3)


@pytest.mark.parametrize("adjoint", ["tiled", "plain"])
def test_von_mises_gradient_vs_oracle(adjoint):
    sc = _ice_cream_scene(8, n=120, seed=6)
    say(f"von Mises gradient, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=3, adjoint=adjoint)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    p = O.params_from_scene(sc)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st0 = O.state_from_scene(sc, requires_grad=True)
    st = O.rollout(sc, actions=acts, state=st0, params=p)
    L = O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma)
    L.backward()
    ea = rel(ga[:, 0].double().cpu().numpy(), acts.grad.numpy())
    ex = rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy())
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; actions rel {ea:.2e}, dL/dx0 rel {ex:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert ea <= 1e-4 and ex <= 1e-4


# ---------------------------------------------------------------------------
# Box-yield plastic (section 3.2's plastic material)
# ---------------------------------------------------------------------------
def _plasticine_scene(steps, n=600, seed=7):
    return scenes.tiny(n_particles=n, n_grid=24, steps=steps, seed=seed,
                       kinds=(scenes.BOX, scenes.LIQUID), velocity=3.0, dt=1e-4)


def test_box_yield_forward_vs_oracle():
    sc = _plasticine_scene(20)
    say("Box-yield plastic, 20 steps")
    sim = sim_of(sc)
    sim.step(20)
    compare_states(sim.state_numpy(), oracle_state(sc, 20), liquid_mask(sc), tol_x=1e-5, tol=2e-3)


@pytest.mark.parametrize("adjoint", ["tiled", "plain"])
def test_box_yield_gradient_vs_oracle(adjoint):
    sc = _plasticine_scene(8, n=120, seed=8)
    say(f"Box-yield gradient, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=3, adjoint=adjoint)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    p = O.params_from_scene(sc)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st0 = O.state_from_scene(sc, requires_grad=True)
    st = O.rollout(sc, actions=acts, state=st0, params=p)
    L = O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma)
    L.backward()
    ea = rel(ga[:, 0].double().cpu().numpy(), acts.grad.numpy())
    ex = rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy())
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; actions rel {ea:.2e}, dL/dx0 rel {ex:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert ea <= 1e-4 and ex <= 1e-4


# ---------------------------------------------------------------------------
# launch shapes, extreme sizes and degenerate inputs
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("threads,part_wgs,grid_wgs,share", [(128, 512, 512, 1), (256, 4096, 2048, 2),
                                                              (256, 1024, 1024, 0), (256, 2048, 512, 1),
                                                              (512, 1024, 1024, 1)])
def test_config2_launch_shapes_vs_oracle(threads, part_wgs, grid_wgs, share):
    """Every launch shape the autotuner can pick gives the oracle's answer
    (config 2 at full size, 3 steps), with blocks of more than `share`
    chunks shared by two workgroups (0: never)."""
    sc = scenes.config2()
    say(f"config 2, launch shape {threads} threads, {part_wgs} particle / {grid_wgs} grid workgroups, "
        f"share above {share} chunks")
    sim = sim_of(sc)
    sim.set_option(_lib.MPM_OPT_PART_THREADS, threads)
    sim.set_option(_lib.MPM_OPT_PART_WGS, part_wgs)
    sim.set_option(_lib.MPM_OPT_GRID_WGS, grid_wgs)
    sim.set_option(_lib.MPM_OPT_SHARE_CHUNKS, share)
    sim.step(3)
    compare_states(sim.state_numpy(), oracle_state(sc, 3), liquid_mask(sc), tol_x=1e-6, tol=1e-3)


def test_single_particle():
    """One particle (a single block, a single lane): free fall with the
    oracle's answer."""
    sc = scenes.tiny(n_particles=1, n_grid=16, steps=5, seed=9, kinds=(scenes.ELASTIC,), with_cylinder=False)
    say("single particle, 5 steps")
    sim = sim_of(sc)
    sim.step(5)
    g, ref = sim.state_numpy(), oracle_state(sc, 5)
    ex, ev = rel(g["x"], ref["x"]), rel(g["v"], ref["v"])
    # C and F - I are round-off on both sides (uniform velocity), so they are
    # compared in absolute terms against the velocity gradient scale |v| / dx
    scale = np.abs(ref["v"]).max() * sc.n_grid
    eC = np.abs(g["C"] - ref["C"]).max() / scale
    eF = np.abs(g["F"] - ref["F"]).max()
    say(f"  rel err x {ex:.2e} v {ev:.2e}; |C - C_ref| / (|v|/dx) {eC:.2e}, |F - F_ref| {eF:.2e}")
    assert ex <= 1e-6 and ev <= 1e-5 and eC <= 1e-5 and eF <= 1e-6


def test_config5_largest_scene_first_steps_vs_oracle():
    """The largest single scene (config 5: 1M sand particles on 256^3, in
    floor contact), 2 steps against the oracle."""
    sc = scenes.config5(steps=2)
    say("config 5 (1M particles, 256^3), 2 steps")
    sim = sim_of(sc)
    sim.step(2)
    compare_states(sim.state_numpy(), oracle_state(sc, 2), liquid_mask(sc), tol_x=1e-6, tol=1e-3)


@pytest.mark.parametrize("adjoint", ["tiled"])
def test_long_horizon_pose_chunks_vs_oracle(adjoint):
    """300 steps: the manipulator poses are formed in chunks of 256 steps and
    their adjoint in chunks of 128, so both carry across chunk boundaries;
    loss and action gradient against the oracle."""
    sc = scenes.tiny(n_particles=90, n_grid=16, steps=300, seed=4, velocity=0.05)
    say(f"long horizon: {sc.horizon} steps, {adjoint} adjoint")
    sim = sim_of(sc, requires_grad=True, ckpt_every=50, adjoint=adjoint)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga = sim.backward(g[0:3], torch.zeros_like(g[0:3]))[:, 0].double().cpu().numpy()
    L, gref = O.loss_and_action_grad(sc)
    e = rel(ga, gref.numpy())
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; grad rel err {e:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert e <= 3e-4   # (1.0e-4 measured: FP32 over 300 steps)


def test_records_of_every_step_vs_oracle():
    """ckpt_every = 0: the forward keeps a block-sorted record of every step
    and the backward recomputes nothing.  The rollout runs in three calls
    (3 + 1 + 4 steps), so that the row maps across call boundaries are used;
    loss, action gradient and dL/d(x0, v0) against the oracle, and the plain
    adjoint and sample logging are refused for such a context."""
    sc = scenes.tiny(n_particles=90, n_grid=16, steps=8, seed=1)
    say("records of every step: 8 steps in calls of 3, 1 and 4")
    sim = sim_of(sc, requires_grad=True, ckpt_every=0)
    for n in (3, 1, 4):
        sim.step(n)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    ga = ga[:, 0].double().cpu().numpy()
    p = O.params_from_scene(sc)
    st0 = O.state_from_scene(sc, requires_grad=True)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st = O.rollout(sc, state=st0, params=p, actions=acts)
    L = O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma)
    L.backward()
    ea = rel(ga, acts.grad.numpy())
    ex = rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy())
    ev = rel(g0[3:6].T.double().cpu().numpy(), st0["v"].grad.numpy())
    say(f"  loss gpu {loss.item():.8f} ref {L.item():.8f}; actions {ea:.2e} dL/dx0 {ex:.2e} dL/dv0 {ev:.2e}")
    assert abs(loss.item() - L.item()) <= 1e-5 * abs(L.item())
    assert ea <= 1e-4 and ex <= 1e-4 and ev <= 1e-4
    with pytest.raises(RuntimeError):
        sim.set_option(_lib.MPM_OPT_ADJOINT, 1)
    buf = torch.zeros(16, 9, dtype=torch.float32, device=sim.device)
    count = torch.zeros(1, dtype=torch.int64, device=sim.device)
    with pytest.raises(_lib.MpmError) as e:
        sim.log_samples(buf, count)
    assert e.value.status == _lib.MPM_ESTATE


@pytest.mark.parametrize("threads,share", [(128, 2), (256, 0), (256, 1), (256, 2), (512, 2)])
def test_deferred_particles_over_several_chunks_vs_oracle(threads, share):
    """Blocks of several chunks whose ill-conditioned solids are left to the
    chunk's FP64 pass: the tile box and the float tile grow over both passes
    of every chunk, and the last pass publishes (every launch shape, blocks
    shared by two workgroups and not).  Tolerances: those of the
    ill-conditioned gradient test's forward state."""
    from parity import ill_conditioned_solids
    sc = scenes.tiny(n_particles=4001, n_grid=16, steps=4, seed=7,
                     kinds=(scenes.ELASTIC, scenes.LIQUID, scenes.SAND, scenes.VONMISES, scenes.BOX))
    n_ill = ill_conditioned_solids(sc, 0)
    assert n_ill > 1000
    sim = sim_of(sc)
    sim.set_option(2, threads)
    sim.set_option(7, share)
    sim.step(sc.horizon)
    say(f"{n_ill} ill-conditioned of {sc.n} particles, {threads} threads, share {share}")
    compare_states(sim.state_numpy(), oracle_state(sc, sc.horizon), liquid_mask(sc), tol_x=1e-6, tol=1e-4,
                   tol_FJ=1e-5, n_grid=sc.n_grid)


@pytest.mark.parametrize("ckpt", [0, 3])
def test_gradient_deferred_particles_over_several_chunks_vs_oracle(ckpt):
    """The same blocks through the tiled adjoint, records kept and recomputed:
    the FP64 second passes of several chunks and the velocity-adjoint tile
    that grows over them.  Tolerances: those of the ill-conditioned gradient
    test."""
    from parity import ill_conditioned_solids
    sc = scenes.tiny(n_particles=4001, n_grid=16, steps=4, seed=7,
                     kinds=(scenes.ELASTIC, scenes.LIQUID, scenes.SAND, scenes.VONMISES, scenes.BOX))
    assert ill_conditioned_solids(sc, 0) > 1000
    sim = sim_of(sc, requires_grad=True, ckpt_every=ckpt)
    sim.step(sc.horizon)
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    p = O.params_from_scene(sc)
    st0 = O.state_from_scene(sc, requires_grad=True)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st = O.rollout(sc, state=st0, params=p, actions=acts)
    O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma).backward()
    e = {"actions": rel(ga[:, 0].double().cpu().numpy(), acts.grad.numpy()),
         "x": rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy()),
         "v": rel(g0[3:6].T.double().cpu().numpy(), st0["v"].grad.numpy()),
         "C": rel(g0[6:15].T.double().cpu().numpy().reshape(-1, 3, 3), st0["C"].grad.numpy())}
    say(f"deferred particles, ckpt {ckpt}: " + " ".join(f"{k} {v:.2e}" for k, v in e.items()))
    assert max(e.values()) <= 1e-4


@pytest.mark.parametrize("n,grid,dt,wgs,share,grad", [(4001, 16, 2e-4, 2048, 2, True), (12001, 32, 2e-4, 64, 2, True),
                                                      (12001, 32, 2e-4, 64, 1, False), (4001, 16, 2e-4, 64, 0, False),
                                                      (20001, 128, 5e-5, 2048, 2, False)])
def test_shared_blocks_vs_oracle(n, grid, dt, wgs, share, grad):
    """Blocks shared by one workgroup per chunk (up to 7 chunks, more than a
    block's most entries), by two (a list longer than the workgroups), by
    none, and more blocks than one tile of the scan holds; forward, and the
    adjoint over the shared records.  Tolerances: those of the tests above."""
    sc = scenes.tiny(n_particles=n, n_grid=grid, steps=4, seed=7, dt=dt,
                     kinds=(scenes.ELASTIC, scenes.LIQUID, scenes.SAND, scenes.VONMISES, scenes.BOX))
    sim = sim_of(sc, requires_grad=grad, **({"ckpt_every": 0} if grad else {}))
    sim.set_option(3, wgs)
    sim.set_option(7, share)
    sim.step(sc.horizon)
    compare_states(sim.state_numpy(), oracle_state(sc, sc.horizon), liquid_mask(sc), tol_x=1e-6, tol=1e-4,
                   tol_FJ=1e-5, n_grid=sc.n_grid)
    if not grad:
        return
    loss, g = sim.loss_blob(sc.target_mu, sc.target_sigma)
    ga, g0 = sim.backward(g[0:3], torch.zeros_like(g[0:3]), want_grad0=True)
    p = O.params_from_scene(sc)
    st0 = O.state_from_scene(sc, requires_grad=True)
    acts = torch.tensor(sc.actions, dtype=torch.float64, requires_grad=True)
    st = O.rollout(sc, state=st0, params=p, actions=acts)
    O.blob_loss(st["x"], p.kind == O.LIQUID, torch.tensor(sc.target_mu, dtype=torch.float64), sc.target_sigma).backward()
    ea = rel(ga[:, 0].double().cpu().numpy(), acts.grad.numpy())
    ex = rel(g0[0:3].T.double().cpu().numpy(), st0["x"].grad.numpy())
    say(f"  shared blocks, {wgs} workgroups: actions {ea:.2e} dL/dx0 {ex:.2e}")
    assert ea <= 1e-4 and ex <= 1e-4


@pytest.mark.parametrize("n", [3, 64, 65, 1023, 1024, 1025, 2050])
def test_import_and_export_at_wavefront_and_table_edges_vs_oracle(n):
    """Particle counts around a wavefront's records and the import's key
    table (1024 particles a workgroup), three kinds; one call of two steps and
    a second call from its result; the rows the kernels do not carry (a
    liquid's F, a solid's J) stay the user's."""
    sc = scenes.tiny(n_particles=n, n_grid=24, steps=4, seed=3)
    liq = liquid_mask(sc)
    sc.F[liq] += 0.25
    sc.J[~liq] = 3.0
    sim = sim_of(sc)
    sim.step(2)
    sim.step(2)
    g = sim.state_numpy()
    assert np.array_equal(g["F"][liq], np.asarray(sc.F, np.float32)[liq])
    assert np.array_equal(g["J"][~liq], np.asarray(sc.J, np.float32)[~liq])
    compare_states(g, oracle_state(sc, 4), liq, tol_x=1e-6, tol=1e-4, tol_FJ=1e-5, n_grid=sc.n_grid)
