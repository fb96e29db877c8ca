"""GPU adjoint (checkpointed recompute + transposed gather + BGK VJP) against
the oracle's discrete adjoint, complex-step and finite differences."""
import numpy as np
import pytest

import oracle
from gpu_common import rel_l2, say, tol_fp32
from synth import jittered_lattice, tgv_initial_velocity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _setup(n_side=10, K=20, m=3, mode=0, seed=21):
    c = jittered_lattice(n_side, seed=seed, length=float(n_side))
    u0x, u0y = tgv_initial_velocity(c.x, c.y, float(n_side), 0.02)
    tx, ty = tgv_initial_velocity(c.x, c.y, float(n_side), 0.015)
    return c, u0x, u0y, tx, ty, K, m, mode


def _gpu_grad(plan, u0x, u0y, tx, ty, steps, segment, store_all=False):
    from paper_2306_01525_amd.autograd import Rollout
    ro = Rollout(plan, steps, segment, store_all)
    ro.forward(u0x, u0y)
    J = ro.loss(tx, ty)
    gx, gy, gt = ro.backward()
    return float(J.item()), gx.cpu().numpy(), gy.cpu().numpy(), float(gt.item())


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("precision", [1, 0])
def test_adjoint_on_imported_weights(mode, precision):
    """Same weights on both sides: FP64 GPU gradient to 1e-10, FP32 to 2e-6
    (12 steps; measured 5.2e-7 for the u0 gradient and J, 1.2e-7 for tau)."""
    from paper_2306_01525_amd import Params, Plan
    c, u0x, u0y, tx, ty, K, m, _ = _setup(mode=mode)
    tau, steps, seg = 0.7, 12, 5
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    J_o, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
    p = Params(dx=1.0, K=K, degree=m, tau=tau, stencil_mode=mode, precision=precision,
               with_adjoint=1)
    plan = Plan.from_arrays(c.x, c.y, nbr, own, W, p)
    J, gx, gy, gt = _gpu_grad(plan, u0x, u0y, tx, ty, steps, seg)
    tol = 1e-10 if precision == 1 else 2e-6
    eg = rel_l2(np.concatenate([gx, gy]), np.concatenate([gx_o, gy_o]))
    say("mode %d prec %d: J %.6e vs %.6e, grad u0 rel %.2e, dtau %.6e vs %.6e"
        % (mode, precision, J, J_o, eg, gt, gt_o))
    assert abs(J - J_o) <= tol * abs(J_o)
    assert eg < tol
    assert abs(gt - gt_o) <= tol * abs(gt_o) + 1e-300
    plan.close()


@pytest.mark.parametrize("precision", [1, 0])
def test_stored_rollout_equals_checkpointed_and_oracle(precision):
    """store_all (every pre-collision state kept by the forward, nothing
    recomputed) against the oracle's discrete adjoint within the bounds of
    the imported-weights test, and against checkpointed rollouts of segment
    lengths 1, 5 (ragged: 13 = 5 + 5 + 3) and 13."""
    from paper_2306_01525_amd import Params, Plan
    c, u0x, u0y, tx, ty, K, m, mode = _setup(seed=31)
    tau, steps = 0.75, 13
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    J_o, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
    p = Params(dx=1.0, K=K, degree=m, tau=tau, stencil_mode=mode, precision=precision,
               with_adjoint=1)
    plan = Plan.from_arrays(c.x, c.y, nbr, own, W, p)
    J, gx, gy, gt = _gpu_grad(plan, u0x, u0y, tx, ty, steps, 1, store_all=True)
    tol = 1e-10 if precision == 1 else 2e-6
    eg = rel_l2(np.concatenate([gx, gy]), np.concatenate([gx_o, gy_o]))
    say("stored, prec %d: J %.6e vs %.6e, grad u0 rel %.2e, dtau %.6e vs %.6e"
        % (precision, J, J_o, eg, gt, gt_o))
    assert abs(J - J_o) <= tol * abs(J_o)
    assert eg < tol
    assert abs(gt - gt_o) <= tol * abs(gt_o)
    for seg in (1, 5, steps):
        Jc, gxc, gyc, gtc = _gpu_grad(plan, u0x, u0y, tx, ty, steps, seg)
        d = max(np.abs(gx - gxc).max(), np.abs(gy - gyc).max()) / np.abs(
            np.concatenate([gx, gy])).max()
        say("segment %d: J diff %.2e, grad u0 max diff %.2e, dtau diff %.2e"
            % (seg, abs(J - Jc), d, abs(gt - gtc)))
        assert abs(J - Jc) <= 1e-14 * abs(J)
        assert d <= (1e-13 if precision == 1 else 1e-6)
        assert abs(gt - gtc) <= (1e-13 if precision == 1 else 1e-6) * abs(gt)
    plan.close()


def test_adjoint_end_to_end_gpu_build_and_autograd():
    """GPU-built weights, autograd.Function, against the oracle gradient and
    central finite differences of the GPU forward in FP64."""
    from paper_2306_01525_amd import Params, Plan
    from paper_2306_01525_amd.autograd import rollout_loss
    c, u0x, u0y, tx, ty, K, m, mode = _setup(n_side=14, K=25, m=2, seed=5)
    steps, seg = 20, 8
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    J_o, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, 0.8, steps, 1.0, u0x, u0y, tx, ty)
    p = Params(dx=1.0, K=K, degree=m, tau=0.8, stencil_mode=mode, precision=1, with_adjoint=1)
    plan = Plan.build(c.x, c.y, c.period, p)
    dev = torch.device("cuda")
    ux = torch.tensor(u0x, device=dev, requires_grad=True)
    uy = torch.tensor(u0y, device=dev, requires_grad=True)
    tau = torch.tensor(0.8, dtype=torch.float64, device=dev, requires_grad=True)
    txt, tyt = torch.tensor(tx, device=dev), torch.tensor(ty, device=dev)
    J = rollout_loss(plan, ux, uy, tau, steps, txt, tyt, seg)
    J.backward()
    eg = rel_l2(np.concatenate([ux.grad.cpu().numpy(), uy.grad.cpu().numpy()]),
                np.concatenate([gx_o, gy_o]))
    say("e2e: J %.8e vs oracle %.8e; grad rel %.2e; dtau %.8e vs %.8e"
        % (J.item(), J_o, eg, tau.grad.item(), gt_o))
    assert abs(J.item() - J_o) < 1e-8 * abs(J_o)
    assert eg < 1e-7
    assert abs(tau.grad.item() - gt_o) < 1e-7 * abs(gt_o)
    # the same through the autograd function with every state stored
    ux2 = torch.tensor(u0x, device=dev, requires_grad=True)
    uy2 = torch.tensor(u0y, device=dev, requires_grad=True)
    tau2 = torch.tensor(0.8, dtype=torch.float64, device=dev, requires_grad=True)
    rollout_loss(plan, ux2, uy2, tau2, steps, txt, tyt, seg, store_all=True).backward()
    for a, b in ((ux2.grad, ux.grad), (uy2.grad, uy.grad), (tau2.grad, tau.grad)):
        assert float((a - b).abs().max()) <= 1e-13 * float(b.abs().max())
    # central finite difference of the GPU forward with respect to tau
    h = 1e-5
    with torch.no_grad():
        jp = rollout_loss(plan, ux, uy, torch.tensor(0.8 + h, dtype=torch.float64), steps,
                          txt, tyt, seg).item()
        jm = rollout_loss(plan, ux, uy, torch.tensor(0.8 - h, dtype=torch.float64), steps,
                          txt, tyt, seg).item()
    fd = (jp - jm) / (2 * h)
    say("fd dJ/dtau %.8e vs adjoint %.8e" % (fd, tau.grad.item()))
    assert abs(fd - tau.grad.item()) < 1e-5 * abs(fd)
    plan.close()


def test_two_rollouts_at_different_tau_each_differentiate_at_their_own():
    """Two losses on one plan at different tau, both formed before either
    backward: each gradient equals the oracle's discrete adjoint at its own
    tau (the recomputation must not use whatever tau the plan holds by then),
    and the plan keeps the tau set last."""
    from paper_2306_01525_amd import Params, Plan
    from paper_2306_01525_amd.autograd import rollout_loss
    c, u0x, u0y, tx, ty, K, m, mode = _setup(n_side=12, K=20, m=3, seed=7)
    steps, seg = 15, 6
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    p = Params(dx=1.0, K=K, degree=m, tau=0.8, stencil_mode=mode, precision=1, with_adjoint=1)
    plan = Plan.build(c.x, c.y, c.period, p)
    dev = torch.device("cuda")
    txt, tyt = torch.tensor(tx, device=dev), torch.tensor(ty, device=dev)
    runs = []
    for tau in (0.8, 0.95):
        ux = torch.tensor(u0x, device=dev, requires_grad=True)
        uy = torch.tensor(u0y, device=dev, requires_grad=True)
        tt = torch.tensor(tau, dtype=torch.float64, device=dev, requires_grad=True)
        runs.append((tau, ux, uy, tt, rollout_loss(plan, ux, uy, tt, steps, txt, tyt, seg)))
    for tau, ux, uy, tt, J in runs:          # the first loss is differentiated after the second forward
        J.backward()
        J_o, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
        eg = rel_l2(np.concatenate([ux.grad.cpu().numpy(), uy.grad.cpu().numpy()]),
                    np.concatenate([gx_o, gy_o]))
        say("tau %.2f: J %.8e vs %.8e, grad rel %.2e, dtau %.8e vs %.8e"
            % (tau, J.item(), J_o, eg, tt.grad.item(), gt_o))
        assert abs(J.item() - J_o) < 1e-10 * abs(J_o)
        assert eg < 1e-10
        assert abs(tt.grad.item() - gt_o) < 1e-10 * abs(gt_o)
        assert plan.params.tau == 0.95
    plan.close()


def _adjoint_draw(count=8, seed=77):
    r = np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(count):
        m = int(r.integers(2, 5))
        M = (m + 1) * (m + 2) // 2
        n_side = int(r.integers(8, 17))
        K = int(r.integers(M + 6, min(48, 64 - M, n_side * n_side - 1) + 1))
        out.append(dict(n_side=n_side, K=K, m=m, mode=int(r.integers(0, 2)),
                        tau=float(r.uniform(0.55, 1.2)), steps=int(r.integers(6, 15)),
                        seg=int(r.integers(2, 6)), seed=int(r.integers(1, 10_000))))
    return out


ADJ_CASES = _adjoint_draw()


@pytest.mark.parametrize("case", ADJ_CASES, ids=["n%d-K%d-m%d-mode%d-s%d" % (
    c["n_side"], c["K"], c["m"], c["mode"], c["steps"]) for c in ADJ_CASES])
@pytest.mark.parametrize("precision", [1, 0])
def test_adjoint_sweep_against_oracle(case, precision):
    """Seeded random stencil sizes, degrees, rules, relaxation times, step
    counts and checkpoint intervals, on the oracle's weights: FP64 to 1e-10.
    In FP32, J and its gradient come from the misfit u(T) - u*, so the
    rounding of u is amplified by |u*| / |u(T) - u*| (from 2 to 84 here); the
    bound is tol_fp32(steps) times that ratio plus one (measured: at most 0.28
    of it, 1e-7 to 2e-7 per unit of the ratio)."""
    from paper_2306_01525_amd import Params, Plan
    c, u0x, u0y, tx, ty, K, m, mode = _setup(n_side=case["n_side"], K=case["K"], m=case["m"],
                                             mode=case["mode"], seed=case["seed"])
    tau, steps, seg = case["tau"], case["steps"], case["seg"]
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    J_o, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
    p = Params(dx=1.0, K=K, degree=m, tau=tau, stencil_mode=mode, precision=precision,
               with_adjoint=1)
    plan = Plan.from_arrays(c.x, c.y, nbr, own, W, p)
    J, gx, gy, gt = _gpu_grad(plan, u0x, u0y, tx, ty, steps, seg)
    ratio = float(np.sqrt((tx ** 2 + ty ** 2).sum() / (2.0 * J_o)))
    tol = 1e-10 if precision == 1 else tol_fp32(steps) * (ratio + 1.0)
    eg = rel_l2(np.concatenate([gx, gy]), np.concatenate([gx_o, gy_o]))
    say("%s prec %d: J rel %.2e, grad u0 rel %.2e, dtau rel %.2e (misfit ratio %.1f, tol %.1e)"
        % (case, precision, abs(J - J_o) / abs(J_o), eg, abs(gt - gt_o) / abs(gt_o), ratio, tol))
    assert abs(J - J_o) <= tol * abs(J_o)
    assert eg < tol
    assert abs(gt - gt_o) <= tol * abs(gt_o)
    assert plan.device_error() == 0
    plan.close()


# (nodes a row, rows, K, degree, mode): whole, partly filled and missing groups of
# 64 nodes in the last tile; seven, four and eleven triples of row entries; and a
# size on each side of the line between the small and the large workgroups
REVERSED_CASES = [(8, 8, 20, 3, 0), (9, 13, 12, 2, 1), (16, 17, 20, 3, 0), (33, 31, 30, 4, 0),
                  (221, 222, 12, 2, 0), (222, 222, 12, 2, 0)]


@pytest.mark.parametrize("case", REVERSED_CASES, ids=["%dx%d-K%d-mode%d" % (
    c[0], c[1], c[2], c[4]) for c in REVERSED_CASES])
@pytest.mark.parametrize("precision", [1, 0])
def test_several_reversed_steps_equal_single_ones_and_oracle(case, precision):
    """steps_adjoint, in one call and cut in two, gives the adjoint of single
    reversed steps bit for bit, whose sums of dJ/dtau it takes in another order:
    at most some 40 roundings of 1.1e-16 deep, with terms up to a hundred times
    the partial sums, 1e-12 of these. The gradient meets the oracle's within the
    bounds of the imported-weights test; so does dJ/dtau in FP64, while in FP32 it
    is a difference of populations that shrinks with the spacing over the
    wavelength and has no bound of that kind (49,062 nodes: 1.9e-5)."""
    from paper_2306_01525_amd import Params, Plan
    nx, ny, K, m, mode = case
    c = jittered_lattice(nx, seed=nx, length=float(nx), ny=ny, length_y=float(ny))
    u0x, u0y = tgv_initial_velocity(c.x, c.y, float(nx), 0.02)
    tx, ty = tgv_initial_velocity(c.x, c.y, float(nx), 0.015)
    tau, steps = 0.7, 3
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    p = Params(dx=1.0, K=K, degree=m, tau=tau, stencil_mode=mode, precision=precision,
               with_adjoint=1)
    plan = Plan.from_arrays(c.x, c.y, nbr, own, W, p)
    rec = torch.empty((steps + 1, 9, c.n), dtype=plan.state_dtype, device="cuda")
    plan.init_f(u0x, u0y, f=rec[0])
    plan.step_record(plan.collide(rec[0]), plan.new_state(), steps, rec[1:])
    seed, _ = plan.loss_seed(rec[steps], tx, ty)
    dtau = torch.zeros(1, dtype=torch.float64, device="cuda")
    lam, other = seed.clone(), torch.empty_like(seed)
    for t in reversed(range(steps)):
        plan.step_adjoint(rec[t], lam, other, dtau)
        lam, other = other, lam
    one, _, parts = plan.steps_adjoint(rec, steps, seed.clone(), torch.empty_like(seed))
    a, b, cut = plan.steps_adjoint(rec[1:], steps - 1, seed.clone(), torch.empty_like(seed))
    a, b, cut = plan.steps_adjoint(rec, 1, a, b, cut)
    assert torch.equal(one, lam) and torch.equal(a, lam)
    assert torch.equal(parts, cut)
    total = plan.adjoint_tau(parts, torch.zeros_like(dtau))
    scale = float(parts.abs().sum())
    say("reversed %s prec %d: dtau %.15e, single steps %.15e" % (case, precision, float(total),
                                                              float(dtau)))
    assert abs(float(total) - float(dtau)) <= 1e-12 * scale
    _, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
    gx, gy = plan.init_adjoint(u0x, u0y, a)
    tol = 1e-10 if precision == 1 else 2e-6
    eg = rel_l2(np.concatenate([gx.cpu().numpy(), gy.cpu().numpy()]),
                np.concatenate([gx_o, gy_o]))
    assert eg < tol
    if precision == 1:
        assert abs(float(total) - gt_o) <= tol * abs(gt_o)
    plan.close()


@pytest.mark.parametrize("order", ["lattice", "scattered"])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("precision", [1, 0])
def test_imported_stencils_may_repeat_a_member(precision, mode, order):
    """Members repeated in every stencil, the weight split between the places: a
    transposed row then holds an arriving node several times. In lattice order the
    tiles have inverse halos; with the nodes numbered at random a tile's 256 nodes
    are read from all over the cloud, more than an inverse halo holds, and rows are
    gathered from global memory. Gradient against the oracle's on the same stencils
    within the bounds of the imported-weights test."""
    from paper_2306_01525_amd import Params, Plan
    c, u0x, u0y, tx, ty, K, m, _ = _setup(n_side=48, seed=29)
    nbr, own, W = oracle.build_plan(c, 1.0, K, m, mode)
    nbr = np.concatenate([nbr, nbr[:, [0, 5, 5]]], axis=1)
    W = np.concatenate([W, W[:, :, [0, 5, 5]]], axis=2)
    W[:, :, 0] *= 0.25
    W[:, :, K] *= 0.75
    W[:, :, 5] *= 0.5
    W[:, :, K + 1:] *= 0.25
    if order == "scattered":
        at = np.random.Generator(np.random.PCG64(8)).permutation(c.n)   # new index of a node
        old = np.argsort(at)
        nbr, own, W = at[nbr[old]], at[own[old]], W[old]
        u0x, u0y, tx, ty = u0x[old], u0y[old], tx[old], ty[old]
        c.x, c.y = c.x[old], c.y[old]
    tau, steps = 0.7, 3
    _, gx_o, gy_o, gt_o = oracle.adjoint(nbr, own, W, tau, steps, 1.0, u0x, u0y, tx, ty)
    plan = Plan.from_arrays(c.x, c.y, nbr, own, W,
                            Params(dx=1.0, K=K + 3, degree=m, tau=tau, stencil_mode=mode,
                                   precision=precision, with_adjoint=1))
    halos = plan.export("tdescT")
    say("%s mode %d prec %d: inverse halos of %d to %d nodes" % (order, mode, precision,
                                                              halos.min(), halos.max()))
    assert (halos == 0).all() if order == "scattered" else (halos > 0).all()
    J, gx, gy, gt = _gpu_grad(plan, u0x, u0y, tx, ty, steps, 2)
    eg = rel_l2(np.concatenate([gx, gy]), np.concatenate([gx_o, gy_o]))
    say("  grad u0 rel %.2e, dtau %.6e vs %.6e" % (eg, gt, gt_o))
    assert eg < (1e-10 if precision == 1 else 2e-6)
    if precision == 1:
        assert abs(gt - gt_o) <= 1e-10 * abs(gt_o)
    assert plan.device_error() == 0
    plan.close()


def test_an_empty_first_call_of_reversed_steps_clears_the_sums():
    """steps_adjoint of no steps leaves the adjoint in place and its parts zero,
    whatever their memory held; a later call adds to them, bit for bit what one
    call gives. A negative count is refused by name."""
    import ctypes
    from paper_2306_01525_amd import MLBMError, Params, Plan, _lib
    c, u0x, u0y, tx, ty, K, m, mode = _setup(n_side=17, seed=3)
    plan = Plan.build(c.x, c.y, c.period, Params(dx=1.0, K=K, degree=m, tau=0.8, precision=1,
                                                 with_adjoint=1))
    f = plan.init_f(u0x, u0y)
    rec = torch.stack([f, 1.01 * f])
    lam = torch.linspace(-1.0, 1.0, f.numel(), dtype=f.dtype, device="cuda").reshape(f.shape)
    ref, _, whole = plan.steps_adjoint(rec, 2, lam.clone(), torch.empty_like(f))
    parts = torch.full_like(whole, float("nan"))
    a, b = lam.clone(), torch.empty_like(f)
    rb = ctypes.c_int32(7)
    st = torch.cuda.current_stream().cuda_stream
    call = _lib.load().mlbm_steps_adjoint
    assert call(plan._h, rec.data_ptr(), 0, a.data_ptr(), b.data_ptr(), parts.data_ptr(), 1,
                ctypes.byref(rb), st) == 0
    assert rb.value == 0 and torch.equal(a, lam) and (parts == 0).all()
    got, _, parts = plan.steps_adjoint(rec, 2, a, b, parts)
    assert torch.equal(got, ref) and torch.equal(parts, whole)
    empty = plan.steps_adjoint(rec, 0, a, b)[2]
    assert float(plan.adjoint_tau(empty, torch.ones(1, dtype=torch.float64, device="cuda"))) == 1.0
    with pytest.raises(MLBMError, match="negative"):
        plan.steps_adjoint(rec, -1, a, b)
    plan.close()


# either side of the lines between the reversed step's workgroups of one, two and
# four groups of 64 nodes: FP64 20,480 and 36,864 nodes, or 49,152 for K 18 to 40;
# FP32 36,864, or 49,152 from K 24
GROUP_CASES = [(64, 64, 12, 2, 1), (143, 143, 12, 2, 0), (144, 143, 12, 2, 0), (192, 192, 12, 2, 1),
               (193, 192, 12, 2, 1), (193, 192, 24, 3, 0), (222, 222, 24, 3, 0),
               (193, 192, 41, 2, 1)]


@pytest.mark.parametrize("case", GROUP_CASES, ids=["%dx%d-K%d-mode%d" % (
    c[0], c[1], c[2], c[4]) for c in GROUP_CASES])
@pytest.mark.parametrize("precision", [1, 0])
def test_reversed_steps_on_either_side_of_the_lines(case, precision):
    """As the test of several reversed steps."""
    test_several_reversed_steps_equal_single_ones_and_oracle(case, precision)
