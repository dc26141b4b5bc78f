"""GPU parity: the HIP path, called through the C boundary, against the CPU oracle on the
same seeded inputs.  Integer state (periods, counters, due sets) must be bit-exact; fp32
parameters within relative 1e-4 after one step and 1e-3 over the run (bf16-operand
configurations within 2e-2), measured as max-abs difference over max-abs value and as
relative L2 error, per replica."""
import numpy as np
import pytest
import torch

import workloads
from paper_2509_03110_amd import lsam
from util import bn_away_from_zero, close_enough, oracle_from, rel_l2, rel_max

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def make_pair(w, init=None):
    init = workloads.init_params(w) if init is None else init
    cfg, keep = lsam.config_from_workload(w)
    return lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)


def to_dev(X, labels, w):
    Xd = torch.from_numpy(X).to(DEV)
    if w.gemm_dtype == 1 and not w.n_conv:      # the convolutional model takes fp32 images
        Xd = Xd.to(torch.bfloat16)
    return Xd.contiguous(), torch.from_numpy(labels).to(DEV)


def check_state(g, o, tol, what, tol_v=None):
    """Parameters, velocities and iterate sums of every replica plus the center, and the
    integer schedule state (bit-exact)."""
    worst = 0.0
    for i in list(range(o.K)) + [-1]:
        a, b = g.lsam_get_params(i), o.get_params(i)
        worst = max(worst, close_enough(a, b, tol, "%s: params of replica %d" % (what, i)))
    for i in range(o.K):
        for which, ref, name, t in ((lsam.BUF_VELOCITY, o.v[i], "v", tol_v or tol),
                                    (lsam.BUF_ITER_SUM, o.S[i], "S", tol)):
            a = g.lsam_get_buffer(which, i)
            if np.max(np.abs(ref)) == 0.0:
                assert np.max(np.abs(a)) == 0.0
                continue
            close_enough(a, ref, t, "%s: %s of replica %d" % (what, name, i))
    tau, cnt, ty = g.lsam_get_schedule()
    otau, ocnt, oty = o.get_schedule()
    assert (tau, cnt, ty) == (otau, ocnt, oty), what
    return worst


def anchor(g, o):
    """Restarts the GPU from the oracle's current state (rounded to fp32), so that the next
    step is compared from a common starting point."""
    for i in range(o.K):
        g.lsam_set_buffer(lsam.BUF_PARAMS, i, o.x[i])
        g.lsam_set_buffer(lsam.BUF_VELOCITY, i, o.v[i])
        g.lsam_set_buffer(lsam.BUF_ITER_SUM, i, o.S[i])
    g.lsam_set_buffer(lsam.BUF_PARAMS, -1, o.y)
    if o.gprev is not None:
        g.lsam_set_buffer(lsam.BUF_CENTER_DIR, -1, o.gprev)


def run_mlp(w, steps, tol1, tol_run, check_every=1, margin=False, tol_flip=5e-2,
            anchor_after=None, margin_ratio=None, min_margin=1e-3, fused=True, init_fn=None):
    """Runs GPU and oracle side by side.

    margin=True starts from parameters whose hidden pre-activations are far from zero, so no
    ReLU decision can differ between fp32 and float64: then gradients, velocities, sums and
    parameters must all agree to the tight tolerance, layer by layer.  With the natural
    initialisation a pre-activation within rounding distance of zero flips now and then
    (about one unit per replica-step at the cfg2 shape), each flip moving the gradient by
    ~1/sqrt(B*width) of its norm; parameters still have to meet the tight bound, velocities
    and gradients the looser tol_flip.  Flips also make two free-running trajectories drift
    apart (the dynamics amplify each one), so from step `anchor_after` on the GPU state is
    reset to the oracle's before every step and each step is held to the one-step bound tol1.
    margin_ratio: keep the workload's own step size and start with hidden biases that many
    standard deviations of the data-dependent part away from zero (the default margin
    initialisation uses 8 and needs the smaller step size 0.01 to keep its margin)."""
    if margin and margin_ratio is None:
        w = w.scaled(lr=0.01)     # slow enough that the margin survives the whole run
    if margin:
        init = workloads.init_params_margin(w, ratio=margin_ratio or 8.0)
    else:
        init = workloads.init_params(w)
    if init_fn is not None:
        init = init_fn(w, init)
    g, o = make_pair(w, init)
    fused_step = bool(g.lsam_set_fused_step(fused)) and w.rho != 0.0
    tol_v = None if margin else tol_flip
    loss_d = torch.zeros(w.K, dtype=torch.float32, device=DEV)
    worst = 0.0
    for t in range(steps):
        anchored = anchor_after is not None and t >= anchor_after
        if anchored:
            anchor(g, o)
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        g.lsam_step(Xd, ld, loss_d)
        ol = o.step(X, lab)
        if margin:
            assert o.model.last_margin > min_margin, "margin initialisation lost its margin"
        gl = loss_d.cpu().numpy()
        assert np.allclose(gl, ol, rtol=max(tol_run, 1e-5), atol=1e-6), (t, gl, ol)
        if t == 0:
            norms = g.lsam_get_norms()
            assert np.allclose(norms, o.last_norm, rtol=(tol1 if margin else tol_flip)), (norms, o.last_norm)
            for i in range(w.K):
                g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
                # with the fused step neither gradient of a weight matrix is ever stored (their
                # effect is checked through x~, v and x); the bias parts hold g2 as always
                if fused_step or margin:
                    for l, (o0, o1, o2) in enumerate(o.model.offsets):
                        t_g = tol1 if margin else tol_flip
                        if not fused_step:
                            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], t_g, "dW%d of replica %d" % (l + 1, i))
                        close_enough(g2[o1:o2], o.last_g2[i][o1:o2], t_g, "db%d of replica %d" % (l + 1, i))
                else:
                    close_enough(g2, o.last_g2[i], tol_flip, "g2 of replica %d" % i)
        ng, no = g.lsam_sync(), o.sync()
        assert ng == no, (t, ng, no)
        if t == 0:
            check_state(g, o, tol1, "%s step 1" % w.name, tol_v)
        elif (t + 1) % check_every == 0 or t == steps - 1:
            tol = tol1 if anchored else tol_run
            e = check_state(g, o, tol, "%s step %d" % (w.name, t + 1), tol_v)
            print("%s margin=%s step %d: worst parameter error %.3e" % (w.name, margin, t + 1, e))
            worst = max(worst, e)
    g.close()
    return worst


# ---- raw-vector mode: norm + perturb + descent + center ----------------------------------------
@pytest.mark.parametrize("d,K,tau", [(1000, 3, (2, 3, 4)), (4099, 2, (1, 2)), (65536 * 3 + 64, 4, None),
                                     (7, 1, (1,))])
@pytest.mark.parametrize("nesterov", [1, 0])
def test_raw_mode_matches_oracle(d, K, tau, nesterov):
    w = workloads.WORKLOADS["cfg4"].scaled(K=K, d_raw=d, tau=tau, nesterov=nesterov, steps=12,
                                           grad_std=1e-2)
    g, o = make_pair(w)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        norms = g.lsam_get_norms()
        assert np.allclose(norms, o.last_norm, rtol=1e-5)
        for i in range(K):
            xt = g.lsam_get_buffer(lsam.BUF_PERTURBED, i)
            assert rel_max(xt, o.last_perturbed[i]) < 1e-6
        assert g.lsam_sync() == o.sync()
        check_state(g, o, 1e-4, "raw d=%d step %d" % (d, t + 1))
    g.close()


def test_raw_mode_separate_initial_points_and_fixed_lambda():
    w = workloads.WORKLOADS["cfg4"].scaled(K=3, d_raw=2048, tau=(2, 2, 5), lambda_abs=0.7,
                                           beta=0.5, lr_center=0.8, momentum=0.5, steps=11)
    rng = np.random.default_rng(1)
    init = rng.standard_normal((w.K + 1) * w.d_raw).astype(np.float32)
    g, o = make_pair(w, init)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert g.lsam_sync() == o.sync()
    check_state(g, o, 1e-4, "raw separate init")
    a = g.lsam_get_buffer(lsam.BUF_CENTER_DIR, -1)
    assert rel_max(a, o.gprev) < 1e-4
    g.close()


def test_redraw_schedule_stays_bit_exact():
    w = workloads.WORKLOADS["cfg4"].scaled(K=5, d_raw=256, tau_min=1, tau_max=4, sched_seed=77,
                                           sched_mode=workloads.SCHED_REDRAW, steps=40)
    g, o = make_pair(w)
    z = torch.zeros(w.K, w.d_raw, device=DEV)
    for t in range(w.steps):
        g.lsam_step_grads(z, z)
        o.step_grads(np.zeros((w.K, w.d_raw)), np.zeros((w.K, w.d_raw)))
        assert g.lsam_sync() == o.sync()
        assert g.lsam_get_schedule() == o.get_schedule()
    g.close()


def test_set_scalars_changes_step_size_and_radius():
    w = workloads.WORKLOADS["cfg4"].scaled(K=2, d_raw=512, tau=(3, 3), steps=6)
    g, o = make_pair(w)
    for t in range(w.steps):
        lr, rho = 0.1 / np.sqrt(t + 1), 0.05 / np.sqrt(t + 1)   # the theorems' decaying schedules
        g.lsam_set_scalars(lr, rho)
        o.set_scalars(np.float32(lr), np.float32(rho))
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert g.lsam_sync() == o.sync()
    check_state(g, o, 1e-4, "decaying scalars")
    g.close()


# ---- fp32 MLP configurations ----------------------------------------------------------------------
@pytest.mark.parametrize("margin", [True, False])
def test_cfg1_twenty_steps(margin):
    w = workloads.WORKLOADS["cfg1"]
    worst = run_mlp(w, w.steps, 1e-4, 1e-3, margin=margin)
    print("cfg1 margin=%s worst relative error over 20 steps: %.3e" % (margin, worst))


@pytest.mark.parametrize("margin", [True, False])
def test_cfg2_fifty_steps(margin):
    w = workloads.WORKLOADS["cfg2"]
    worst = run_mlp(w, 12 if margin else w.steps, 1e-4, 1e-3, check_every=5, margin=margin,
                    anchor_after=None if margin else 10)
    print("cfg2 margin=%s worst relative error over 50 steps: %.3e" % (margin, worst))


def test_cfg2_free_running_at_its_own_step_size():
    """Config 2 at its own lr = 0.1, momentum 0.9, seeded periods, 22 steps with no reset of
    any kind: parameters, velocities, iterate sums and the center within 1e-4 after the first
    step and 1e-3 after 20 and more.  The initialisation keeps every hidden pre-activation at
    least 1e-2 away from zero over these steps (the oracle checks it each step), so that no
    ReLU decision depends on rounding."""
    w = workloads.WORKLOADS["cfg2"]
    worst = run_mlp(w, 22, 1e-4, 1e-3, check_every=5, margin=True, margin_ratio=32.0, min_margin=5e-3)
    print("cfg2 free-running, lr %.2f: worst relative error over 22 steps: %.3e" % (w.lr, worst))


def test_cfg2_natural_initialisation_free_running_error_is_reported():
    """The same 20 steps from the workload's own initialisation, free-running, where now and
    then a pre-activation within rounding distance of zero is rectified differently in fp32
    and in float64 and the dynamics (lr 0.1, momentum 0.9) amplify the difference.  Reported
    as relative L2 and worst-element error; held only to a loose bound (the per-step agreement
    of this run is what test_cfg2_fifty_steps and the attribution test below hold)."""
    w = workloads.WORKLOADS["cfg2"]
    g, o = make_pair(w)
    loss_d = torch.zeros(w.K, dtype=torch.float32, device=DEV)
    for t in range(20):
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        g.lsam_step(Xd, ld, loss_d)
        o.step(X, lab)
        assert g.lsam_sync() == o.sync()
        if t in (0, 4, 9, 14, 19):
            errs = [rel_max(g.lsam_get_params(i), o.get_params(i)) for i in list(range(w.K)) + [-1]]
            l2 = [rel_l2(g.lsam_get_params(i), o.get_params(i)) for i in list(range(w.K)) + [-1]]
            print("cfg2 natural init, free-running, step %d: worst-element error of x_i, y: %s; "
                  "relative L2: %s" % (t + 1, " ".join("%.2e" % e for e in errs),
                                       " ".join("%.2e" % e for e in l2)))
    assert max(errs) < 1e-1 and max(l2) < 1e-1
    assert g.lsam_get_schedule() == o.get_schedule()
    g.close()


def _hidden_mismatches(g, o, w, i, which_pass):
    """Hidden units of replica i whose ReLU decision differs between the GPU (activation read
    back) and the oracle: {(layer, sample, unit): (|z| of the oracle, magnitude |a||w| + |b| of
    the sum)}."""
    out = {}
    for l, (Z, mag) in enumerate(o.last_hidden[i][which_pass]):
        A = g.lsam_get_activation(l + 1, i)
        diff = (A > 0) != (Z > 0)
        for b, j in zip(*np.nonzero(diff)):
            out[(l + 1, int(b), int(j))] = (abs(Z[b, j]), mag[b, j])
    return out


@pytest.mark.parametrize("rho", [0.0, 0.05])
def test_cfg2_differences_come_from_relu_decisions_at_rounding_distance(rho):
    """What the allowance in the parity criterion rests on, tested at the config-2 shape with
    its own initialisation, every step started from the oracle's state:
      * a ReLU decision differs between the two sides only where the oracle's pre-activation is
        within a few fp32 roundings of zero (|z| <= 8 * 2^-24 * (|a||w| + |b|)) -- or, in the
        pass at the perturbed point, for the very unit and sample whose first-pass decision
        differed: that difference changes row j of g1 by dA[b,j] X[b], so x~ moves z~[b,j] by
        rho/||g1|| dA[b,j] |X[b]|^2, far more than rounding, while z~[b,j] is still near zero;
      * a replica-step in which all decisions agree meets the tight bound everywhere, gradient
        included, with no element excepted.
    The decisions of the pass at the perturbed point are read from the activations the step
    leaves behind.  Those of the first pass are read from a second context with rho = 0 that
    takes the same step from the same state: its single pass runs the same kernels on the same
    values as the first pass of the other and is deterministic."""
    w = workloads.WORKLOADS["cfg2"].scaled(rho=rho)
    g, o = make_pair(w)
    g0 = None
    if rho != 0.0:
        cfg0, keep0 = lsam.config_from_workload(w.scaled(rho=0.0))
        g0 = lsam.Lsam(cfg0, workloads.init_params(w), device=DEV, keep=keep0)
    o.model.keep_hidden = True
    loss_d = torch.zeros(w.K, dtype=torch.float32, device=DEV)
    clean = flipped = 0
    for t in range(8):
        anchor(g, o)
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        if g0 is not None:
            anchor(g0, o)
            g0.lsam_step(Xd, ld, loss_d)
        g.lsam_step(Xd, ld, loss_d)
        o.step(X, lab)
        for i in range(w.K):
            bad = _hidden_mismatches(g, o, w, i, 1)
            first = _hidden_mismatches(g0, o, w, i, 0) if g0 is not None else {}
            for where, (z, mag) in first.items():
                assert z <= 8 * 2.0 ** -24 * mag, ("first pass", t, i, where, z, mag)
            for where, (z, mag) in bad.items():
                assert z <= 8 * 2.0 ** -24 * mag or where in first, ("second pass", t, i, where, z, mag)
            bad.update(first)
            g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
            if not bad:
                clean += 1
                assert rel_max(g2, o.last_g2[i]) < 2e-5, (t, i)
                assert rel_max(g.lsam_get_params(i), o.get_params(i)) < 1e-6, (t, i)
                assert rel_max(g.lsam_get_buffer(lsam.BUF_VELOCITY, i), o.v[i]) < 2e-5, (t, i)
            else:
                flipped += 1
                close_enough(g2, o.last_g2[i], 5e-2, "g2 of replica %d at step %d" % (i, t))
        assert g.lsam_sync() == o.sync()
        if g0 is not None:
            g0.lsam_sync()
    print("rho=%g: %d replica-steps with all ReLU decisions equal (held to 2e-5 on every element), "
          "%d with a decision at rounding distance" % (rho, clean, flipped))
    assert clean >= 4
    g.close()
    if g0 is not None:
        g0.close()


@pytest.mark.parametrize("dims,B,K", [((50, 37, 19, 7), 5, 3), ((8, 3), 1, 1), ((100, 300, 10), 70, 2),
                                      ((24, 130, 260, 66, 5), 33, 2)])
def test_fp32_ragged_shapes(dims, B, K):
    w = workloads.WORKLOADS["cfg1"].scaled(name="ragged", K=K, dims=dims, batch=B, tau=(2,) * K,
                                           n_classes=dims[-1], steps=5, data_seed=9)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=False)


# ---- bf16-operand configurations at reduced width (same depth, K and schedule) ---------------------
@pytest.mark.parametrize("name,width,B", [("cfg3", 256, 32), ("cfg5", 128, 64)])
def test_bf16_reduced_shapes(name, width, B):
    full = workloads.WORKLOADS[name]
    dims = (full.dims[0] // 8,) + (width,) * (len(full.dims) - 2) + (full.dims[-1],)
    w = full.scaled(dims=dims, batch=B, steps=10)
    worst = run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
    print("%s reduced, margin init: worst relative error %.3e" % (name, worst))
    worst = run_mlp(w, w.steps, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=2)
    print("%s reduced: worst relative error %.3e" % (name, worst))
    # the same with the sampler step as a kernel of its own (g2 stored and compared)
    run_mlp(w, 4, 2e-2, 2e-2, margin=True, fused=False)


@pytest.mark.parametrize("name,width,B", [("cfg3", 256, 32), ("cfg5", 128, 64)])
def test_bf16_reduced_shapes_free_running_twenty_steps(name, width, B):
    """The bf16-operand configurations at reduced width, their own step size, 20 steps with no
    reset: everything within 2e-2 at every step."""
    full = workloads.WORKLOADS[name]
    dims = (full.dims[0] // 8,) + (width,) * (len(full.dims) - 2) + (full.dims[-1],)
    w = full.scaled(dims=dims, batch=B, steps=20)
    worst = run_mlp(w, w.steps, 2e-2, 2e-2, margin=True, margin_ratio=64.0, min_margin=1e-4)
    print("%s reduced, free-running, lr %.2f: worst relative error over 20 steps %.3e" % (name, w.lr, worst))


@pytest.mark.parametrize("dims,B,K,tau,nesterov", [
    ((384, 256, 256, 256, 100), 32, 3, (2, 3, 4), 1),
    ((40, 72, 100, 9), 20, 2, (1, 2), 0),              # widths that are no multiples of 4, 8 or 32
    ((352, 288, 288, 160), 160, 2, (2, 3), 1),         # ragged tiles in rows, columns and k-steps
    ((512, 512, 520, 24), 256, 2, (2, 2), 1),          # full tiles and a ragged last column tile
    ((1040, 1536, 2048, 24), 32, 2, (2, 3), 1)])       # norms from Gram products of 33, 48 and 64 k-steps
def test_fused_sampler_step_equals_the_separate_kernel(dims, B, K, tau, nesterov):
    """The fused path (norm of the first-pass weight gradients from Gram matrices or from a
    norm-only product, ascent in the epilogue of the recomputed products, sampler step in the
    epilogues of the second pass) against the same step with every gradient stored and the
    streaming kernels run on it (which the other bf16 tests hold to the oracle).  Where the
    two sum the squares of the same values in another order the norm may differ in its last
    bits; everything else is the same arithmetic on the same values.  So: norms equal to 2e-6,
    the bf16 operand copy of x~ equal except for a few elements on a rounding boundary (one
    bf16 step apart), parameters, velocities, iterate sums and the center equal to 2e-6 after
    several steps and center updates."""
    w = workloads.WORKLOADS["cfg3"].scaled(name="fuse", K=K, dims=dims, batch=B, tau=tau,
                                           nesterov=nesterov, n_classes=dims[-1], batch_pool=0)
    _fused_equals_separate(w, 5)


def _fused_equals_separate(w, steps):
    """One context with the fused path, one with every gradient stored and the streaming kernels
    run on it, same inputs: norms, parameters, velocities, iterate sums, center to 2e-6; the operand
    copy of x~ equal but for elements on a rounding boundary."""
    K = w.K
    init = workloads.init_params(w)
    cfg, keep = lsam.config_from_workload(w)
    a = lsam.Lsam(cfg, init, device=DEV, keep=keep)
    b = lsam.Lsam(cfg, init, device=DEV, keep=keep)
    assert a.lsam_set_fused_step(True) == 1 and b.lsam_set_fused_step(False) == 0
    for t in range(steps):
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        a.lsam_step(Xd, ld, None)
        b.lsam_step(Xd, ld, None)
        assert np.allclose(a.lsam_get_norms(), b.lsam_get_norms(), rtol=2e-6, atol=0), (t, w.dims)
        assert a.lsam_sync() == b.lsam_sync()
        for i in list(range(K)) + [-1]:
            assert rel_max(a.lsam_get_params(i), b.lsam_get_params(i)) < 2e-6, (t, i, w.dims)
        for i in range(K):
            for which in (lsam.BUF_VELOCITY, lsam.BUF_ITER_SUM):
                assert rel_max(a.lsam_get_buffer(which, i), b.lsam_get_buffer(which, i)) < 2e-6, (t, i, which)
            pa, pb = a.lsam_get_buffer(lsam.BUF_PERTURBED, i), b.lsam_get_buffer(lsam.BUF_PERTURBED, i)
            differ = pa != pb
            assert np.mean(differ) < 1e-3, (t, i, np.mean(differ))
            assert np.all(np.abs(pa - pb)[differ] <= 2.0 ** -7 * np.abs(pb)[differ]), (t, i)
    a.close()
    b.close()


def _random_bf16_mlp(rng):
    """A bf16 dense model drawn at random: 2 to 4 layers with widths that are and are not
    multiples of 4, 8, 32 and of the tile sides, some wide enough for the norm to come from Gram
    products, a batch that is or is not a multiple of 32, 1 to 5 replicas."""
    widths = [40, 72, 100, 128, 160, 288, 352, 520, 1040, 1536]
    L = int(rng.integers(2, 5))
    dims = [int(rng.choice([40, 352, 384, 1040]))]
    budget = 2.5e6                                  # weights per replica, so the oracle stays quick
    for _ in range(L - 1):
        fits = [v for v in widths if dims[-1] * v <= budget]
        dims.append(int(rng.choice(fits)))
        budget -= dims[-2] * dims[-1]
    classes = int(rng.choice([9, 24, 100, 160]))
    dims.append(classes)
    K = int(rng.integers(1, 6))
    B = int(rng.choice([20, 32, 64, 160, 256]))
    tau = tuple(int(v) for v in rng.integers(1, 5, size=K))
    return workloads.WORKLOADS["cfg3"].scaled(name="rand16", K=K, dims=tuple(dims), batch=B, tau=tau,
                                               nesterov=int(rng.integers(0, 2)), n_classes=classes,
                                               steps=4, batch_pool=0, data_seed=int(rng.integers(1, 1000)))


@pytest.mark.parametrize("seed", range(12))
def test_randomly_drawn_bf16_dense_models(seed):
    w = _random_bf16_mlp(np.random.default_rng(2000 + seed))
    print("seed %d: dims %s, B=%d, K=%d, tau=%s, nesterov=%d" % (seed, w.dims, w.batch, w.K, w.tau, w.nesterov))
    _fused_equals_separate(w, 4)
    # and the fused path against the oracle, from the oracle's state at every step past the first
    # (natural initialisation: a ReLU decided the other way moves single rows, which tol_flip covers)
    run_mlp(w, 3, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=1)


@pytest.mark.parametrize("seed", range(12))
def test_randomly_drawn_fp32_dense_models(seed):
    """fp32 dense models drawn at random (1 to 3 hidden layers; widths, batches and class counts
    on both sides of every kernel's limits: the narrow-head kernels up to 16 classes, contractions
    split over workgroups, ragged tiles) against the oracle: parameters to 1e-4 at every step."""
    rng = np.random.default_rng(3000 + seed)
    dims = [int(rng.choice([20, 100, 784, 1030]))]
    for _ in range(int(rng.integers(1, 4))):
        dims.append(int(rng.choice([10, 24, 37, 64, 128, 200, 264, 1024])))
    classes = int(rng.choice([3, 10, 16, 17, 40]))
    dims.append(classes)
    K = int(rng.integers(1, 5))
    w = workloads.WORKLOADS["cfg1"].scaled(name="rand32", K=K, dims=tuple(dims), batch=int(rng.choice([8, 20, 32, 128])),
                                           tau=tuple(int(v) for v in rng.integers(1, 5, size=K)),
                                           nesterov=int(rng.integers(0, 2)), n_classes=classes, steps=4,
                                           data_seed=int(rng.integers(1, 1000)))
    print("seed %d: dims %s, B=%d, K=%d, tau=%s, nesterov=%d" % (seed, w.dims, w.batch, w.K, w.tau, w.nesterov))
    run_mlp(w, 4, 1e-4, 1e-3, margin=False, anchor_after=1)


def test_bf16_ragged_shapes():
    w = workloads.WORKLOADS["cfg3"].scaled(name="ragged16", K=2, dims=(40, 72, 100, 9), batch=20,
                                           tau=(2, 3), n_classes=9, steps=6, batch_pool=0)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=2)


def test_bf16_wide_layers_with_long_gram_products():
    # contractions of 1040, 1536 and 2048 (33, 48, 64 steps of 32) of the B x B Gram products behind the
    # norm, the first of them ragged
    w = workloads.WORKLOADS["cfg3"].scaled(name="wide16", K=2, dims=(1040, 1536, 2048, 24), batch=32,
                                           tau=(2, 3), n_classes=24, steps=4, batch_pool=0)
    # (64 k pre-activations per layer leave no initialisation with a margin: natural one, anchored)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=1)


def test_bf16_ring_kernel_ragged_tiles_and_short_contractions():
    # shapes that leave ragged row and column tiles (160, 288, 352 are not multiples of 64) and a
    # k-step count (5 steps of 32) that is not a multiple of the rings' four and eight stages.
    # (Larger tiles: test_large_tiles_with_remainders.)
    w = workloads.WORKLOADS["cfg3"].scaled(name="ring16", K=2, dims=(352, 288, 288, 160), batch=160,
                                           tau=(2, 3), n_classes=160, steps=4, batch_pool=0)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=2)


def test_wrong_mode_calls_fail_cleanly():
    w = workloads.WORKLOADS["cfg4"].scaled(K=1, d_raw=64, tau=(1,))
    g, o = make_pair(w)
    z = torch.zeros(64, device=DEV)
    with pytest.raises(lsam.LsamError) as e:
        g.lsam_step(z, z.to(torch.int32), None)
    assert e.value.code == lsam.ESTATE
    with pytest.raises(lsam.LsamError):
        lsam._check(lsam.lib().lsam_get_params(g._h, 3, z.cpu().numpy().ctypes.data, 64))
    g.close()


# ---- comparators on the same kernels: synchronous data-parallel baseline, one-pass rho = 0 ---------
@pytest.mark.parametrize("rho", [0.05, 0.0])
def test_data_parallel_baseline_fp32(rho):
    """DP-SAM (DP-SGD for rho = 0): gradients averaged over the replicas at both passes."""
    w = workloads.WORKLOADS["cfg1"].scaled(name="dp32", K=3, tau=(2, 3, 4), steps=8, rho=rho,
                                           algorithm=lsam.ALG_DATA_PARALLEL)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=False)


def test_data_parallel_baseline_bf16():
    full = workloads.WORKLOADS["cfg3"]
    dims = (full.dims[0] // 8,) + (256,) * (len(full.dims) - 2) + (full.dims[-1],)
    w = full.scaled(name="dp16", K=4, dims=dims, batch=32, steps=6,
                    algorithm=lsam.ALG_DATA_PARALLEL)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=2)


@pytest.mark.parametrize("d,K", [(1000, 3), (65536 + 12, 4)])
def test_data_parallel_baseline_raw_mode(d, K):
    w = workloads.WORKLOADS["cfg4"].scaled(K=K, d_raw=d, tau=None, steps=6,
                                           algorithm=lsam.ALG_DATA_PARALLEL)
    g, o = make_pair(w)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-5)
        for i in range(K):
            assert rel_max(g.lsam_get_buffer(lsam.BUF_PERTURBED, i), o.last_perturbed[i]) < 1e-6
        assert g.lsam_sync() == 0 and o.sync() == 0
        check_state(g, o, 1e-4, "data-parallel raw d=%d step %d" % (d, t + 1))
    g.close()


@pytest.mark.parametrize("bf16", [0, 1])
def test_rho_zero_takes_one_pass_and_matches_two_pass_oracle(bf16):
    """With rho = 0 the step makes a single forward/backward pass (the ESGD / EASGD family);
    the oracle still walks through both passes of Algorithm 2 and must agree."""
    if bf16:
        full = workloads.WORKLOADS["cfg5"]
        dims = (full.dims[0] // 8,) + (128,) * (len(full.dims) - 2) + (full.dims[-1],)
        w = full.scaled(name="esgd16", dims=dims, batch=64, steps=6, rho=0.0)
        run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
    else:
        w = workloads.WORKLOADS["cfg1"].scaled(name="esgd32", steps=10, rho=0.0)
        run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
        run_mlp(w, w.steps, 1e-4, 1e-3, margin=False)


def test_rho_zero_raw_mode():
    w = workloads.WORKLOADS["cfg4"].scaled(K=3, d_raw=5000, tau=(2, 3, 4), steps=9, rho=0.0)
    g, o = make_pair(w)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-5)
        assert g.lsam_sync() == o.sync()
        check_state(g, o, 1e-4, "rho=0 raw step %d" % (t + 1))
    g.close()


# ---- Algorithm 1 mode and the theorems' step-size / radius schedules on a convex toy ---------------
def test_algorithm_one_mode_constant_versus_decaying_perturbation():
    """K = 1, tau = 1, beta = 0, eta' = alpha is Algorithm 1 (x-update with coupling, then
    y <- alpha x + (1 - alpha) y).  On f(x) = x'Ax/2 with exact gradients, a constant radius
    leaves ||grad f|| hovering at a floor set by rho (the constant-perturbation theorem's
    O(rho^2) term), while rho_t = rho_0/sqrt(t+1) with eta_t = eta_0/sqrt(t+1) keeps
    descending (the decaying-perturbation theorem).  Every step is also held to the oracle."""
    d, alpha, lam, T = 64, 0.3, 0.5, 1500
    rng = np.random.default_rng(3)
    A = np.linspace(0.1, 1.0, d)
    x0 = rng.standard_normal(d).astype(np.float32)
    finals = {}
    for decaying in (False, True):
        w = workloads.WORKLOADS["cfg4"].scaled(K=1, d_raw=d, tau=(1,), beta=0.0, lr_center=alpha,
                                               momentum=0.0, lambda_abs=lam, rho=0.5, lr=0.5,
                                               gamma=1e-12)
        g, o = make_pair(w, x0)
        for t in range(T):
            lr, rho = (0.5 / np.sqrt(t + 1), 0.5 / np.sqrt(t + 1)) if decaying else (0.5, 0.5)
            g.lsam_set_scalars(lr, rho)
            o.set_scalars(np.float32(lr), np.float32(rho))
            x = o.get_params(0)          # the gradient oracle follows the CPU side's iterate
            g1 = A * x
            xt = x + np.float64(np.float32(rho)) * g1 / (np.linalg.norm(g1) + 1e-12)
            g2 = A * xt
            g1f, g2f = g1.astype(np.float32)[None], g2.astype(np.float32)[None]
            g.lsam_step_grads(torch.from_numpy(g1f).to(DEV), torch.from_numpy(g2f).to(DEV))
            o.step_grads(g1f, g2f)
            assert g.lsam_sync() == 1 and o.sync() == 1
            if t % 250 == 0 or t == T - 1:
                # both sides are fed the gradients of the oracle's iterate, so they can only
                # differ by rounding that the contraction of the update keeps damping
                close_enough(g.lsam_get_params(0), o.get_params(0), 1e-4, "x at step %d" % t)
                close_enough(g.lsam_get_params(-1), o.get_params(-1), 1e-4, "y at step %d" % t)
        finals[decaying] = float(np.linalg.norm(A * g.lsam_get_params(0).astype(np.float64)))
        g.close()
    print("||grad f|| after %d steps: constant rho %.3e, decaying %.3e" % (T, finals[False], finals[True]))
    assert finals[False] > 1e-2               # the floor of the constant radius
    assert finals[True] < 0.2 * finals[False]


# ---- Langevin (SGLD) sampler: Philox-driven Gaussian noise inside the descent kernel ---------------
@pytest.mark.parametrize("d,K", [(4096, 2), (1003, 3), (65536 * 2 + 7, 2)])
def test_langevin_noise_raw_mode(d, K):
    w = workloads.WORKLOADS["cfg4"].scaled(K=K, d_raw=d, tau=(2,) * K, steps=7, noise_scale=0.3,
                                           noise_seed=(91 << 32) | 17)
    g, o = make_pair(w)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert g.lsam_sync() == o.sync()
        check_state(g, o, 1e-4, "langevin raw d=%d step %d" % (d, t + 1))
    # the noise really is there: sigma sqrt(2 eta) = 0.13 per step dwarfs the 1e-2 gradients
    assert np.std(g.lsam_get_params(0) - workloads.init_params(w)) > 0.1
    g.close()


def test_langevin_noise_fp32_mlp_ragged_widths():
    # widths that are not multiples of 4 or 8: the noise must skip the padding of every row
    w = workloads.WORKLOADS["cfg1"].scaled(name="sgld32", K=2, dims=(50, 37, 19, 7), batch=5,
                                           tau=(2, 3), n_classes=7, steps=6, data_seed=9,
                                           noise_scale=1e-3, noise_seed=5)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=False)


def test_langevin_noise_bf16_mlp():
    full = workloads.WORKLOADS["cfg3"]
    dims = (full.dims[0] // 8,) + (256,) * (len(full.dims) - 2) + (full.dims[-1],)
    w = full.scaled(name="sgld16", K=3, dims=dims, batch=32, steps=6, noise_scale=1e-3,
                    noise_seed=2 ** 40 + 3)
    run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)


# ---- limits and degenerate inputs ------------------------------------------------------------------
def test_maximum_replica_count_raw_mode():
    K = 64                                          # LSAM_MAX_REPLICAS
    w = workloads.WORKLOADS["cfg4"].scaled(K=K, d_raw=777, tau=None, tau_min=2, tau_max=6,
                                           sched_seed=12, steps=8)
    g, o = make_pair(w)
    for t in range(w.steps):
        g1, g2 = workloads.raw_grads(w, t)
        g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
        o.step_grads(g1, g2)
        assert g.lsam_sync() == o.sync()
    # v carries lambda (x - y) with |x|, |y| ~ 1 but |x - y| ~ 1e-2 and gradients ~ 1e-2: the fp32
    # rounding of x and y (1e-7) is a 1e-4 relative error of v once the center moves every tick,
    # as it does with 64 replicas; parameters, sums and the center keep the tight bound
    check_state(g, o, 1e-4, "K=64", tol_v=1e-3)
    g.close()


@pytest.mark.parametrize("bf16", [0, 1])
def test_maximum_depth_mlp(bf16):
    dims = (24,) + (16,) * 39 + (5,)               # LSAM_MAX_LAYERS = 40 dense layers
    w = workloads.WORKLOADS["cfg1"].scaled(name="deep", K=2, dims=dims, batch=6, tau=(2, 3),
                                           n_classes=5, steps=4, data_seed=4, gemm_dtype=bf16)
    if bf16:
        # (the fused path with every table of per-layer offsets full; Langevin noise as well, which
        # takes the unfused kernels and the largest argument block)
        run_mlp(w, w.steps, 2e-2, 2e-2, margin=True)
        run_mlp(w.scaled(noise_scale=1e-4, noise_seed=3), w.steps, 2e-2, 2e-2, margin=True)
    else:
        run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
        run_mlp(w.scaled(noise_scale=1e-4, noise_seed=3), w.steps, 1e-4, 1e-3, margin=True)
    cfg, keep = lsam.config_from_workload(w.scaled(dims=dims[:-1] + (16, 5)))
    assert lsam.lsam_workspace_bytes(cfg) == 0 and "n_layers" in lsam.last_error()


def test_zero_gradients_leave_only_the_coupling():
    """g1 = g2 = 0: the norm is 0, the perturbation rho * 0 / (0 + gamma) = 0, and the step is
    the pure pull toward the center."""
    w = workloads.WORKLOADS["cfg4"].scaled(K=2, d_raw=4096, tau=(1, 2), steps=4)
    rng = np.random.default_rng(8)
    init = rng.standard_normal(3 * w.d_raw).astype(np.float32)       # distinct x_0, x_1, y
    g, o = make_pair(w, init)
    z = np.zeros((2, w.d_raw), dtype=np.float32)
    for t in range(w.steps):
        before = [g.lsam_get_params(i) for i in range(2)]
        g.lsam_step_grads(torch.from_numpy(z).to(DEV), torch.from_numpy(z).to(DEV))
        o.step_grads(z, z)
        assert np.all(g.lsam_get_norms() == 0.0)
        for i in range(2):       # the perturbed point is the point itself, bit for bit
            assert np.array_equal(g.lsam_get_buffer(lsam.BUF_PERTURBED, i), before[i])
        assert g.lsam_sync() == o.sync()
        check_state(g, o, 1e-4, "zero gradients step %d" % (t + 1))
    g.close()


@pytest.mark.parametrize("dims,B", [((40, 33, 17), 9),        # 17 classes: one more than the fused head takes
                                    ((1100, 12), 7),          # head input wider than its LDS staging
                                    ((16, 24, 3), 600)])      # batch beyond the head's dZ staging
def test_fp32_classifier_head_fallbacks(dims, B):
    w = workloads.WORKLOADS["cfg1"].scaled(name="headfb", K=2, dims=dims, batch=B, tau=(2, 3),
                                           n_classes=dims[-1], steps=3, data_seed=6)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=True)
    run_mlp(w, w.steps, 1e-4, 1e-3, margin=False)


def test_peak_probe_reports_plausible_ceilings():
    scratch = torch.empty(1 << 26, dtype=torch.float32, device=DEV)      # 256 MiB
    copy_gbs, bf16_tf, f32_tf = lsam.lsam_probe_peaks(scratch)
    assert 1000.0 < copy_gbs < 8000.0 * 1.05        # below the HBM datasheet figure
    assert 500.0 < bf16_tf < 2500.0 * 1.05
    assert 50.0 < f32_tf < 157.3 * 1.05
    with pytest.raises(lsam.LsamError):
        lsam.lsam_probe_peaks(scratch[:16])          # too small


@pytest.mark.parametrize("name", ["cfg1", "bf16", "cnn", "residual"])
def test_step_can_be_captured_and_replayed_as_a_hip_graph(name):
    """`lsam_step` allocates nothing and never synchronises, so a caller may capture it.  Four
    replays of the captured step, with eager work and synchronisations between them, must
    leave exactly the state of four eager steps on the same batch (the kernels are
    deterministic; the host-side counters are not part of what a graph replays, so no sync
    point is crossed here)."""
    if name == "cfg1":
        w = workloads.WORKLOADS["cfg1"].scaled(tau=(100, 100))
    elif name == "cnn":
        # all three ways a convolution is served: first-layer kernels, unfolding inside the
        # GEMM, stored unfolded image
        w = workloads.Workload("cnn_graph", K=2, dims=(3, 32, 32, 24, 40, 10), batch=8, n_conv=4,
                               img_h=8, img_w=8, pool_mask=0b0110, rho=0.05, lr=0.05,
                               tau=(100, 100), n_classes=10, data_seed=41)
    elif name == "residual":
        # batch normalisation, a strided projection block, then a pre-activation variant of the
        # same layers is not needed: the two differ in kernels' arguments only
        w = workloads.Workload("res_graph", K=2, dims=(3, 8, 16, 16, 16, 16, 5), batch=6, n_conv=5, img_h=8,
                               img_w=8, bn_mask=0b11111, stride_mask=0b00010, skip_mask=0b10100,
                               proj_mask=0b00100, global_avg_pool=1, rho=0.05, lr=0.05, tau=(100, 100),
                               n_classes=5, data_seed=51)
    else:
        full = workloads.WORKLOADS["cfg3"]
        dims = (full.dims[0] // 8,) + (256,) * (len(full.dims) - 2) + (full.dims[-1],)
        w = full.scaled(K=2, dims=dims, batch=32, tau=(100, 100))
    init = workloads.init_params(w)
    X, lab = workloads.batch(w, 0)
    st = torch.cuda.Stream(device=DEV)
    with torch.cuda.stream(st):
        Xd, ld = to_dev(X, lab, w)
        loss_a = torch.zeros(w.K, device=DEV)
        loss_b = torch.zeros(w.K, device=DEV)
        cfg, keep = lsam.config_from_workload(w)
        a = lsam.Lsam(cfg, init, device=DEV, keep=keep, stream=st)
        b = lsam.Lsam(cfg, init, device=DEV, keep=keep, stream=st)
        for _ in range(4):
            a.lsam_step(Xd, ld, loss_a)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            b.lsam_step(Xd, ld, loss_b)
        scratch = torch.zeros(1 << 20, device=DEV)
        for r in range(4):
            graph.replay()
            scratch.add_(1.0)               # the program's own eager work between replays
            st.synchronize()
            assert np.all(np.isfinite(loss_b.cpu().numpy())), r
        assert np.array_equal(loss_a.cpu().numpy(), loss_b.cpu().numpy())
        for i in range(w.K):
            for which in (lsam.BUF_PARAMS, lsam.BUF_VELOCITY, lsam.BUF_ITER_SUM, lsam.BUF_GRAD):
                assert np.array_equal(a.lsam_get_buffer(which, i), b.lsam_get_buffer(which, i)), (i, which)
        a.close()
        b.close()


# ---- convolutional model -------------------------------------------------------------------------
CNN_SMALL = workloads.Workload("cnn_small", K=2, dims=(3, 8, 16, 24, 5), batch=6, n_conv=2,
                               img_h=8, img_w=8, pool_mask=0b11, rho=0.05, lr=0.05, tau=(2, 3),
                               n_classes=5, data_seed=31)


@pytest.mark.parametrize("name,over", [
    ("pool after both", {}),
    ("no pool below a convolution", dict(pool_mask=0b10)),
    ("no pool at all", dict(pool_mask=0, img_h=4, img_w=6)),
    ("head directly on the image", dict(dims=(3, 8, 16, 10), n_classes=10)),
    ("wide softmax output", dict(dims=(3, 8, 16, 40, 20), n_classes=20)),
    ("one convolution, odd input channels", dict(dims=(5, 16, 12, 3), n_conv=1, pool_mask=1,
                                                 n_classes=3, img_h=6, img_w=10)),
    ("three convolutions", dict(dims=(1, 8, 8, 16, 32, 4), n_conv=3, pool_mask=0b101, n_classes=4,
                                batch=9)),
    # channel counts that are multiples of 32: the GEMMs then read the unfolded images straight
    # from the images (forward, dW and dX), with and without a pool below the layer
    ("unfolding inside the GEMM", dict(dims=(3, 32, 32, 64, 10), n_conv=3, pool_mask=0b101,
                                       n_classes=10, batch=5)),
    # first layers with 1..3 input channels and 32 | C_out have kernels of their own
    ("one-channel first layer, 64 filters", dict(dims=(1, 64, 16, 4), n_conv=1, pool_mask=1,
                                                 n_classes=4, img_h=6, img_w=10, batch=5)),
    ("two-channel first layer, no pool", dict(dims=(2, 32, 8, 24, 5), n_conv=2, pool_mask=0b10,
                                              img_h=4, img_w=6, batch=43)),
    ("four convolutions, one of each kind and two pools", dict(
        dims=(3, 32, 32, 24, 40, 10), n_conv=4, pool_mask=0b0110, n_classes=10, batch=8)),
    # batch normalisation, on each kind of convolution
    ("batch norm on stored-unfold layers", dict(bn_mask=0b11)),
    ("batch norm on the second layer only, no pools", dict(bn_mask=0b10, pool_mask=0, img_h=4, img_w=6)),
    ("batch norm with first-layer kernels and unfolding inside the GEMM", dict(
        dims=(3, 32, 32, 64, 10), n_conv=3, pool_mask=0b101, bn_mask=0b111, n_classes=10, batch=5)),
    ("batch norm in a four-convolution stack", dict(
        dims=(3, 32, 32, 24, 40, 10), n_conv=4, pool_mask=0b0110, bn_mask=0b1010, n_classes=10, batch=8)),
    # degenerate sizes: one sample per replica (normalisation over the pixels only), an image
    # that pools down to a single pixel, the largest replica count
    ("batch of one, normalised", dict(batch=1, bn_mask=0b11, img_h=4, img_w=4)),
    ("2x2 image pooled to one pixel", dict(dims=(3, 32, 32, 7), n_conv=2, pool_mask=0b10, img_h=2,
                                           img_w=2, n_classes=7, batch=9)),
    ("64 replicas", dict(K=64, batch=2, img_h=4, img_w=4, pool_mask=0b01, tau=tuple([2, 3] * 32))),
    ("unfolding inside the GEMM, sides not powers of two", dict(
        dims=(4, 32, 64, 12, 6), n_conv=2, pool_mask=0b10, img_h=6, img_w=10, n_classes=6, batch=7)),
])
def test_cnn_matches_oracle(name, over):
    w = CNN_SMALL.scaled(**over)
    # free-running for two steps, then every step from the oracle's state: one ReLU or pooling
    # decision that falls differently in fp32 (these nets take 10^4 of them per step on batches
    # of 5 to 43) would otherwise be amplified by the momentum into a diverging trajectory
    worst = run_mlp(w, 6, 1e-4, 1e-3, anchor_after=2)
    print("cnn %s: worst parameter error %.3e" % (name, worst))


@pytest.mark.parametrize("name,over", [
    ("stored unfold", {}),
    ("first-layer kernels, unfolding inside the GEMM, batch norm", dict(
        dims=(3, 32, 32, 64, 10), n_conv=3, pool_mask=0b101, bn_mask=0b010, n_classes=10, batch=5)),
    ("four convolutions, wide softmax", dict(
        dims=(3, 32, 32, 24, 40, 48, 20), n_conv=4, pool_mask=0b0110, n_classes=20, batch=8)),
    # enough rows and channels for the plane products and for split contractions
    ("wide layers, many rows", dict(dims=(3, 64, 128, 10), n_conv=2, pool_mask=0b10, n_classes=10,
                                    K=4, batch=96, tau=(2, 2, 3, 3))),
])
def test_cnn_bf16_products_match_oracle(name, over):
    # gemm_dtype = bf16 with convolutions: tensors stay fp32, every matrix product rounds its two
    # operands to bf16.  The oracle rounds the same operands; what is left is accumulation order
    # and operands that sit on a rounding boundary (their fp32 and float64 values can round to
    # neighbouring bf16 numbers, 2^-8 apart), hence the bf16 tolerance.
    w = CNN_SMALL.scaled(gemm_dtype=1, **over)
    worst = run_mlp(w, 5, 2e-2, 2e-2, anchor_after=1)
    print("cnn bf16 %s: worst parameter error %.3e" % (name, worst))


def test_cnn_bf16_exact_operands_tight():
    # grid-valued inputs and parameters (all bf16 numbers, all pre-activations exact): the two
    # convolutions' forward passes are then identical in both arithmetics, every decision
    # coincides, and only the rounding of dZ separates the gradients from the fp32 model's
    w = CNN_SMALL.scaled(K=2, dims=(3, 32, 32, 10), n_conv=2, img_h=16, img_w=16, pool_mask=0b11,
                         batch=64, n_classes=10, rho=0.0, tau=(2, 2), gemm_dtype=1)
    init = workloads.init_params(w).astype(np.float64)
    off = 0
    for l, (fi, fo) in enumerate(w.layer_shapes):
        n = fi * fo + fo
        q = 16.0 * (l + 1) if l < 2 else 256.0
        init[off:off + n] = np.round(init[off:off + n] * q) / q
        off += n
    X, lab = workloads.batch(w, 0)
    X = (np.round(X * 2.0) / 2.0).astype(np.float32)
    g, o = make_pair(w, init.astype(np.float32))
    loss_d = torch.zeros(w.K, dtype=torch.float32, device=DEV)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), loss_d)
    ol = o.step(X, lab)
    assert np.allclose(loss_d.cpu().numpy(), ol, rtol=1e-3)
    for i in range(w.K):
        gi = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        close_enough(gi, o.last_g1[i], 1e-2, "gradient of replica %d" % i)
    check_state(g, o, 1e-4, "grid-valued bf16 cnn")
    g.close()


def test_cnn_gradients_layer_by_layer():
    # one step from a common point: both gradients and the norm, every layer on its own
    w = CNN_SMALL.scaled(K=3, batch=10, tau=(2, 2, 2))
    g, o = make_pair(w)
    X, lab = workloads.batch(w, 0)
    Xd, ld = to_dev(X, lab, w)
    g.lsam_step(Xd, ld)
    o.step(X, lab)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-4)
    for i in range(w.K):
        g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], 1e-3, "dW%d of replica %d" % (l + 1, i))
            close_enough(g2[o1:o2], o.last_g2[i][o1:o2], 1e-3, "db%d of replica %d" % (l + 1, i))
        xt = g.lsam_get_buffer(lsam.BUF_PERTURBED, i)
        assert rel_max(xt, o.last_perturbed[i]) < 1e-5
    g.close()


def test_cnn_exact_decisions_tight_gradients():
    # Inputs and parameters on coarse binary grids: every pre-activation of the two convolutions
    # is then a short sum of exactly representable products, the same number in fp32 (in any
    # summation order) and in float64, so every ReLU mask and every pooling choice -- ties
    # included, which the grid makes frequent -- is the same on both sides and the gradients
    # must agree to fp32 rounding.  rho = 0: one pass, at the grid point itself.
    w = CNN_SMALL.scaled(K=2, dims=(3, 32, 32, 10), n_conv=2, img_h=16, img_w=16, pool_mask=0b11,
                         batch=64, n_classes=10, rho=0.0, tau=(2, 2))
    init = workloads.init_params(w).astype(np.float64)
    off = 0
    for l, (fi, fo) in enumerate(w.layer_shapes):
        n = fi * fo + fo
        if l < 2:                       # multiples of 1/16 (first layer) and 1/32 (second)
            q = 16.0 * (l + 1)
            init[off:off + n] = np.round(init[off:off + n] * q) / q
        off += n
    X, lab = workloads.batch(w, 0)
    X = (np.round(X * 2.0) / 2.0).astype(np.float32)          # multiples of 1/2
    g, o = make_pair(w, init.astype(np.float32))
    loss_d = torch.zeros(w.K, dtype=torch.float32, device=DEV)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), loss_d)
    ol = o.step(X, lab)
    assert np.allclose(loss_d.cpu().numpy(), ol, rtol=1e-6)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-5)
    for i in range(w.K):
        gi = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            assert rel_max(gi[o0:o1], o.last_g1[i][o0:o1]) < 1e-5, (i, l)
            assert rel_max(gi[o1:o2], o.last_g1[i][o1:o2]) < 1e-5, (i, l)
    check_state(g, o, 1e-6, "grid-valued cnn")
    g.close()


def test_batchnorm_gradients_layer_by_layer():
    # gamma, beta and everything below a normalised layer, one step from a common point; the
    # batch is large enough that the chunked statistics span several chunks and a ragged one
    w = CNN_SMALL.scaled(K=2, batch=11, img_h=8, img_w=8, bn_mask=0b11, tau=(2, 2))
    g, o = make_pair(w)
    X, lab = workloads.batch(w, 0)
    X = X + np.float32(3.0)            # a mean far from zero: the variance must not lose digits
    Xd, ld = to_dev(X, lab, w)
    g.lsam_step(Xd, ld)
    o.step(X, lab)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-4)
    for i in range(w.K):
        g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], 1e-3, "dW%d of replica %d" % (l + 1, i))
        for l, (g0, g1, g2_) in o.model.bn_offsets.items():
            close_enough(g2[g0:g1], o.last_g2[i][g0:g1], 1e-3, "dgamma%d of replica %d" % (l + 1, i))
            close_enough(g2[g1:g2_], o.last_g2[i][g1:g2_], 1e-3, "dbeta%d of replica %d" % (l + 1, i))
        # the bias below a normalisation has no influence: its gradient is rounding noise
        for l in o.model.bn_offsets:
            o0, o1, o2 = o.model.offsets[l]
            assert np.max(np.abs(g2[o1:o2])) < 1e-4 * np.max(np.abs(g2[o0:o1]))
    g.close()


def test_cnn_data_parallel_and_langevin():
    for over in (dict(algorithm=lsam.ALG_DATA_PARALLEL), dict(noise_scale=0.01, noise_seed=5),
                 dict(rho=0.0), dict(noise_scale=0.01, noise_seed=6, bn_mask=0b01)):
        w = CNN_SMALL.scaled(**over)
        run_mlp(w, 4, 1e-4, 1e-3)


def test_cnn_rejects_what_it_cannot_run():
    for over, msg in ((dict(dims=(3, 8, 12, 24, 5)), "multiples of 8"),
                      (dict(img_h=6, img_w=6), "even image sides"),
                      (dict(n_conv=4), "at least one dense layer"),
                      (dict(bn_mask=0b100), "no convolution"),
                      (dict(bn_mask=0b1, bn_eps=0.0), "bn_eps")):
        w = CNN_SMALL.scaled(**over)
        cfg, keep = lsam.config_from_workload(w)
        assert lsam.lsam_workspace_bytes(cfg) == 0
        assert msg in lsam.last_error(), lsam.last_error()


# ---- graph replay across sync points; checkpoint and resume in a new context ------------------------
@pytest.mark.parametrize("name", ["cfg1", "bf16"])
def test_replayed_steps_with_eager_syncs_cross_sync_points(name):
    """A captured step replayed twelve times, each replay followed by lsam_note_replay and an
    eager lsam_sync, against twelve eager ticks on the same batch: the schedules must stay equal
    tick by tick (several center updates happen on the way) and the final state bit for bit."""
    if name == "cfg1":
        w = workloads.WORKLOADS["cfg1"].scaled(tau=(2, 3))
    else:
        full = workloads.WORKLOADS["cfg3"]
        dims = (full.dims[0] // 8,) + (256,) * (len(full.dims) - 2) + (full.dims[-1],)
        w = full.scaled(K=3, dims=dims, batch=32, tau=(2, 3, 5))
    init = workloads.init_params(w)
    X, lab = workloads.batch(w, 0)
    st = torch.cuda.Stream(device=DEV)
    with torch.cuda.stream(st):
        Xd, ld = to_dev(X, lab, w)
        loss_a = torch.zeros(w.K, device=DEV)
        loss_b = torch.zeros(w.K, device=DEV)
        cfg, keep = lsam.config_from_workload(w)
        a = lsam.Lsam(cfg, init, device=DEV, keep=keep, stream=st)
        b = lsam.Lsam(cfg, init, device=DEV, keep=keep, stream=st)
        served_a = []
        for _ in range(13):
            a.lsam_step(Xd, ld, loss_a)
            served_a.append((a.lsam_sync(), a.lsam_get_schedule()))
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            b.lsam_step(Xd, ld, loss_b)          # capture: advances the counters, runs nothing
        # the capture counted as a tick although no kernel ran: take it back
        cnt = b.lsam_get_counters()
        cnt[:w.K] = 0
        cnt[2 * w.K + 2] = 0
        b.lsam_set_counters(cnt)
        served_b = []
        scratch = torch.zeros(1 << 18, device=DEV)
        for r in range(13):
            graph.replay()
            b.lsam_note_replay()
            scratch.add_(1.0)
            served_b.append((b.lsam_sync(), b.lsam_get_schedule()))
            st.synchronize()
        assert served_a == served_b
        assert sum(n for n, _ in served_a) >= 8
        assert np.array_equal(loss_a.cpu().numpy(), loss_b.cpu().numpy())
        for i in list(range(w.K)) + [-1]:
            assert np.array_equal(a.lsam_get_params(i), b.lsam_get_params(i)), i
        for i in range(w.K):
            for which in (lsam.BUF_VELOCITY, lsam.BUF_ITER_SUM):
                assert np.array_equal(a.lsam_get_buffer(which, i), b.lsam_get_buffer(which, i)), (i, which)
        assert np.array_equal(a.lsam_get_buffer(lsam.BUF_CENTER_DIR, -1), b.lsam_get_buffer(lsam.BUF_CENTER_DIR, -1))
        # what a replay cannot follow is refused
        wn = w.scaled(noise_scale=0.1)
        cfgn, keepn = lsam.config_from_workload(wn)
        n = lsam.Lsam(cfgn, init, device=DEV, keep=keepn, stream=st)
        with pytest.raises(lsam.LsamError) as e:
            n.lsam_note_replay()
        assert e.value.code == lsam.ESTATE
        for eng in (a, b, n):
            eng.close()


@pytest.mark.parametrize("mode", ["raw_redraw_noise", "mlp"])
def test_checkpoint_mid_period_resumes_in_a_new_context(mode):
    """Run A takes 9 ticks.  Run B takes 5, is read out (buffers, integer state), destroyed, and
    a fresh context restored from that snapshot takes the other 4: the schedule must be
    bit-exact and the state equal to run A's (same kernels on the same values: bit for bit),
    which also keeps it within tolerance of the oracle.  The snapshot falls between syncs, with
    non-zero local counts, iterate sums, a previous center direction, and -- in the raw-vector
    case -- redrawn periods, a generator state and a Langevin step counter to carry over."""
    if mode == "mlp":
        w = workloads.WORKLOADS["cfg1"].scaled(K=3, tau=(2, 3, 4), steps=9)
    else:
        w = workloads.WORKLOADS["cfg4"].scaled(K=4, d_raw=3000, tau=None, tau_min=2, tau_max=4,
                                               sched_seed=99, sched_mode=workloads.SCHED_REDRAW,
                                               noise_scale=0.05, noise_seed=7, steps=9)
    init = workloads.init_params(w)
    cfg, keep = lsam.config_from_workload(w)

    def tick(eng, t, ora=None):
        if mode == "mlp":
            X, lab = workloads.batch(w, t)
            Xd, ld = to_dev(X, lab, w)
            eng.lsam_step(Xd, ld, None)
            if ora is not None:
                ora.step(X, lab)
        else:
            g1, g2 = workloads.raw_grads(w, t)
            eng.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
            if ora is not None:
                ora.step_grads(g1, g2)
        n = eng.lsam_sync()
        if ora is not None:
            assert n == ora.sync()
        return n

    a, o = make_pair(w, init)
    for t in range(9):
        tick(a, t, o)
    b = lsam.Lsam(cfg, init, device=DEV, keep=keep)
    for t in range(5):
        tick(b, t)
    tau, cnt, ty = b.lsam_get_schedule()
    assert ty > 0 and max(cnt) > 0, "the snapshot should fall inside a period, after a sync"
    snap = {"counters": b.lsam_get_counters(),
            "x": [b.lsam_get_params(i) for i in range(w.K)], "y": b.lsam_get_params(-1),
            "v": [b.lsam_get_buffer(lsam.BUF_VELOCITY, i) for i in range(w.K)],
            "S": [b.lsam_get_buffer(lsam.BUF_ITER_SUM, i) for i in range(w.K)],
            "gprev": b.lsam_get_buffer(lsam.BUF_CENTER_DIR, -1)}
    b.close()
    c = lsam.Lsam(cfg, np.zeros_like(init), device=DEV, keep=keep)     # nothing carried by init
    for i in range(w.K):
        c.lsam_set_buffer(lsam.BUF_PARAMS, i, snap["x"][i])
        c.lsam_set_buffer(lsam.BUF_VELOCITY, i, snap["v"][i])
        c.lsam_set_buffer(lsam.BUF_ITER_SUM, i, snap["S"][i])
    c.lsam_set_buffer(lsam.BUF_PARAMS, -1, snap["y"])
    c.lsam_set_buffer(lsam.BUF_CENTER_DIR, -1, snap["gprev"])
    c.lsam_set_counters(snap["counters"])
    assert c.lsam_get_schedule() == (tau, cnt, ty)
    for t in range(5, 9):
        tick(c, t)
    assert c.lsam_get_schedule() == a.lsam_get_schedule() == o.get_schedule()
    assert np.array_equal(c.lsam_get_counters(), a.lsam_get_counters())
    for i in list(range(w.K)) + [-1]:
        assert np.array_equal(c.lsam_get_params(i), a.lsam_get_params(i)), i
    for i in range(w.K):
        assert np.array_equal(c.lsam_get_buffer(lsam.BUF_ITER_SUM, i), a.lsam_get_buffer(lsam.BUF_ITER_SUM, i))
        assert np.array_equal(c.lsam_get_buffer(lsam.BUF_VELOCITY, i), a.lsam_get_buffer(lsam.BUF_VELOCITY, i))
    check_state(c, o, 1e-3 if mode == "mlp" else 1e-4, "resumed run", tol_v=5e-2 if mode == "mlp" else None)
    # a snapshot with impossible values is refused and changes nothing
    bad = snap["counters"].copy()
    bad[w.K] = 0                      # a period of zero
    with pytest.raises(lsam.LsamError):
        c.lsam_set_counters(bad)
    assert np.array_equal(c.lsam_get_counters(), a.lsam_get_counters())
    a.close()
    c.close()


# ---- residual networks: stride-2 convolutions, parameter-free shortcuts, global average pooling -----
RES_SMALL = workloads.Workload("res_small", K=2, dims=(3, 8, 8, 8, 5), batch=6, n_conv=3, img_h=8,
                               img_w=8, bn_mask=0b111, skip_mask=0b100, global_avg_pool=1, rho=0.05,
                               lr=0.05, tau=(2, 3), n_classes=5, data_seed=51)


@pytest.mark.parametrize("name,over", [
    ("a stem and one block on the same shape", {}),
    ("a block that halves the image and doubles the channels, then one on the new shape", dict(
        dims=(3, 8, 16, 16, 16, 16, 5), n_conv=5, bn_mask=0b11111, stride_mask=0b00010, skip_mask=0b10100)),
    ("stride without shortcut or normalisation, flattened image into the dense layers", dict(
        dims=(3, 8, 16, 12, 5), n_conv=2, bn_mask=0, stride_mask=0b10, skip_mask=0, global_avg_pool=0)),
    ("a shortcut that only widens, image sides that are no powers of two, two dense layers", dict(
        dims=(4, 8, 8, 24, 12, 5), n_conv=3, img_h=6, img_w=10)),
    ("blocks on 32- and 64-channel images (unfolding inside the GEMM), first-layer kernels", dict(
        dims=(3, 32, 32, 32, 64, 64, 10), n_conv=5, bn_mask=0b11111, stride_mask=0b01000,
        skip_mask=0b10100, n_classes=10, batch=4)),
    ("stride on the first convolution, a pool after the block", dict(
        dims=(3, 8, 8, 8, 5), stride_mask=0b001, pool_mask=0b100, img_h=16, img_w=8)),
    ("three stages of one block each, ResNet-20's shape in small", dict(
        dims=(3, 16, 16, 16, 32, 32, 64, 64, 10), n_conv=7, bn_mask=0b1111111, stride_mask=0b0101000,
        skip_mask=0b1010100, img_h=16, img_w=16, n_classes=10, batch=4, K=3, tau=(2, 3, 4))),
])
def test_residual_model_matches_oracle(name, over):
    w = RES_SMALL.scaled(**over)
    worst = run_mlp(w, 6, 1e-4, 1e-3, anchor_after=2)
    print("residual %s: worst parameter error %.3e" % (name, worst))


def test_residual_model_gradients_layer_by_layer():
    """One step of a two-stage residual model from the common start: every layer's dW, db,
    dgamma and dbeta of the pass at the perturbed point against the oracle's."""
    w = RES_SMALL.scaled(dims=(3, 8, 16, 16, 16, 16, 5), n_conv=5, bn_mask=0b11111, stride_mask=0b00010,
                         skip_mask=0b10100, batch=16)
    g, o = make_pair(w)
    X, lab = workloads.batch(w, 0)
    Xd, ld = to_dev(X, lab, w)
    loss_d = torch.zeros(w.K, device=DEV)
    g.lsam_step(Xd, ld, loss_d)
    ol = o.step(X, lab)
    assert np.allclose(loss_d.cpu().numpy(), ol, rtol=1e-5)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-3)
    for i in range(w.K):
        g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], 2e-3, "dW%d of replica %d" % (l + 1, i))
            if l in o.model.bn_offsets:
                b0, b1, b2 = o.model.bn_offsets[l]
                close_enough(g2[b0:b1], o.last_g2[i][b0:b1], 2e-3, "dgamma%d of replica %d" % (l + 1, i))
                close_enough(g2[b1:b2], o.last_g2[i][b1:b2], 2e-3, "dbeta%d of replica %d" % (l + 1, i))
            else:
                close_enough(g2[o1:o2], o.last_g2[i][o1:o2], 2e-3, "db%d of replica %d" % (l + 1, i))
    g.close()


def test_residual_model_with_bf16_products_and_the_comparators():
    w = RES_SMALL.scaled(dims=(3, 8, 16, 16, 16, 16, 5), n_conv=5, bn_mask=0b11111, stride_mask=0b00010,
                         skip_mask=0b10100)
    # velocities see each rounding-boundary difference of a bf16 operand undamped: the looser bound
    # of the other bf16 runs
    run_mlp(w.scaled(gemm_dtype=1, batch=16), 5, 2e-2, 2e-2, anchor_after=1, tol_flip=1e-1)
    run_mlp(w.scaled(algorithm=lsam.ALG_DATA_PARALLEL), 4, 1e-4, 1e-3, anchor_after=1)
    run_mlp(w.scaled(noise_scale=1e-3, noise_seed=11), 4, 1e-4, 1e-3, anchor_after=1)


# ---- projection shortcuts (1x1 convolution + batch normalisation where a block changes shape) ----
PROJ_SMALL = RES_SMALL.scaled(dims=(3, 8, 16, 16, 16, 16, 5), n_conv=5, bn_mask=0b11111, stride_mask=0b00010,
                              skip_mask=0b10100, proj_mask=0b00100)


@pytest.mark.parametrize("name,over", [
    ("a projection that halves the image and doubles the channels, then a plain block", {}),
    ("a projection on equal shapes", dict(dims=(3, 8, 8, 8, 5), n_conv=3, bn_mask=0b111, stride_mask=0,
                                          skip_mask=0b100, proj_mask=0b100)),
    ("a projection to fewer channels without stride, then a strided one; sides no powers of two", dict(
        dims=(4, 24, 16, 8, 8, 8, 16, 16, 5), n_conv=7, bn_mask=0b1111111, stride_mask=0b0100000,
        skip_mask=0b1010100, proj_mask=0b1000100, img_h=6, img_w=10)),
    ("projections on 32- to 64-channel images (unfolding inside the GEMM beside them)", dict(
        dims=(3, 32, 32, 32, 64, 64, 10), n_conv=5, bn_mask=0b11111, stride_mask=0b01000,
        skip_mask=0b10100, proj_mask=0b10000, n_classes=10, batch=4)),
    ("four stages of one block each, ResNet-18's shape in small", dict(
        dims=(3, 8, 8, 8, 16, 16, 32, 32, 64, 64, 10), n_conv=9, bn_mask=(1 << 9) - 1,
        stride_mask=0b010101000, skip_mask=0b101010100, proj_mask=0b101010000, img_h=16, img_w=16,
        n_classes=10, batch=4, K=3, tau=(2, 3, 4))),
])
def test_projection_shortcut_model_matches_oracle(name, over):
    w = PROJ_SMALL.scaled(**over)
    worst = run_mlp(w, 6, 1e-4, 1e-3, anchor_after=2)
    print("projection %s: worst parameter error %.3e" % (name, worst))


def test_projection_shortcut_gradients_group_by_group():
    """One step from the common start: the gradients of the projection's own parameters (W_p,
    gamma_p, beta_p; b_p exactly zero) and of every other group against the oracle's."""
    w = PROJ_SMALL.scaled(batch=16)
    g, o = make_pair(w)
    X, lab = workloads.batch(w, 0)
    Xd, ld = to_dev(X, lab, w)
    loss_d = torch.zeros(w.K, device=DEV)
    g.lsam_step(Xd, ld, loss_d)
    ol = o.step(X, lab)
    assert np.allclose(loss_d.cpu().numpy(), ol, rtol=1e-5)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-3)
    assert list(o.model.proj_offsets) == [2]
    p0, p1, p2, p3, p4 = o.model.proj_offsets[2]
    for i in range(w.K):
        g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        close_enough(g2[p0:p1], o.last_g2[i][p0:p1], 2e-3, "dW_p of replica %d" % i)
        close_enough(g2[p2:p3], o.last_g2[i][p2:p3], 2e-3, "dgamma_p of replica %d" % i)
        close_enough(g2[p3:p4], o.last_g2[i][p3:p4], 2e-3, "dbeta_p of replica %d" % i)
        assert np.all(g2[p1:p2] == 0.0) and np.max(np.abs(o.last_g2[i][p1:p2])) < 1e-12
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], 2e-3, "dW%d of replica %d" % (l + 1, i))
            if l in o.model.bn_offsets:
                b0, b1, b2 = o.model.bn_offsets[l]
                close_enough(g2[b0:b2], o.last_g2[i][b0:b2], 2e-3, "dgamma, dbeta %d of replica %d" % (l + 1, i))
    g.close()


def test_projection_shortcut_with_bf16_products_the_comparators_and_noise():
    w = PROJ_SMALL
    run_mlp(w.scaled(gemm_dtype=1, batch=16), 5, 2e-2, 2e-2, anchor_after=1, tol_flip=1e-1)
    run_mlp(w.scaled(algorithm=lsam.ALG_DATA_PARALLEL), 4, 1e-4, 1e-3, anchor_after=1)
    # the noise of the projection's four groups has counters of its own
    run_mlp(w.scaled(noise_scale=1e-3, noise_seed=11), 4, 1e-4, 1e-3, anchor_after=1)
    run_mlp(w.scaled(rho=0.0), 4, 1e-4, 1e-3, anchor_after=1)


def test_maximum_depth_residual_model():
    """LSAM_MAX_LAYERS = 40 layers: 39 convolutions (a stem and 19 blocks, three of them with a
    projection, bits above 31 of every mask in use) and one dense layer."""
    n_conv = 39
    dims = [3, 8]
    stride = proj = skip = 0
    for b in range(19):
        l = 1 + 2 * b
        c = 8 if b < 6 else 16 if b < 12 else 24
        if b in (6, 12, 17):
            proj |= 1 << (l + 1)
            if b != 17:
                stride |= 1 << l
        skip |= 1 << (l + 1)
        dims += [c, c]
    w = RES_SMALL.scaled(dims=tuple(dims) + (5,), n_conv=n_conv, bn_mask=(1 << n_conv) - 1, stride_mask=stride,
                         skip_mask=skip, proj_mask=proj, img_h=8, img_w=8, batch=4, noise_scale=1e-4,
                         noise_seed=3)
    assert len(w.dims) - 1 == 40 and proj >> 32 and skip >> 32
    worst = run_mlp(w, 3, 2e-4, 2e-3, anchor_after=1)
    print("40-layer residual model: worst parameter error %.3e" % worst)
    cfg, keep = lsam.config_from_workload(w.scaled(dims=tuple(dims) + (7, 5)))
    assert lsam.lsam_workspace_bytes(cfg) == 0 and "n_layers" in lsam.last_error()


# ---- pre-activation blocks (wide residual networks) ----------------------------------------------
def _wrn_small(widths, n, **over):
    dims, stride, skip, proj = [3, 8], 0, 0, 0
    l = 1
    for s, c in enumerate(widths):
        for b in range(n):
            if b == 0 and (s > 0 or c != 8):
                proj |= 1 << (l + 1)
            if b == 0 and s > 0:
                stride |= 1 << l
            skip |= 1 << (l + 1)
            dims += [c, c]
            l += 2
    kw = dict(dims=tuple(dims) + (5,), n_conv=l, bn_mask=(1 << l) - 1, stride_mask=stride, skip_mask=skip,
              proj_mask=proj, preact=1)
    kw.update(over)
    return RES_SMALL.scaled(**kw)


@pytest.mark.parametrize("name,w", [
    ("one identity block", _wrn_small((8,), 1)),
    ("a widening projection without stride, then an identity block", _wrn_small((16,), 2)),
    ("three stages of two blocks, WRN-16's shape in small", _wrn_small((16, 32, 64), 2, img_h=16, img_w=16, batch=4,
                                                                          K=3, tau=(2, 3, 4))),
    ("chained identity blocks (a sum's gradient travels down three shortcuts)", _wrn_small((8,), 4)),
    ("32- and 64-channel images (unfolding inside the GEMM)", _wrn_small((32, 64), 1, batch=4)),
])
def test_preactivation_model_matches_oracle(name, w):
    # with normalisation parameters that keep every ReLU decision away from zero the step must
    # agree to 1e-5; with the workload's own initialisation the one-step bound of the other
    # small convolutional models holds but for the last case, whose 64 to 256 positions per
    # channel make a single decision at rounding distance worth up to 1/64 of a gradient row
    tight = run_mlp(w, 6, 1e-5, 1e-5, anchor_after=2, init_fn=bn_away_from_zero)
    worst = run_mlp(w, 6, 1e-3 if "unfolding" in name else 1e-4, 1e-3, anchor_after=2)
    print("pre-activation %s: worst parameter error %.3e (decisions away from zero: %.3e)" % (name, worst, tight))


def test_preactivation_gradients_group_by_group_and_other_modes():
    w = _wrn_small((16, 32), 2, batch=16)
    g, o = make_pair(w)
    X, lab = workloads.batch(w, 0)
    Xd, ld = to_dev(X, lab, w)
    loss_d = torch.zeros(w.K, device=DEV)
    g.lsam_step(Xd, ld, loss_d)
    ol = o.step(X, lab)
    assert np.allclose(loss_d.cpu().numpy(), ol, rtol=1e-5)
    assert np.allclose(g.lsam_get_norms(), o.last_norm, rtol=1e-3)
    assert sorted(o.model.proj_offsets) == [2, 6]
    for i in range(w.K):
        g2 = g.lsam_get_buffer(lsam.BUF_GRAD, i)
        for l, (p0, p1, p2, p3, p4) in o.model.proj_offsets.items():
            assert p4 == p2
            close_enough(g2[p0:p1], o.last_g2[i][p0:p1], 2e-3, "dW_p %d of replica %d" % (l + 1, i))
            assert np.all(g2[p1:p2] == 0.0) and np.max(np.abs(o.last_g2[i][p1:p2])) < 1e-12
        for l, (o0, o1, o2) in enumerate(o.model.offsets):
            close_enough(g2[o0:o1], o.last_g2[i][o0:o1], 2e-3, "dW%d of replica %d" % (l + 1, i))
            if l in o.model.bn_offsets:
                b0, b1, b2 = o.model.bn_offsets[l]
                close_enough(g2[b0:b2], o.last_g2[i][b0:b2], 2e-3, "dgamma, dbeta %d of replica %d" % (l + 1, i))
    g.close()
    # bf16 products: a value that differs in its last fp32 bit between the two sides now and then
    # rounds to the other bfloat16 neighbour, a change of 2^-8 of that operand, and this model's
    # gradient is sensitive to it: the oracle's own gradient moves by 1e-2 to 4e-2 (3e-4 with
    # decisions away from zero) when gamma and beta are changed by 1e-7 of their size
    # (test_bf16_gradient_of_a_normalised_network_is_sensitive_to_the_last_bit).  Hence the
    # bounds: 1e-1 on gradients with decisions away from zero, 3e-1 with the natural start.
    run_mlp(w.scaled(gemm_dtype=1), 5, 2e-2, 2e-2, anchor_after=1, tol_flip=1e-1, init_fn=bn_away_from_zero)
    run_mlp(w.scaled(gemm_dtype=1), 5, 2e-2, 2e-2, anchor_after=1, tol_flip=3e-1)
    run_mlp(w.scaled(batch=6, algorithm=lsam.ALG_DATA_PARALLEL), 4, 1e-4, 1e-3, anchor_after=1)
    run_mlp(w.scaled(batch=6, noise_scale=1e-3, noise_seed=11), 4, 1e-4, 1e-3, anchor_after=1)


def test_residual_configurations_that_cannot_run_are_rejected():
    for over, msg in ((dict(skip_mask=0b010), "two convolutions below"),
                      (dict(bn_mask=0b011), "must be batch-normalised"),
                      (dict(pool_mask=0b010), "no pool"),
                      (dict(stride_mask=0b110), "does not fit"),
                      (dict(dims=(3, 16, 8, 8, 5)), "does not fit"),
                      (dict(stride_mask=0b1000), "no convolution"),
                      (dict(proj_mask=0b010), "closes no residual block"),
                      (dict(preact=1, bn_mask=0b110), "every convolution batch-normalised"),
                      (dict(preact=1, dims=(3, 8, 8, 16, 5)), "does not fit"),
                      (dict(preact=2), "preact must be"),
                      (dict(img_h=6, img_w=6, stride_mask=0b011), "even image sides")):
        cfg, keep = lsam.config_from_workload(RES_SMALL.scaled(**over))
        assert lsam.lsam_workspace_bytes(cfg) == 0, over
        assert msg in lsam.last_error(), (over, lsam.last_error())


def test_layer_info_reports_which_kernels_serve_a_layer():
    def table(w):
        cfg, keep = lsam.config_from_workload(w)
        eng = lsam.Lsam(cfg, workloads.init_params(w), device=DEV, keep=keep)
        out = [eng.lsam_layer_info(l) for l in range(len(w.dims) - 1)]
        with pytest.raises(lsam.LsamError):
            eng.lsam_layer_info(len(w.dims) - 1)
        eng.close()
        return out
    # fp32 MLP with a narrow head: GEMM layers, then the fused head kernels; gradients stored
    t = table(workloads.WORKLOADS["cfg1"])
    assert [r[0] for r in t] == [lsam.LAYER_DENSE, lsam.LAYER_HEAD] and all(r[2] == 0 for r in t)
    assert t[0][3:] == (32, 784, 128, 0, 0)
    # bf16 MLP: fused path; the Gram route only where 2 B (out + in) <= out in
    w = workloads.WORKLOADS["cfg3"].scaled(K=2, dims=(384, 256, 256, 40), batch=32, tau=(2, 3), n_classes=40)
    assert [r[2] for r in table(w)] == [2, 2, 1] and [r[2] for r in table(w.scaled(rho=0.0))] == [0, 0, 0]
    # convolutions: first-layer kernels, unfolding inside the GEMM, stored unfold (24 channels);
    # the input gradient of the 24-output layer goes through a stored unfolded gradient
    w = workloads.Workload("kinds", K=2, dims=(3, 32, 32, 24, 40, 10), batch=8, n_conv=4, img_h=8,
                           img_w=8, pool_mask=0b0110, tau=(2, 2), n_classes=10, data_seed=41)
    t = table(w)
    assert [r[0] for r in t] == [lsam.LAYER_CONV_FIRST, lsam.LAYER_CONV_DIRECT, lsam.LAYER_CONV_DIRECT,
                                 lsam.LAYER_CONV_STORED, lsam.LAYER_HEAD]
    assert [r[1] for r in t[:4]] == [0, 0, 1, 1] and [r[3] for r in t] == [512, 512, 128, 32, 8]


# ---- randomly drawn residual configurations -----------------------------------------------------------
def _random_residual_workload(rng):
    """A valid configuration drawn at random: a stem, then blocks that keep, halve or change
    the shape, closed by a parameter-free shortcut where that fits and by a projection where it
    does not (or by choice), plain convolutions and pools in between; post- or pre-activation."""
    preact = int(rng.integers(0, 2))
    chans = [8, 16, 24, 32]
    H0, W0 = int(rng.choice([8, 12, 16])), int(rng.choice([8, 16]))
    h, w = H0, W0
    dims = [int(rng.choice([2, 3, 4])), int(rng.choice(chans[:2]))]
    stride = skip = proj = pool = 0
    l = 1                                       # index of the next convolution
    for _ in range(int(rng.integers(1, 4))):
        cin, st = dims[-1], 1
        kind = rng.choice(["same", "widen", "halve", "narrow"])
        cout = cin
        if kind == "widen":
            cout = int(rng.choice([c for c in chans if c >= cin]))
        elif kind == "narrow":
            cout = int(rng.choice([c for c in chans if c <= cin]))
        elif kind == "halve" and h % 2 == 0 and w % 2 == 0 and min(h, w) >= 4:
            st, cout = 2, int(rng.choice([c for c in chans if c >= cin]))
            h, w = h // 2, w // 2
        if st == 2:
            stride |= 1 << l
        dims += [cout, cout]
        skip |= 1 << (l + 1)
        fits_plain = (cout == cin and st == 1) if preact else cout >= cin
        if not fits_plain or rng.integers(0, 3) == 0:
            proj |= 1 << (l + 1)
        l += 2
        if not preact and rng.integers(0, 4) == 0:
            # a plain convolution between two blocks, with a pool when the image allows; a block's
            # input has to be a convolution's ReLU output, so a pool is followed by one more
            dims.append(int(rng.choice(chans)))
            l += 1
            if h % 2 == 0 and w % 2 == 0 and min(h, w) >= 4 and rng.integers(0, 2) == 0:
                pool |= 1 << (l - 1)
                h, w = h // 2, w // 2
                dims.append(int(rng.choice(chans)))
                l += 1
    gap = int(rng.integers(0, 2)) if h * w * dims[-1] <= 512 else 1
    classes = int(rng.choice([3, 5, 10]))
    dense = [classes] if rng.integers(0, 2) else [int(rng.choice([12, 20])), classes]
    K = int(rng.integers(1, 4))
    return workloads.Workload(
        "rand_res", K=K, dims=tuple(dims + dense), batch=int(rng.choice([3, 4, 6])), n_conv=l, img_h=H0, img_w=W0,
        bn_mask=(1 << l) - 1, stride_mask=stride, skip_mask=skip, proj_mask=proj, pool_mask=pool, preact=preact,
        global_avg_pool=gap, rho=0.05, lr=0.05, tau=tuple(int(t) for t in rng.integers(1, 4, K)),
        n_classes=classes, data_seed=int(rng.integers(1, 1000)))


@pytest.mark.parametrize("seed", range(24))
def test_randomly_drawn_residual_configurations_match_oracle(seed):
    w = _random_residual_workload(np.random.default_rng(1000 + seed))
    cfg, keep = lsam.config_from_workload(w)
    assert lsam.lsam_workspace_bytes(cfg) > 0, (w, lsam.last_error())
    # decisions away from zero: the step has to agree to 1e-5 whatever the structure
    worst = run_mlp(w, 4, 1e-5, 1e-5, anchor_after=2, init_fn=bn_away_from_zero)
    print("seed %d: %d convolutions, preact=%d, skip=%s, proj=%s, stride=%s, pool=%s, gap=%d, K=%d: %.2e"
          % (seed, w.n_conv, w.preact, bin(w.skip_mask), bin(w.proj_mask), bin(w.stride_mask), bin(w.pool_mask),
             w.global_avg_pool, w.K, worst))


@pytest.mark.parametrize("seed", range(8))
def test_randomly_drawn_residual_configurations_with_bf16_products(seed):
    """The same draw with both operands of every matrix product rounded to bf16 on their way into
    the matrix unit: 2e-2 on the parameters, step by step from the oracle's state.  (The bf16
    gradient of a normalised network moves by percent when an operand moves by its last bit, see
    the oracle's pin of that, hence the looser bound on gradients and velocities.)"""
    w = _random_residual_workload(np.random.default_rng(1000 + seed)).scaled(gemm_dtype=1)
    worst = run_mlp(w, 4, 2e-2, 2e-2, anchor_after=1, tol_flip=3e-1, init_fn=bn_away_from_zero)
    print("seed %d, bf16 products: %d convolutions, preact=%d, K=%d: %.2e" % (seed, w.n_conv, w.preact, w.K, worst))


# ---- iterate sums restart after a center update without being zeroed in memory ----------------------
def _restart_case(kind):
    if kind == "raw":
        w = workloads.WORKLOADS["cfg4"].scaled(name="restart_raw", K=3, d_raw=4099, tau=(1, 2, 3))
        g, o = make_pair(w)
        rng = np.random.default_rng(5)
        def step(t):
            g1 = (rng.standard_normal((w.K, w.d_raw)) * 1e-2).astype(np.float32)
            g2 = (rng.standard_normal((w.K, w.d_raw)) * 1e-2).astype(np.float32)
            g.lsam_step_grads(torch.from_numpy(g1).to(DEV), torch.from_numpy(g2).to(DEV))
            o.step_grads(g1.astype(np.float64), g2.astype(np.float64))
        return w, g, o, step
    dt = {"fp32": 0, "bf16": 1}[kind]
    w = workloads.WORKLOADS["cfg3"].scaled(name="restart_" + kind, K=3, dims=(40, 72, 100, 9), batch=20, tau=(1, 2, 3),
                                           n_classes=9, batch_pool=0, gemm_dtype=dt)
    g, o = make_pair(w)
    def step(t):
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        g.lsam_step(Xd, ld, None)
        o.step(X, lab)
    return w, g, o, step


@pytest.mark.parametrize("kind", ["raw", "fp32", "bf16"])
def test_iterate_sums_restart_after_a_center_update(kind):
    """A replica the center update has just served reads back an iterate sum of exact zeros, the
    others keep theirs; one step later its sum is exactly its new parameters (0 + x); a replica
    served at every tick (period 1) goes through that at every step; a sum written through the
    boundary right after a center update counts from what was written."""
    w, g, o, step = _restart_case(kind)
    for t in range(7):
        step(t)
        before = [g.lsam_get_buffer(lsam.BUF_ITER_SUM, i) for i in range(w.K)]
        count = g.lsam_get_schedule()[1]
        due = [i for i in range(w.K) if count[i] >= w.tau[i]]
        assert g.lsam_sync() == o.sync() == len(due)
        for i in range(w.K):
            S = g.lsam_get_buffer(lsam.BUF_ITER_SUM, i)
            if i in due:
                assert not np.any(S), (t, i)
            else:
                assert np.array_equal(S, before[i]) and np.any(S), (t, i)
            assert not np.any(o.S[i]) or rel_max(S, o.S[i]) < (2e-2 if kind == "bf16" else 1e-4), (t, i)
        if t == 3:
            # replica 1 was served at this tick (period 2): give it a sum of its own choosing
            assert 1 in due
            z = np.linspace(-1.0, 1.0, g.lsam_get_params(1).size).astype(np.float32)
            g.lsam_set_buffer(lsam.BUF_ITER_SUM, 1, z)
            o.S[1] = z.astype(np.float64)
            assert np.array_equal(g.lsam_get_buffer(lsam.BUF_ITER_SUM, 1), z)
    step(7)
    # replica 0 (period 1) was served at tick 6: its sum is its parameters, bit for bit
    assert np.array_equal(g.lsam_get_buffer(lsam.BUF_ITER_SUM, 0), g.lsam_get_params(0))
    for i in range(w.K):
        assert rel_max(g.lsam_get_buffer(lsam.BUF_ITER_SUM, i), o.S[i]) < (2e-2 if kind == "bf16" else 1e-4), i
    g.close()

