"""The convolution products on plane tensors (one bfloat16 plane, or the exact three-plane split of
fp32) against the CPU oracle, at the edges of their tiles: patches that touch several images, image
widths that do and do not divide a tile, ragged tile rows, channel counts with a tap per k-step,
several taps per k-step and odd remainders, one and several column tiles, split contractions,
strides, 1x1 projections, and infinite operands.

The layers are large enough for the plane products (3e8 multiply-adds each, 1e8 up to 32 channels).
Normalisation parameters keep ReLU decisions away from zero.  Every parameter group is compared twice:
  by the whole gradient's norm: an fp32 sum of n = 4e4 terms is good to sqrt(n) 2^-24 = 1.2e-5 of the norm
    of its terms, which lie below the whole (bound 3e-6; the fp32-storage products measure up to 6e-7; with
    bf16 products, where a last fp32 bit decides a bfloat16 neighbour, 2^-8 of an operand, 1e-3);
  by its own (group_bounds), which for a group in front of a normalisation is 1e-2 to 1e-5 of the whole:
    most of its terms cancel.
tests/test_plane_bounds.py plants mistakes in the oracle and shows that these bounds reject them."""
import numpy as np
import pytest
import torch

import workloads
from paper_2509_03110_amd import lsam
from util import bn_away_from_zero, oracle_from, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def net(dims, side, batch, K=2, stride=0, skip=0, proj=0, preact=0, bf16=0, pool=0, bn=1):
    n = len(dims) - 2
    return workloads.Workload("planes", K=K, dims=dims, batch=batch, n_conv=n, img_h=side[0], img_w=side[1],
                              bn_mask=(1 << n) - 1 if bn else 0, stride_mask=stride, skip_mask=skip, proj_mask=proj, preact=preact,
                              pool_mask=pool, global_avg_pool=1, gemm_dtype=bf16, tau=(2,) * K, rho=0.05, lr=0.02,
                              n_classes=dims[-1], data_seed=77)


def groups(w):
    """(first, last) of every parameter group of the flat vector."""
    at, out = 0, []
    for l, (fan_in, fo) in enumerate(w.layer_shapes):
        sizes = [fan_in * fo, fo]
        if l < w.n_conv:
            if (w.bn_mask >> l) & 1:
                sizes += [fo, fo]
            if (w.proj_mask >> l) & 1:
                sizes += [fo * w.dims[l - 1], fo] + ([] if w.preact else [fo, fo])
        for n in sizes:
            out.append((at, at + n))
            at += n
    assert at == w.d
    return out


def step_both(w, X=None):
    init = spread(w)
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    Xb, lab = workloads.batch(w, 0)
    X = Xb if X is None else X(Xb)
    loss = torch.zeros(w.K, device=DEV)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), loss)
    with np.errstate(all="ignore"):
        ol = o.step(X, lab)
    return g, o, loss.cpu().numpy(), np.asarray(ol)


def spread(w):
    """Initial parameters whose normalised layers keep three channels of four positive everywhere and
    the fourth negative everywhere (gamma 0.25, beta +-1.5; shortcuts agree in sign).  Without
    normalisation: weights a fifth of their size and biases +-1, eight spreads from zero."""
    init = bn_away_from_zero(w, workloads.init_params(w))
    model = oracle_from(w.scaled(K=1, tau=(1,)), init).model
    if not w.bn_mask:
        at = 0
        for fan_in, fo in w.layer_shapes[:w.n_conv]:
            init[at:at + fan_in * fo] *= 0.2
            at += fan_in * fo
            init[at:at + fo] = np.where(np.arange(fo) % 4 == 3, -1.0, 1.0)
            at += fo
    ranges = [(b1, b2) for b0, b1, b2 in model.bn_offsets.values()]
    ranges += [(p[3], p[4]) for p in model.proj_offsets.values()]
    for lo, hi in ranges:
        init[lo:hi] = np.where(np.arange(hi - lo) % 4 == 3, -1.5, 1.5)
    return init


NETS = {
    # a 32-wide image: tiles of whole rows; 20 rows: a tile may end one image and begin the next
    "32 wide, 64 channels": dict(dims=(3, 64, 64, 64, 10), side=(20, 32), batch=7),
    # 16-wide: several images per patch, ragged last tile; one 32-channel block, two column tiles
    "16 wide, 32 to 96 channels": dict(dims=(3, 32, 96, 32, 10), side=(16, 16), batch=23),
    # widths that do not divide a tile, odd heights
    "28 wide": dict(dims=(3, 32, 64, 64, 10), side=(7, 28), batch=43),
    "33 wide": dict(dims=(3, 64, 64, 10), side=(5, 33), batch=27),
    # images smaller than a tile row: many per patch, or (2 x 2) too many: the ring
    "4 wide": dict(dims=(3, 64, 128, 64, 10), side=(4, 4), batch=131),
    "2 wide": dict(dims=(3, 64, 128, 64, 10), side=(2, 2), batch=521),
    "8 wide, 160 channels": dict(dims=(3, 32, 160, 160, 10), side=(8, 8), batch=53),
    # four and two taps per k-step, an unfolded first layer of 45 values, small column tiles
    "8 and 16 channels": dict(dims=(5, 8, 16, 16, 10), side=(32, 32), batch=45),
    # a channel count that needs a stored unfolded image (taken with one plane only)
    "24 channels": dict(dims=(3, 24, 64, 24, 10), side=(16, 32), batch=22),
    # stride 2 forward and dW by address, dX in classes of pixels; both kinds of shortcut
    "stride and projection": dict(dims=(3, 32, 64, 64, 10), side=(32, 32), batch=33, stride=0b010, skip=0b100, proj=0b100),
    "stride, columns that leave a tile half empty": dict(dims=(3, 96, 64, 32, 10), side=(16, 16), batch=90, stride=0b010),
    "parameter-free shortcut": dict(dims=(3, 64, 64, 64, 10), side=(16, 16), batch=17, skip=0b100),
    # sums in front of the normalisation: a projection and an identity, pools
    "pre-activation": dict(dims=(3, 32, 64, 64, 64, 64, 10), side=(16, 32), batch=65, stride=0b00010, skip=0b10100,
                           proj=0b00100, preact=1),
    "pools": dict(dims=(3, 32, 64, 64, 10), side=(16, 32), batch=129, pool=0b011),
    # no normalisation: a kernel of its own writes the gradient's planes, below a pool and elsewhere
    "pools, no normalisation": dict(dims=(3, 32, 64, 64, 64, 10), side=(16, 32), batch=129, pool=0b0011, bn=0),
}


def jittered(o, seed):
    """The oracle with every operand of every product off by up to four last fp32 bits."""
    rng, q = np.random.default_rng(seed), o.model.q
    o.model.q = lambda a: q(a * (1 + rng.uniform(-2.0**-22, 2.0**-22, np.shape(a))))
    return o


def group_bounds(w, ref, moved):
    """Largest error of every group of `ref`, as a norm.  fp32: 1.2e-5 of the norm of the terms, which in front
    of a normalisation cancel to a hundredth or less (bound 1e-3 of what they leave, measured up to 2e-4;
    without normalisation 3e-6, measured 1.3e-7).  bf16 products: what last fp32 bits decide, four times
    the distance of `moved`, gradients of jittered oracles, from `ref` (measured up to 2.3 times), and at
    least bfloat16's own rounding, 2^-9, of the group.  Biases in front of a normalisation are exactly zero."""
    out = []
    for lo, hi in groups(w):
        own = np.linalg.norm(ref[lo:hi])
        if own < 1e-12 * np.linalg.norm(ref):
            out.append(0.0)
        elif w.gemm_dtype:
            out.append(max([2.0**-9 * own] + [4 * np.linalg.norm(m[lo:hi] - ref[lo:hi]) for m in moved]))
        else:
            out.append((1e-3 if w.bn_mask else 3e-6) * own)
    return out


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_plane_products_match_oracle(name, bf16):
    w = net(bf16=bf16, **NETS[name])
    g, o, loss, ol = step_both(w)
    assert np.allclose(loss, ol, rtol=2e-2 if bf16 else 1e-5)
    moved = []
    for seed in range(2 if bf16 else 0):
        moved.append(jittered(oracle_from(w, spread(w)), seed))
        moved[-1].step(*workloads.batch(w, 0))
    worst, own = 0.0, 0.0
    for i in range(w.K):
        g2, ref = g.lsam_get_buffer(lsam.BUF_GRAD, i), np.asarray(o.last_g2[i])
        bounds = group_bounds(w, ref, [np.asarray(m.last_g2[i]) for m in moved])
        for at, ((lo, hi), bound) in enumerate(zip(groups(w), bounds)):
            e = np.linalg.norm(g2[lo:hi] - (ref[lo:hi] if bound else 0.0))
            worst, own = max(worst, e / np.linalg.norm(ref)), max(own, e / bound if bound else 0.0)
            assert e <= bound, "group %d: error %.2e, bound %.2e" % (at, e, bound)
        assert rel_l2(g.lsam_get_params(i), o.get_params(i)) <= (1e-4 if bf16 else 1e-6)
    print("%s bf16=%d: worst group %.2e of the whole, %.2f of its bound" % (name, bf16, worst, own))
    assert worst <= (1e-3 if bf16 else 3e-6)
    g.close()


def test_layer_info_reports_planes():
    """Layers that the plane products serve say so: by size, and in fp32 arithmetic by channel count."""
    def table(w):
        cfg, keep = lsam.config_from_workload(w)
        g = lsam.Lsam(cfg, workloads.init_params(w), device=DEV, keep=keep)
        out = [g.lsam_layer_planes(l) for l in range(len(w.dims) - 1)]
        assert all(len(g.lsam_layer_info(l)) == 8 for l in range(len(w.dims) - 1))
        g.close()
        return out
    over = dict(dims=(3, 32, 64, 24, 64, 10), side=(16, 32), batch=40)
    assert table(net(**over)) == [0, 3, 0, 0, 0]
    assert table(net(bf16=1, **over)) == [0, 1, 1, 1, 0]
    assert table(net(**dict(over, batch=2))) == [0, 0, 0, 0, 0]


@pytest.mark.parametrize("name", ["32 wide, 64 channels", "8 and 16 channels", "2 wide"])
def test_infinite_operands(name):
    """An infinite pixel, without normalisation and with positive weights, stays infinite (never infinity
    less infinity) up to the loss; the other replica is computed as ever, and so is the step after the
    state is restored."""
    net_of = dict(NETS[name])
    w = net(**net_of).scaled(bn_mask=0)
    init = np.abs(workloads.init_params(w)) * 0.1
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    X, lab = workloads.batch(w, 0)
    bad = X.copy()
    bad.reshape(w.K, -1)[0, 0] = np.inf
    loss = torch.zeros(w.K, device=DEV)
    ol = o.step(X, lab)
    for pixels in (bad, X):
        for i in range(w.K):
            g.lsam_set_buffer(lsam.BUF_PARAMS, i, init)
            g.lsam_set_buffer(lsam.BUF_VELOCITY, i, np.zeros(w.d, np.float32))
        g.lsam_step(torch.from_numpy(pixels).to(DEV), torch.from_numpy(lab).to(DEV), loss)
        first = 1 if pixels is bad else 0
        assert np.isfinite(loss.cpu().numpy()).tolist() == [pixels is X, True]
        for i in range(first, w.K):
            assert np.isclose(loss[i].item(), ol[i], rtol=1e-5)
            assert rel_l2(g.lsam_get_buffer(lsam.BUF_GRAD, i), o.last_g2[i]) <= 3e-6
    g.close()


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name,over", [
    ("32 wide, 64 channels", dict(bn=0)), ("16 wide, 32 to 96 channels", dict(bn=0)), ("2 wide", dict(bn=0)),
    ("8 and 16 channels", dict(bn=0)), ("24 channels", dict(bn=0)), ("pools, no normalisation", {}),
    ("stride and projection", dict(bn=0, skip=0, proj=0)), ("stride and projection", {}), ("pre-activation", {}),
])
def test_infinite_operands_of_one_replica_leave_no_trace(name, over, bf16):
    """What an infinite pixel does to one replica is its own affair: the other's gradient and loss are the
    same bit for bit, and so are both in the next step, once the state is restored.  (Normalised
    layers turn infinity into NaN, and the ReLU that into 0: the others hand it on.)"""
    w = net(bf16=bf16, **dict(NETS[name], **over))
    init = spread(w)
    cfg, keep = lsam.config_from_workload(w)
    g = lsam.Lsam(cfg, init, device=DEV, keep=keep)
    X, lab = workloads.batch(w, 0)
    bad = X.copy()
    bad.reshape(w.K, -1)[0, 5] = np.inf
    lab = torch.from_numpy(lab).to(DEV)
    seen = []
    for pixels in (X, bad, X):
        for i in range(w.K):
            g.lsam_set_buffer(lsam.BUF_PARAMS, i, init)
            g.lsam_set_buffer(lsam.BUF_VELOCITY, i, np.zeros(w.d, np.float32))
        loss = torch.zeros(w.K, device=DEV)
        g.lsam_step(torch.from_numpy(pixels).to(DEV), lab, loss)
        seen.append([np.append(g.lsam_get_buffer(lsam.BUF_GRAD, i), loss[i].item()) for i in range(w.K)])
    first, poisoned, after = seen
    assert not np.all(np.isfinite(poisoned[0]))
    assert np.array_equal(poisoned[1], first[1])
    assert np.array_equal(after[0], first[0]) and np.array_equal(after[1], first[1])
    g.close()


@pytest.mark.parametrize("dims,side,batch", [((32, 64, 10), (16, 16), 33), ((64, 64, 10), (2, 2), 1100), ((16, 16, 10), (32, 32), 45)])
@pytest.mark.parametrize("exponent,bound", [(-100, 3e-6), (-118, 3e-6 + 2.0**-16)])
def test_small_operands(dims, side, batch, exponent, bound):
    """The split of a number is exact down to 2^-110; below, an operand is off by up to 2^-134, here 2^-16
    of pixels at 2^-118.  (Weight gradient of a layer that reads such pixels; the classifier's
    weights bring the other operand up, so that no product falls among the subnormal numbers.)"""
    w = net(dims, side, batch, bn=0).scaled(rho=0.0)
    init = spread(w)
    init[-(dims[1] * 10 + 10):-10] *= np.float32(2.0**30)
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    X, lab = workloads.batch(w, 0)
    X = X * np.float32(2.0**exponent)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), torch.zeros(w.K, device=DEV))
    o.step(X, lab)
    n = 9 * dims[0] * dims[1]
    for i in range(w.K):
        err = rel_l2(g.lsam_get_buffer(lsam.BUF_GRAD, i)[:n], np.asarray(o.last_g2[i])[:n])
        print("%s 2^%d: %.2e" % (dims, exponent, err))
        assert err <= bound
    g.close()


# x = m 2^e with a rounding to bfloat16 that goes up, so that the product of the leading pieces of two
# such numbers is too large and the small products are negative
M = 1 + 2.0**-7 - 2.0**-10


@pytest.mark.parametrize("product", ["forward", "input gradient", "weight gradient"])
@pytest.mark.parametrize("c0,c1,side,batch,stride", [
    (32, 64, 16, 32, 0),         # patches, 64-wide
    (32, 32, 16, 64, 0),         # patches, up to 32 columns
    (16, 16, 32, 64, 0),         # 16 channels: weight gradient through the ring
    (64, 64, 2, 1100, 0),        # images too small for a patch: the ring
    (8, 8, 32, 90, 0),           # several taps per k-step
    (64, 64, 32, 32, 0b10),      # stride 2, input gradient in pixel classes
])
def test_finite_operands_whose_products_overflow(c0, c1, side, batch, stride, product):
    """Every term of the overflowing sums is positive and above the largest float, so each result is
    +infinity, in the forward products (an infinite activation reaches the loss; NaN would end as the
    ReLU's zero), in the input gradient (seen in the bias gradient of the layer below) and in the
    weight gradient.  The other replica, of ordinary numbers, stays finite."""
    w = net((c0, c1, c1, 10), (side, side), batch, stride=stride, bn=0).scaled(rho=0.0)
    lab = np.ones((w.K, batch), np.int32)
    ones = np.ones((w.K, batch, side, side, c0), np.float32)
    shapes, rows = w.layer_shapes, batch * (side // (2 if stride else 1))**2

    def run(x, w1, w2, w3):
        """Gradient of replica 0 by layer, and the losses, with constant data and weights."""
        X = ones * np.float32(M)
        X[0] *= np.float32(x)
        init = np.concatenate([np.concatenate([np.full(fi * fo, v, np.float32), np.zeros(fo, np.float32)])
                               for (fi, fo), v in zip(shapes, (w1 * M, w2 * M, 0.0))])
        init[-shapes[2][0] * 10 - 10:][:shapes[2][0]] = w3 * M      # class 0 of the dense layer
        cfg, keep = lsam.config_from_workload(w)
        g = lsam.Lsam(cfg, init, device=DEV, keep=keep)
        loss = torch.zeros(w.K, device=DEV)
        g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), loss)
        grad = g.lsam_get_buffer(lsam.BUF_GRAD, 0)
        g.close()
        out, at = [], 0
        for fi, fo in shapes:
            out.append((grad[at:at + fi * fo].reshape(fo, fi), grad[at + fi * fo:at + fi * fo + fo]))
            at += fi * fo + fo
        return out, loss.cpu().numpy()

    # the second layer's output is ordinary, its gradient comes down at 2^70 a pixel
    up = 2.0**70 * rows
    if product == "forward":             # 9 c0 terms of 2^140 in the first layer, of 2^70 in the other replica
        _, loss = run(2.0**70, 2.0**70, 2.0**-80, 2.0**-10)
        assert not np.isfinite(loss[0]) and np.isfinite(loss[1])
    elif product == "input gradient":    # 2^70 2^70
        grads, _ = run(1.0, 2.0**-70, 2.0**70, up)
        assert np.all(grads[0][1] == np.inf)
    else:                                # 2^70 2^70, activations of the first layer at 2^70
        grads, _ = run(1.0, 2.0**70, 2.0**-70, up)
        assert np.all(grads[1][0] == np.inf)


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("c,batch", [(8, 350), (16, 90)])
def test_infinite_filter_stays_in_its_class_of_pixels(c, batch, bf16):
    """An infinite filter of a stride-2 layer enters the input gradient of the pixels its tap meets and of
    no other (with 8 or 16 channels the classes of pixels share k-steps).  The filter, -infinity at
    row 1, column 2, belongs to an output that is dead, and the pixels it meets are dead in the
    layer below, whose ReLU drops the NaN of 0 times infinity: every gradient is what it is with a
    filter of zeros."""
    w = net((c, c, c, 10), (32, 32), batch, stride=0b10, bf16=bf16, bn=0).scaled(rho=0.0)
    X = np.ones((w.K, batch, 32, 32, c), np.float32)
    X[:, :, 0::2, 1::2] = -1.0                                     # seen by (1, 2): even rows, odd columns
    lab = np.zeros((w.K, batch), np.int32)
    n = 9 * c * c
    grads = []
    for filt in (0.0, -np.inf):
        rng = np.random.default_rng(3)
        init = rng.uniform(0.01, 0.1, w.d).astype(np.float32)
        first, second = init[:n].reshape(c, 9, c), init[n + c:2 * n + c].reshape(c, 9, c)
        first[:, [0, 1, 2, 3, 5, 6, 7, 8]] = 0.0                   # the pixel itself only
        init[n:n + c] = 0.0
        second[0] = 0.0
        second[0, 5] = filt
        init[2 * n + c] = -1.0                                     # output 0: dead
        cfg, keep = lsam.config_from_workload(w)
        g = lsam.Lsam(cfg, init, device=DEV, keep=keep)
        loss = torch.zeros(w.K, device=DEV)
        g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), loss)
        assert np.all(np.isfinite(loss.cpu().numpy()))
        grads.append(g.lsam_get_buffer(lsam.BUF_GRAD, 0))
        g.close()
    assert np.any(grads[0][:n]) and np.array_equal(grads[1], grads[0])


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", ["8 and 16 channels", "stride and projection", "pre-activation", "pools, no normalisation"])
def test_captured_and_concurrent_steps(name, bf16):
    """Four steps of a captured graph, with eager work and synchronisations between the replays, and four
    steps of each of two contexts on streams of their own, side by side, leave what four eager steps
    leave, bit for bit."""
    w = net(bf16=bf16, **NETS[name]).scaled(tau=(100, 100))
    init = spread(w)
    X, lab = (torch.from_numpy(t).to(DEV) for t in workloads.batch(w, 0))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(device=DEV) for _ in range(4)]
    cfg, keep = lsam.config_from_workload(w)
    eager, captured, one, two = (lsam.Lsam(cfg, init, device=DEV, keep=keep, stream=st) for st in streams)
    losses = [torch.zeros(w.K, device=DEV) for _ in range(4)]
    torch.cuda.synchronize()
    for _ in range(4):
        eager.lsam_step(X, lab, losses[0])
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[1]):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=streams[1]):
            captured.lsam_step(X, lab, losses[1])
        scratch = torch.zeros(1 << 20, device=DEV)
        for _ in range(4):
            graph.replay()
            scratch.add_(1.0)
            streams[1].synchronize()
    for _ in range(4):
        one.lsam_step(X, lab, losses[2])
        two.lsam_step(X, lab, losses[3])
    torch.cuda.synchronize()
    for g, loss in zip((captured, one, two), losses[1:]):
        assert torch.equal(loss, losses[0])
        for i in range(w.K):
            for which in (lsam.BUF_PARAMS, lsam.BUF_VELOCITY, lsam.BUF_ITER_SUM, lsam.BUF_GRAD):
                assert np.array_equal(g.lsam_get_buffer(which, i), eager.lsam_get_buffer(which, i)), (i, which)
    for g in (eager, captured, one, two):
        g.close()
