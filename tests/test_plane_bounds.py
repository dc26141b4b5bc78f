"""That the bounds of tests/test_gpu_plane_products.py reject what they are for: mistakes of the kind a
wrong kernel makes, planted in the oracle.  A product loses one tap, its last ragged tile of pixels, or
a group of the gradient is not written; at least one group must then be off by more than its bound."""
import numpy as np
import pytest

import workloads
from test_gpu_plane_products import NETS, group_bounds, groups, jittered, net, spread
from util import oracle_from


def roles(w):
    """What the oracle rounds, call by call, in one forward and backward pass: (layer, operand)."""
    out = []
    convs, dense = range(w.n_conv), range(w.n_conv, len(w.dims) - 1)
    for l in convs:
        out += [(l, "image"), (l, "filters")] + [(l, "proj image"), (l, "proj filters")] * ((w.proj_mask >> l) & 1)
    for l in dense:
        out += [(l, "dense")] * 2
    for l in reversed(dense):
        out += [(l, "dense")] * 4
    for l in reversed(convs):
        out += [(l, "proj dW gradient"), (l, "proj dW image"), (l, "proj dX gradient"), (l, "proj dX filters")] * ((w.proj_mask >> l) & 1)
        out += [(l, "dW gradient"), (l, "dX gradient"), (l, "dW image"), (l, "dX filters")]
    return out


def tap_lost(a):
    a[:, 0, 2] = 0.0


def tile_lost(a):
    """The last ragged tile: what 128 pixels leave over, or one tile of 128."""
    rows = a.reshape(-1, a.shape[-1])
    rows[-(len(rows) % 128 or 128):] = 0.0


def bottom_lost(a):
    """The same of an image with its rim: the last image's lower half."""
    a[-1, a.shape[1] // 2:] = 0.0


def gradient(w, X, lab, plant=None, seed=None):
    """The oracle's gradient, with `plant` = ((layer, operand), change) or jitter."""
    o = oracle_from(w.scaled(K=1, tau=(2,)), spread(w))
    if seed is not None:
        jittered(o, seed)
    if plant is not None:
        where, change = plant
        order, q = iter(roles(w)), o.model.q
        seen = []

        def planted(a):
            out = q(a)
            if next(order) == where:
                out = np.array(out)
                change(out)
                seen.append(1)
            return out
        o.model.q = planted
    g = o.model.loss_and_grad(np.asarray(spread(w), np.float64), X[0], lab[0])[1]
    if plant is not None:
        assert seen == [1] and next(order, None) is None
    return np.asarray(g)


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", ["33 wide", "8 and 16 channels", "stride and projection", "pre-activation",
                                  "pools, no normalisation"])
def test_bounds_reject_planted_mistakes(name, bf16):
    w = net(bf16=bf16, **NETS[name])
    X, lab = workloads.batch(w, 0)
    ref = gradient(w, X, lab)
    moved = [gradient(w, X, lab, seed=s) for s in range(2 if bf16 else 0)]
    bounds = group_bounds(w, ref, moved)

    def over(g):
        """The largest error of a group in units of its bound."""
        return max(np.linalg.norm(g[lo:hi] - ref[lo:hi]) / b for (lo, hi), b in zip(groups(w), bounds) if b)

    weakest = {}
    for at, ((lo, hi), b) in enumerate(zip(groups(w), bounds)):
        if b:
            g = ref.copy()
            g[lo:hi] = 0.0
            weakest["group %d not written" % at] = over(g)
    at = 0
    for l, (fan_in, fo) in enumerate(w.layer_shapes[:w.n_conv]):
        g = ref.copy()
        g[groups(w)[at][0]:groups(w)[at][1]].reshape(fo, 9, -1)[:, 2] = 0.0
        weakest["dW of layer %d without a tap" % l] = over(g)
        at += 2 + 2 * ((w.bn_mask >> l) & 1) + (0 if not (w.proj_mask >> l) & 1 else 2 if w.preact else 4)
    for where in roles(w):
        l, what = where
        changes = {"filters": tap_lost if l else None, "dX filters": None, "image": bottom_lost, "dW gradient": tile_lost,
                   "dX gradient": tile_lost if l else None, "proj dW gradient": tile_lost, "proj dX gradient": tile_lost,
                   "proj image": bottom_lost}
        change = changes.get(what)
        if change is not None:
            weakest["%s of layer %d: %s" % (what, l, change.__name__)] = over(gradient(w, X, lab, (where, change)))
    print(name, bf16, sorted((round(v, 1), k) for k, v in weakest.items())[:4])
    assert min(weakest.values()) > 1.0, sorted((v, k) for k, v in weakest.items())[:6]
