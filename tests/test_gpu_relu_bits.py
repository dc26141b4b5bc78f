"""Normalised convolutions whose outputs are kept as planes and sign bits, with and without the floats beside them, and whose
column sums are taken where the products are written: chains, ragged last tiles, shortcuts that read the floats, projections,
products cut over workgroups, whose sums kernels of their own take; pools joined with the normalisation in front of them or
behind a bare ReLU, and the global average with and without a shortcut that hands its gradient on.

Unlike the nets of test_gpu_plane_products.py half of all values are rectified, pixel by pixel, so a bit of another pixel
or channel shows: half of the gradient's terms would be wrong.  In fp32 no value lies where rounding decides: the shift of
every channel (the normalisation's, without one the bias) goes to the middle of the widest gap between the channel's values
around zero, 2.6e-4 or more on either side where fp32 sums are good to some 1e-6, and data are taken whose pooled windows have
their largest values 4e-6 apart; rho is 0, so that both passes take the same decisions.  Every parameter group is then held as in
test_gpu_plane_products.py.  With operands
rounded to bfloat16 decisions within 2^-8 differ, of which the gradient's norm shows sqrt(2^-8) = 6e-2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle.lsam_oracle  # noqa: E402
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402
from test_gpu_plane_products import DEV, group_bounds, groups, net  # noqa: E402
from util import oracle_from, rel_l2  # noqa: E402

pytestmark = pytest.mark.gpu

NETS = {
    "chain": dict(dims=(3, 32, 64, 32, 10), side=(16, 32), batch=24),
    "chain, products cut over workgroups": dict(dims=(3, 128, 128, 128, 10), side=(8, 8), batch=64),
    "ragged tiles": dict(dims=(3, 40, 72, 40, 10), side=(18, 14), batch=37),
    "pools": dict(dims=(3, 32, 40, 64, 10), side=(16, 28), batch=27, pool=0b011),
    "pool at the end": dict(dims=(3, 64, 32, 10), side=(12, 20), batch=40, pool=0b010),
    "pools without normalisation": dict(dims=(3, 32, 40, 64, 10), side=(16, 24), batch=31, pool=0b111, bn=0),
    "small layers": dict(dims=(5, 8, 24, 8, 10), side=(8, 12), batch=9, pool=0b101),
    "pools on the fp32-storage product": dict(dims=(8, 32, 48, 10), side=(8, 12), batch=9, pool=0b01, bn=0),
    "pool behind a block": dict(dims=(3, 32, 32, 32, 48, 10), side=(16, 32), batch=24, skip=0b0100, pool=0b0100),
    "pool behind a pre-activation block": dict(dims=(3, 32, 32, 32, 48, 10), side=(16, 32), batch=24, skip=0b0100, pool=0b0100, preact=1),
    "average behind a shortcut": dict(dims=(3, 32, 32, 32, 10), side=(16, 20), batch=24, skip=0b100),
    "average of few positions behind a shortcut": dict(dims=(3, 32, 32, 32, 10), side=(4, 4), batch=300, skip=0b100),
    "average of few positions behind a projection": dict(dims=(3, 24, 48, 48, 10), side=(8, 8), batch=170, stride=0b010, skip=0b100,
                                                         proj=0b100),
    "identity shortcut": dict(dims=(3, 32, 32, 32, 32, 32, 10), side=(16, 32), batch=24, skip=0b10100),
    "stride and projection": dict(dims=(3, 24, 48, 48, 48, 10), side=(32, 32), batch=16, stride=0b0010, skip=0b0100, proj=0b0100),
    "stored input gradient": dict(dims=(3, 136, 64, 32, 10), side=(16, 16), batch=90, stride=0b010),
    "pre-activation": dict(dims=(3, 32, 64, 64, 64, 64, 10), side=(16, 32), batch=33, stride=0b00010, skip=0b10100, proj=0b00100,
                           preact=1),
}


class Decided:
    """numpy for one pass of the oracle's model over parameters x, which moves every channel's shift away from its values as
    the pass comes to them; `margin` and `gap`: the smallest distance from zero, and between a pooled window's two largest values."""

    def __init__(self, model, x):
        self.model, self.x, self.layer, self.margin, self.gap = model, x, 0, np.inf, np.inf

    def __getattr__(self, name):
        return getattr(np, name)

    def maximum(self, z, zero):
        lo, hi = self.model.bn_offsets.get(self.layer, self.model.offsets[self.layer])[1:]
        self.layer += 1
        move = np.zeros(hi - lo)
        for c in range(hi - lo):
            near = np.sort(z[..., c], axis=None)
            near = np.concatenate(([-0.05], near[np.abs(near) < 0.05], [0.05]))
            at = np.argmax(np.diff(near))
            move[c] = np.float32(self.x[lo + c] - (near[at] + near[at + 1]) / 2) - self.x[lo + c]
        self.x[lo:hi] += move
        self.margin = min(self.margin, np.abs(z + move).min())
        return np.maximum(z + move, zero)

    def argmax(self, windows, axis):
        top = np.sort(windows, axis=axis)
        self.gap = min(self.gap, (top[..., -1] - top[..., -2])[top[..., -1] > 0].min())
        return np.argmax(windows, axis=axis)


def decided(w, monkeypatch):
    """(oracle with such parameters, batch, labels)"""
    for seed in range(77, 117):
        o = oracle_from(w, workloads.init_params(w))
        X, lab = workloads.batch(w.scaled(data_seed=seed), 0)
        ok = True
        for i in range(w.K):
            seen = Decided(o.model, o.x[i])
            with monkeypatch.context() as m:
                m.setattr(oracle.lsam_oracle, "np", seen)
                o.model.loss_and_grad(o.x[i], X[i], lab[i])
            assert seen.margin > 2e-4
            ok = ok and seen.gap > 4e-6
        if ok:
            return o, X, lab
    raise AssertionError("no data without ties")


@pytest.mark.parametrize("name", sorted(NETS))
def test_rectified_values_against_the_oracle(name, monkeypatch):
    w = net(**NETS[name]).scaled(rho=0.0)
    o, X, lab = decided(w, monkeypatch)
    cfg, keep = lsam.config_from_workload(w)
    g = lsam.Lsam(cfg, workloads.init_params(w), device=DEV, keep=keep)
    for i in range(w.K):
        g.lsam_set_buffer(lsam.BUF_PARAMS, i, o.x[i].astype(np.float32))
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), torch.zeros(w.K, device=DEV))
    o.step(X, lab)
    worst, own = 0.0, 0.0
    for i in range(w.K):
        got, ref = g.lsam_get_buffer(lsam.BUF_GRAD, i), np.asarray(o.last_g2[i])
        for at, ((lo, hi), bound) in enumerate(zip(groups(w), group_bounds(w, ref, []))):
            e = np.linalg.norm(got[lo:hi] - (ref[lo:hi] if bound else 0.0))
            worst, own = max(worst, e / np.linalg.norm(ref)), max(own, e / bound if bound else 0.0)
            assert e <= bound, "group %d: error %.2e, bound %.2e" % (at, e, bound)
    print("%s: worst group %.2e of the whole, %.2f of its bound" % (name, worst, own))
    assert worst <= 3e-6
    g.close()


@pytest.mark.parametrize("name", sorted(NETS))
def test_rectified_values_with_rounded_operands(name):
    w = net(bf16=1, **NETS[name])
    init = workloads.init_params(w)
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    X, lab = workloads.batch(w, 0)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), torch.zeros(w.K, device=DEV))
    o.step(X, lab)
    for i in range(w.K):
        got, want = g.lsam_get_buffer(lsam.BUF_VELOCITY, i), o.v[i]
        assert rel_l2(got, want) < 6e-2, (i, rel_l2(got, want))
    g.close()


def test_statistics_of_values_far_from_zero():
    """Sums 600 spreads from zero: taken as they are, their squares' last bits, 600^2 2^-24, are 2 % of the variance."""
    w = net(dims=(3, 32, 64, 32, 10), side=(16, 32), batch=24)
    init = workloads.init_params(w)
    at = 0
    for l, (fan_in, fo) in enumerate(w.layer_shapes[:w.n_conv]):
        init[at + fan_in * fo:at + fan_in * fo + fo] = 300.0
        at += fan_in * fo + 3 * fo
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    X, lab = workloads.batch(w, 0)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), torch.zeros(w.K, device=DEV))
    o.step(X, lab)
    for i in range(w.K):
        # (a sum's own last bit, 300 2^-24, moves 1e-4 of the rectified values' decisions)
        assert rel_l2(g.lsam_get_buffer(lsam.BUF_VELOCITY, i), o.v[i]) < 1e-2
    g.close()
