"""Normalised convolutions whose outputs are kept as planes and sign bits, with and without the floats beside them, and whose
column sums are taken where the products are written: chains, ragged last tiles, shortcuts that read the floats, projections,
products cut over workgroups, whose sums kernels of their own take; pools joined with the normalisation in front of them or
behind a bare ReLU, and the global average with and without a shortcut that hands its gradient on.

Unlike the nets of test_gpu_plane_products.py half of all values are rectified, pixel by pixel, so a bit of another pixel
or channel shows: half of the gradient's terms would be wrong.  A value within rounding of zero (1e-6 of its
spread in fp32, one in 1e6) may be decided differently from the oracle.  Of the smallest image's V = 1.5e5 values (135000
behind the pre-activation blocks) half carry gradient, one of them (2 / V)^(1/2) = 3.7e-3 of its norm on average; four times
that for the largest is 1.5e-2, the bound (measured: 2e-7 to 5e-7, with one such decision 8e-5, 4.5e-4 and 4.8e-3).  With operands
rounded to bfloat16 decisions within 2^-8 differ, of which the gradient's norm shows sqrt(2^-8) = 6e-2."""
import pytest

torch = pytest.importorskip("torch")
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402
from test_gpu_plane_products import DEV, net  # noqa: E402
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
    "identity shortcut": dict(dims=(3, 32, 32, 32, 32, 32, 10), side=(16, 32), batch=24, skip=0b10100),
    "stride and projection": dict(dims=(3, 24, 48, 48, 48, 10), side=(32, 32), batch=16, stride=0b0010, skip=0b0100, proj=0b0100),
    "stored input gradient": dict(dims=(3, 136, 64, 32, 10), side=(16, 16), batch=90, stride=0b010),
    "pre-activation": dict(dims=(3, 32, 64, 64, 64, 64, 10), side=(16, 32), batch=33, stride=0b00010, skip=0b10100, proj=0b00100,
                           preact=1),
}


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_rectified_values_against_the_oracle(name, bf16):
    w = net(bf16=bf16, **NETS[name])
    init = workloads.init_params(w)
    cfg, keep = lsam.config_from_workload(w)
    g, o = lsam.Lsam(cfg, init, device=DEV, keep=keep), oracle_from(w, init)
    X, lab = workloads.batch(w, 0)
    g.lsam_step(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), torch.zeros(w.K, device=DEV))
    o.step(X, lab)
    for i in range(w.K):
        got, want = g.lsam_get_buffer(lsam.BUF_VELOCITY, i), o.v[i]
        assert rel_l2(got, want) < (6e-2 if bf16 else 1.5e-2), (i, rel_l2(got, want))
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
