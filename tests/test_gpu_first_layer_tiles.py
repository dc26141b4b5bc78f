"""First convolution layers whose workgroups take several tiles of 32 pixels a wavefront, the last ones ragged, on image rows
that do and do not hold whole runs of 8 pixels, and whose output gradient is formed where the weight gradient reads it or,
where a shortcut hands it on, by the normalisation; held to the oracle's groups as the other convolutions are."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import test_gpu_plane_products as planes  # noqa: E402
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402

pytestmark = pytest.mark.gpu

NETS = {
    "four tiles, rows of 36": dict(dims=(3, 8, 10), side=(30, 36), batch=245),
    "two tiles, rows of 40": dict(dims=(2, 40, 10), side=(27, 40), batch=121),
    "one tile, rows of 6": dict(dims=(1, 64, 10), side=(11, 6), batch=31),
    "six pixels": dict(dims=(3, 40, 8, 10), side=(2, 3), batch=1, bn=0),
    "four images of one pixel": dict(dims=(2, 16, 10), side=(1, 1), batch=4, bn=0),
    "twelve pixels, normalised": dict(dims=(1, 72, 8, 10), side=(2, 2), batch=3),
    "a shortcut's sum": dict(dims=(3, 32, 32, 32, 10), side=(16, 16), batch=33, skip=0b100, preact=1),
    "a shortcut's input": dict(dims=(3, 32, 32, 32, 10), side=(16, 24), batch=23, skip=0b100),
}


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_against_the_oracle(name, bf16, monkeypatch):
    monkeypatch.setitem(planes.NETS, name, NETS[name])
    planes.test_plane_products_match_oracle(name, bf16)


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("dims", [(3, 40, 10), (3, 40, 8, 10)])
@pytest.mark.parametrize("bn", [0, 1])
@pytest.mark.parametrize("side,batch", [((1, 1), 4), ((2, 3), 1), ((2, 3), 2), ((11, 6), 31), ((5, 8), 3)])
def test_the_last_pixels_read_nothing_of_the_next_replica(side, batch, bn, dims, bf16):
    """Sixteen pixels are loaded at a time, and a replica's last ones need not be sixteen: behind them lie the next replica's
    gradients, here infinite or NaN.  The first replica's gradients are the same bit for bit beside any neighbour."""
    w = planes.net(dims=dims, side=side, batch=batch, bn=bn, bf16=bf16)
    init = workloads.init_params(w)
    X, lab = workloads.batch(w, 0)
    bad = X.copy()
    bad[1] = np.inf
    got = []
    for pixels in (X, bad):
        cfg, keep = lsam.config_from_workload(w)
        g = lsam.Lsam(cfg, init, device=planes.DEV, keep=keep)
        g.lsam_step(torch.from_numpy(pixels).to(planes.DEV), torch.from_numpy(lab).to(planes.DEV), None)
        got.append([g.lsam_get_buffer(lsam.BUF_GRAD, 0), g.lsam_get_norms()])
        if pixels is bad and not bn:
            assert not np.isfinite(g.lsam_get_buffer(lsam.BUF_GRAD, 1)).all()
        g.close()
    assert np.isfinite(got[0][0]).all() and np.any(got[0][0])
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1][0] == got[1][1][0]
