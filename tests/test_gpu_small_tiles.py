"""Products of small bf16 dense models on 64x64 tiles: widths and batches around the tile's edges, rings
of four and eight stages with contractions shorter, equal to and longer than the ring, and states
that stay in the caches (ordinary stores) or do not, where ragged 128x128 and 256x128 tiles serve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402
from test_gpu_parity import DEV, _fused_equals_separate, run_mlp, to_dev  # noqa: E402
from util import rel_max  # noqa: E402

pytestmark = pytest.mark.gpu


def _model(dims, B, K):
    return workloads.WORKLOADS["cfg3"].scaled(name="small", K=K, dims=dims, batch=B, tau=(2,) * K, n_classes=dims[-1],
                                              steps=3, batch_pool=0)


@pytest.mark.parametrize("dims,B,K", [
    ((64, 64, 64, 64), 64, 2), ((65, 63, 129, 5), 65, 1), ((128, 127, 257, 33), 33, 3),
    ((250, 300, 130, 70), 96, 2),                # 8 and 10 k-steps: a whole round of the ring and one begun
    ((30, 500, 31, 100), 7, 4), ((385, 66, 700, 17), 129, 2)])
def test_small_models(dims, B, K):
    w = _model(dims, B, K)
    _fused_equals_separate(w, 3)
    run_mlp(w, 3, 2e-2, 2e-2, margin=True)       # the file's bound for bf16 operands


@pytest.mark.parametrize("B", [300, 600])
def test_large_tiles_with_remainders(B):
    """Forward products, input gradients and weight gradients of 128x128 (300 rows) and 256x128 tiles (600), none of
    whose extents and contractions is a multiple of the tile or of a k-step, against the oracle."""
    w = _model((1000, 1400, 1500, 1100, 100), B, 8)
    run_mlp(w, 2, 2e-2, 2e-2, margin=True)
    run_mlp(w, 2, 2e-2, 2e-2, margin=False, tol_flip=1e-1, anchor_after=1)


@pytest.mark.parametrize("dims,B,K", [((1000, 2500, 2300, 300), 300, 8), ((2100, 2300, 300), 4200, 1)])
def test_ragged_tiles_past_the_caches(dims, B, K):
    """285 MB a state vector: streaming stores, 128x128 step, 256x128 products and ascent, the last layer on
    64x64 tiles; 22 MB with a batch that is work enough for a launch a layer all the same.  Fused against separate kernels.  Their norms may differ in the last bit, and among
    7e7 perturbed weights some then round to the other bf16 neighbour, 2^-8 away; a unit sums at least
    1000 of them, so what it computes, and the gradients behind it, move by 2^-8 / sqrt(1000) = 1.2e-4 at most."""
    w = _model(dims, B, K)
    init = workloads.init_params(w)
    cfg, keep = lsam.config_from_workload(w)
    a, b = (lsam.Lsam(cfg, init, device=DEV, keep=keep) for _ in range(2))
    assert a.lsam_set_fused_step(True) == 1 and b.lsam_set_fused_step(False) == 0
    for t in range(2):
        X, lab = workloads.batch(w, t)
        Xd, ld = to_dev(X, lab, w)
        a.lsam_step(Xd, ld, None)
        b.lsam_step(Xd, ld, None)
        assert np.allclose(a.lsam_get_norms(), b.lsam_get_norms(), rtol=2e-6, atol=0)
        assert a.lsam_sync() == b.lsam_sync()
        for i in range(w.K):
            assert rel_max(a.lsam_get_params(i), b.lsam_get_params(i)) < 1.2e-4 * w.lr * (1 + w.momentum) * 2
            for which in (lsam.BUF_VELOCITY, lsam.BUF_ITER_SUM):
                assert rel_max(a.lsam_get_buffer(which, i), b.lsam_get_buffer(which, i)) < 1.2e-4, (t, i, which)
        assert rel_max(a.lsam_get_params(-1), b.lsam_get_params(-1)) < 1.2e-4
    a.close()
    b.close()
