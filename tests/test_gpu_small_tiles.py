"""Products of small bf16 dense models on 64x64 tiles: widths and batches around the tile's edges, rings
of four and eight stages with contractions shorter, equal to and longer than the ring, and states
that stay in the caches (ordinary stores) or do not, where ragged 128x128 and 256x128 tiles serve."""
import pytest

torch = pytest.importorskip("torch")
import workloads  # noqa: E402
from test_gpu_parity import _fused_equals_separate, run_mlp  # noqa: E402

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


def test_ragged_tiles_past_the_caches():
    # 285 MB a state vector: streaming stores, 128x128 step, 256x128 products and ascent, the last on 64x64 tiles
    _fused_equals_separate(_model((1000, 2500, 2300, 300), 300, 8), 2)
