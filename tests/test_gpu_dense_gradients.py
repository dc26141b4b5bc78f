"""fp32 dense models whose gradients come from one launch: widths and batches around the tiles, with the
narrow head and without, the product below the head left to it in one, few and many pieces, and
numbers of partial sums of the norm on both sides of what the perturbation adds up itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402
from test_gpu_parity import CNN_SMALL, make_pair, run_mlp, to_dev  # noqa: E402
from util import rel_l2  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,B,K", [
    ((30, 10), 5, 1),                            # the head alone, on the data
    ((784, 128, 10), 32, 2),                     # the product below the head in 6 pieces
    ((2000, 64, 16), 8, 2), ((3000, 100, 3), 24, 3),     # in 15 and 16 (17-column remainders)
    ((1500, 300, 10), 64, 2),                    # too wide for that: reduced by a launch of its own
    ((65, 63, 129, 17), 33, 2), ((64, 64, 64, 64), 64, 1), ((200, 127, 17, 40), 130, 3),    # no narrow head
    ((520, 700, 640, 12), 100, 4),               # more than 128 partial sums
    ((520, 900, 900, 12), 100, 4),               # 128x128 tiles, none of them full
    ((300, 520, 24, 10), 512, 2),                # the head's largest batch
    ((1024, 1024, 10), 520, 4)])                 # 128x128 tiles beside a narrow product of its own
def test_against_the_oracle(dims, B, K):
    w = workloads.WORKLOADS["cfg1"].scaled(name="dg", lr=0.01, K=K, dims=dims, batch=B, tau=(2,) * K, n_classes=dims[-1], steps=3)
    # (the bounds for fp32; pre-activations at least 2e-5 from zero, some ten roundings)
    run_mlp(w, 3, 1e-4, 1e-3, margin=True, margin_ratio=32.0, min_margin=2e-5)


@pytest.mark.parametrize("dims,B,K", [((3, 8, 650, 700, 10), 40, 8),      # 128x128 tiles with remainders
                                      ((3, 8, 65, 63, 17), 33, 2)])       # 64x64, no narrow head
def test_rounded_operands_behind_a_convolution(dims, B, K):
    w = CNN_SMALL.scaled(name="tail", K=K, dims=dims, n_conv=1, img_h=16, img_w=16, pool_mask=1, batch=B, tau=(2,) * K,
                         n_classes=dims[-1], gemm_dtype=1)
    run_mlp(w, 3, 2e-2, 2e-2, anchor_after=1)        # the bounds of the other models with bf16 products


@pytest.mark.parametrize("dims,B,K", [((784, 128, 10), 512, 1), ((64, 64, 64, 10), 1000, 2), ((64, 64, 64, 10), 4096, 2),
                                      ((100, 300, 10), 4096, 1)])
def test_long_batches_keep_their_digits(dims, B, K):
    """Gradients against 64 bits where thousands of rows are summed.  Carried through n additions (two rows each) a sum
    of changing signs ends about 0.41 2^-24 sqrt(n / 2) of its size off: 1.4e-7 for pieces of 128 rows, 1e-7 for adding up
    32 of them, and as much again comes from the forward pass; 7.8e-7 for 4096 rows at once."""
    w = workloads.WORKLOADS["cfg1"].scaled(name="long", lr=0.01, K=K, dims=dims, batch=B, tau=(2,) * K, n_classes=dims[-1])
    g, o = make_pair(w, workloads.init_params_margin(w, ratio=32.0))
    X, lab = workloads.batch(w, 0)
    Xd, ld = to_dev(X, lab, w)
    g.lsam_step(Xd, ld, None)
    o.step(X, lab)
    assert o.model.last_margin > 2e-5
    for k in range(K):
        got = g.lsam_get_buffer(lsam.BUF_GRAD, k)
        print("%s B=%d: relative error %.2e" % (dims, B, rel_l2(got, o.last_g2[k])))
        assert np.all(np.isfinite(got)) and rel_l2(got, o.last_g2[k]) < 3.5e-7
    g.close()
