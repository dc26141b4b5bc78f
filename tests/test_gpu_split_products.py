"""fp32 dense products on the bf16 matrix units (exact split into three pieces): ragged tiles of 64 and 128 rows, remainders of
columns and of the contraction, products cut over workgroups and not, input gradients, all weight gradients in one launch;
which products take them; and operands past bfloat16's rounding range."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import launches  # noqa: E402
import workloads  # noqa: E402
from paper_2509_03110_amd import lsam  # noqa: E402
from test_gpu_parity import run_mlp  # noqa: E402

NETS = [((1030, 1000, 1000, 10), 255, 8),       # 128 rows, one missing; 30 of a step of 32 left over, forward and input gradient
        ((3001, 1025, 40), 128, 4),             # a column of tiles for one column; cut into pieces
        ((1000, 1150, 1000, 17), 60, 24)]       # 64 rows, four missing


def products(dims, B, K):
    names = launches.names(dict(K=K, dims=dims, batch=B))
    return [n for n in names if n.startswith("split_gemm_kernel<")]


@pytest.mark.parametrize("dims,B,K,rows", [(NETS[0][0], 255, 8, 128), (NETS[2][0], 60, 24, 64),
                                           ((512, 512, 512, 10), 512, 8, 0),        # 1.07e9 multiply-adds
                                           ((1000, 1500, 777, 37), 300, 3, 0),      # a third of the tiles' work for padding
                                           # contractions below 900 on 192 tiles, which would be cut; on 256 tiles; 1000 on 128
                                           ((768, 768, 768, 10), 512, 8, 0), ((512, 3000, 10), 1024, 1, 0),
                                           ((512, 512, 512, 10), 400, 16, 128), ((1000, 1000, 1000, 10), 255, 8, 128),
                                           ((784, 128, 10), 32, 2, 0)])
def test_which_products_are_split(dims, B, K, rows):
    got = products(dims, B, K)
    assert all(n.startswith("split_gemm_kernel<%d," % rows) for n in got) and bool(got) == bool(rows), got
    if rows:
        assert {n.endswith("true,true>") for n in got} == {True, False}, got


@pytest.mark.parametrize("dims,B,K", [((2000, 1000, 10), 250, 12), ((960, 640, 10), 512, 8), ((520, 6000, 100), 700, 1),
                                      ((3001, 1025, 40), 128, 4), ((1000, 1150, 1000, 17), 60, 24)])
def test_pieces_fit_the_chip_at_once(dims, B, K):
    """A product that is cut has at most the 512 workgroups that are resident together."""
    grids = [(l["grid"][0], l["name"]) for l in launches.record(dict(K=K, dims=dims, batch=B))[0]["launches"]
             if l["name"].startswith("split_gemm_kernel<")]
    assert grids and all(n <= 512 for n, _ in grids), grids


@pytest.mark.gpu
@pytest.mark.parametrize("dims,B,K", NETS)
def test_against_the_oracle(dims, B, K):
    assert products(dims, B, K)
    w = workloads.WORKLOADS["cfg1"].scaled(name="split", lr=0.01, K=K, dims=dims, batch=B, tau=(2,) * K, n_classes=dims[-1], steps=1)
    # (the bounds for fp32; pre-activations at least 2e-5 from zero, some ten roundings)
    run_mlp(w, 1, 1e-4, 1e-3, margin=True, margin_ratio=32.0, min_margin=2e-5)


@pytest.mark.gpu
def test_operands_past_the_rounding_range():
    """3.4e38 rounds to infinity in bfloat16 and is cut instead: times 2^-100 it is an ordinary number; times 2 it overflows,
    an infinite operand stays infinite, and no neighbour sees either."""
    w = workloads.WORKLOADS["cfg1"].scaled(K=8, dims=(1030, 1000, 10), batch=255, tau=(2,) * 8, n_classes=10, rho=0.0, lr=0.01)
    init = np.full(w.d, 2.0**-10, np.float32)
    init[:1030 * 1000].reshape(1000, 1030)[7, :] = 2.0
    init[:1030 * 1000].reshape(1000, 1030)[9, :] = 2.0**-100
    cfg, keep = lsam.config_from_workload(w)
    g = lsam.Lsam(cfg, init, device="cuda:0", keep=keep)
    X, lab = workloads.batch(w, 0)
    X[:] = 0.0
    X[:, 3, 5] = 3.4e38
    X[:, 4, 1029] = np.inf
    X[:, 5, :] = 1.0
    g.lsam_step(torch.from_numpy(X).cuda(), torch.from_numpy(lab).cuda(), None)
    for k in (0, 7):
        a = g.lsam_get_activation(1, k)
        assert a[3, 7] == np.inf and np.all(a[4] == np.inf)
        assert np.allclose(a[3, 9], np.float32(3.4e38) * 2.0**-100 + 2.0**-10, rtol=1e-6)
        assert np.allclose(np.delete(a[3], [7, 9]), np.float32(3.4e38) * 2.0**-10, rtol=1e-6)
        assert np.allclose(a[5, 7], 2060.0 + 2.0**-10, rtol=1e-6) and np.allclose(a[0], 2.0**-10, rtol=1e-6)
    g.close()
