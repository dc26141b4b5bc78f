"""The update on gradients that are both at hand (norm, perturbed point and descent in two or three
launches) against the same in 64 bits, at the sizes where its kernels change: words of four and what
is left of one, workgroups' edges, the numbers of partial sums, rows past the caches, gradient rows
at any 4-byte alignment, and a perturbed point that lies over one of the inputs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2509_03110_amd import lsam  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -24
MU, LR, RHO, GAMMA, LAM = (float(np.float32(v)) for v in (0.9, 0.05, 0.05, 1e-12, 0.7))     # as the library holds them


def _state(K, d, g_shift, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    pad = (d + 63) // 64 * 64

    def rows(n, std):
        t = torch.zeros(n, pad, device=DEV)
        t[:, :d] = torch.randn(n, d, generator=gen, device=DEV) * std
        return t
    y = rows(1, 1.0)[0]
    x = rows(K, 0.1)
    x[:, :d] += y[:d]
    # rows of d floats starting g_shift floats past a 16-byte boundary
    flat = [torch.randn(K * d + 4, generator=gen, device=DEV) for _ in range(2)]
    g1, g2 = (f[g_shift:g_shift + K * d].view(K, d) for f in flat)
    return x, rows(K, 0.05), rows(K, 2.0), y, g1, g2


def _want(x, v, S, y, g1, g2, lam, d, nesterov):
    x, v, S, y, g1, g2 = (t[..., :d].double() for t in (x, v, S, y, g1, g2))
    n = g1.norm(dim=1)
    xt = x + (RHO / (n + GAMMA))[:, None] * g1
    G = g2 + lam * (x - y)
    vn = MU * v + G
    xn = x - LR * (G + MU * vn if nesterov else vn)
    # a bound on the rounding of each result: a few roundings of the largest terms that enter it
    big = g2.abs() + lam * (x.abs() + y.abs()) + v.abs()
    return dict(norms=(n, 4 * EPS * n), xt=(xt, 4 * EPS * (x.abs() + (xt - x).abs())), v=(vn, 6 * EPS * big),
                x=(xn, 4 * EPS * x.abs() + 8 * EPS * LR * 3 * big), S=(S + xn, 4 * EPS * (S.abs() + x.abs()) + 8 * EPS * LR * 3 * big))


def _check(got, want, d):
    for name, (value, bound) in want.items():
        err = (got[name][..., :d].double() - value).abs()
        worst = float((err / (bound + 1e-30)).max())
        assert worst <= 1.0, (name, worst)


@pytest.mark.parametrize("K,d,g_shift,nesterov", [
    (1, 1, 1, 1), (3, 3, 0, 1), (2, 5, 3, 0), (5, 1023, 0, 1), (4, 1024, 1, 1), (2, 1025, 2, 0), (7, 2050, 3, 1),
    (3, 4096 * 127 + 1, 1, 1), (2, 4096 * 128, 0, 1), (1, 4096 * 128 + 7, 2, 1),     # 128 partial sums of 4096 and more
    (1, 16384 * 128, 0, 1), (2, 16384 * 128 + 3, 1, 1),                              # the most added up by the descent; one more
    (13, 2_000_003, 3, 1),                                                           # past the caches, sums in the descent
    (9, 16384 * 200 + 1023, 1, 1), (8, 16384 * 200 + 2048, 0, 0)])                   # past the caches, sums apart
def test_static_step_against_64_bits(K, d, g_shift, nesterov):
    x, v, S, y, g1, g2 = _state(K, d, g_shift, seed=K + d)
    lam = LAM
    want = _want(x, v, S, y, g1, g2, lam, d, nesterov)
    xt, norms = torch.full_like(x, 7.0), torch.zeros(K, device=DEV)
    lsam.lsam_step_grads_static(x, v, S, y, g1, g2, xt, norms, [lam] * K, rho=RHO, gamma=GAMMA, lr=LR, momentum=MU,
                                nesterov=nesterov, d=d)
    torch.cuda.synchronize()
    _check(dict(x=x, v=v, S=S, xt=xt, norms=norms), want, d)
    assert bool((xt[:, d:] == 7.0).all()) and bool((x[:, d:] == 0).all())            # nothing past d


@pytest.mark.parametrize("K,d", [(2, 777), (3, 4096 * 128 + 5)])
@pytest.mark.parametrize("over", ["g1", "S"])
def test_perturbed_point_over_an_input(K, d, over):
    """x~ over an array of the step is written before the descent reads that array, as when the
    perturbation was a launch of its own."""
    x, v, S, y, _, _ = _state(K, d, 0, seed=d)
    pad = x.shape[1]
    gen = torch.Generator(device=DEV).manual_seed(5)
    g1, g2 = (torch.randn(K, pad, generator=gen, device=DEV) for _ in range(2))
    want = _want(x, v, S, y, g1, g2, LAM, d, 1)
    if over == "S":                                # the sum starts from what lies there: x~
        value, bound = want["S"]
        want["S"] = (value - S[:, :d].double() + want["xt"][0], bound + want["xt"][1] + 4 * EPS * x[:, :d].abs().double())
        del want["xt"]
    xt = g1 if over == "g1" else S
    norms = torch.zeros(K, device=DEV)
    lsam.lsam_step_grads_static(x, v, S, y, g1, g2, xt, norms, [LAM] * K, rho=RHO, gamma=GAMMA, lr=LR, momentum=MU,
                                nesterov=1, d=d)
    torch.cuda.synchronize()
    _check(dict(x=x, v=v, S=S, xt=xt, norms=norms), want, d)


@pytest.mark.parametrize("K,d,rho", [(3, 5001, 0.05), (2, 4096 * 128 + 2, 0.05), (9, 16384 * 200 + 6, 0.05), (3, 5001, 0.0)])
def test_context_step_and_restarted_sums(K, d, rho):
    """Through a context, across center updates: a served replica's sum starts afresh in the one pass too."""
    cfg, keep = lsam.make_config(d_raw=d, K=K, gamma=GAMMA, momentum=MU, beta=0.9, lambda_abs=LAM, tau=[2] * K, lr=LR, rho=rho)
    gen = torch.Generator(device=DEV).manual_seed(11)
    init = torch.randn(d, generator=gen, device=DEV)
    eng = lsam.Lsam(cfg, init.cpu().numpy(), device=DEV, keep=keep)
    x = init.double().repeat(K, 1)
    y, v, S = init.double(), torch.zeros_like(x), torch.zeros_like(x)
    prev = None
    for t in range(5):
        g1, g2 = (torch.randn(K, d, generator=gen, device=DEV) for _ in range(2))
        eng.lsam_step_grads(g1, g2)
        G = g2.double() + LAM * (x - y)
        v = MU * v + G
        xt = x + (rho / (g1.double().norm(dim=1) + GAMMA))[:, None] * g1.double()
        x = x - LR * (G + MU * v)
        S = S + x
        if eng.lsam_sync():
            gp = S.sum(0) / (2 * K) - y
            y = y + float(cfg.lr_center) * (gp if prev is None else gp + float(np.float32(0.9)) * (gp - prev))
            prev, S = gp, torch.zeros_like(S)
        for k in range(K):
            for buf, val in ((lsam.BUF_PARAMS, x), (lsam.BUF_VELOCITY, v), (lsam.BUF_ITER_SUM, S)) + (
                    ((lsam.BUF_PERTURBED, xt),) if rho else ()):
                a = torch.from_numpy(np.asarray(eng.lsam_get_buffer(buf, k))).double()
                # five steps of the roundings above, terms of a few units
                assert float((a - val[k].cpu()).abs().max()) < 5 * 8 * 8 * EPS, (t, k, buf)
    eng.close()
