"""GPU parity of the approximate EMD (scheduled log-domain Sinkhorn, Kaolin
Sec. 2.5) against the float64 oracle: one iteration from the same potentials
(tight), a full scheduled run (errors add at most linearly: each update is
non-expansive in the potentials' sup norm), the cost, and the fixed-plan
backward."""
import os

import numpy as np
import pytest
import torch

import synth
import gpu_checks as gc
from oracle import emd_oracle

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    import paper_1911_05063_amd as cd
    assert os.path.exists(cd.LIB_PATH), "libcd_hip.so missing: build before running GPU tests"
    yield


import paper_1911_05063_amd as cd  # noqa: E402


def _cmax(X, Y):
    lo = np.minimum(X.min(1), Y.min(1))
    hi = np.maximum(X.max(1), Y.max(1))
    return np.sqrt(((hi - lo).astype(np.float64) ** 2).sum(-1)).max()


def _step_tol(eps, nt, cmax, pmax):
    """Bound on one float32 half-update: distance and hardware square root
    (2^-21 C), the exponent's rounding (2^-24 |z| eps ~ 2^-24 (C + |p|)), the
    float32 running sum over nt terms and the hardware exp2/log2 (2^-21)."""
    return 2.0 ** -20 * cmax + 2.0 ** -22 * pmax + eps * ((nt + 32) * U32 + 2.0 ** -20)


@pytest.mark.parametrize("B,N,M,eps", [(2, 700, 1300, 0.05), (3, 1100, 513, 0.01), (1, 3000, 3000, 0.2),
                                       (2, 1, 257, 0.05), (1, 4500, 90, 0.02), (1000, 5, 7, 0.05)])
def test_one_iteration_matches_oracle(B, N, M, eps):
    print(f"[case] emd step B={B} N={N} M={M} eps={eps}", flush=True)
    X, Y = synth.generate("sphere", B, N, M, 7 + N % 5)
    # Realistic input potentials: a few oracle iterations.
    _, _, G0 = emd_oracle.sinkhorn(X, Y, 0.5, eps, 4)
    G0 = G0.astype(np.float32)
    Xg, Yg = gc.to_gpu(X), gc.to_gpu(Y)
    cost, f, g = cd.emd_forward(Xg, Yg, eps, eps, 1, g_init=gc.to_gpu(G0))
    f, g = gc.to_np(f), gc.to_np(g)
    cmax = _cmax(X, Y)
    F_or, _ = emd_oracle.sinkhorn_step(X, Y, G0, eps)
    tol_f = _step_tol(eps, M, cmax, np.abs(G0).max())
    assert np.max(np.abs(f - F_or)) <= tol_f, (np.max(np.abs(f - F_or)), tol_f)
    # The g-update, from the GPU's own f (the swapped problem's first half-update).
    G_or, _ = emd_oracle.sinkhorn_step(Y, X, f, eps)
    tol_g = _step_tol(eps, N, cmax, np.abs(f).max())
    assert np.max(np.abs(g - G_or)) <= tol_g, (np.max(np.abs(g - G_or)), tol_g)


def test_many_large_groups_match_oracle():
    # 2048 and 640 groups of 256 queries, 16 waves each: 80 targets a wave with a
    # tail for X, 256 for Y (whose last group has 76 queries).  Items are
    # independent: the oracle checks three of the 128.
    B, N, M, iters, e0, e1 = 128, 4096, 1100, 3, 0.3, 0.1
    print(f"[case] emd large groups B={B} N={N} M={M}", flush=True)
    X, Y = synth.generate("sphere", B, N, M, 13)
    cost, f, g = cd.emd_forward(gc.to_gpu(X), gc.to_gpu(Y), e0, e1, iters)
    f, g = gc.to_np(f), gc.to_np(g)
    items = [0, 63, 127]
    _, F_or, G_or = emd_oracle.sinkhorn(X[items], Y[items], e0, e1, iters)
    cmax = _cmax(X[items], Y[items])
    pmax = max(np.abs(F_or).max(), np.abs(G_or).max())
    delta = sum(_step_tol(e, max(N, M), cmax, pmax) for e in emd_oracle.schedule(e0, e1, iters)) * 2
    assert np.max(np.abs(f[items] - F_or)) <= delta, np.max(np.abs(f[items] - F_or))
    assert np.max(np.abs(g[items] - G_or)) <= delta, np.max(np.abs(g[items] - G_or))


def test_full_schedule_cost_and_backward():
    B, N, M, iters, e0, e1 = 2, 1500, 1200, 40, 0.5, 0.02
    X, Y = synth.generate("sphere", B, N, M, 11)
    Xg, Yg = gc.to_gpu(X), gc.to_gpu(Y)
    cost, f, g = cd.emd_forward(Xg, Yg, e0, e1, iters)
    cost, f, g = gc.to_np(cost), gc.to_np(f), gc.to_np(g)
    c_or, F_or, G_or = emd_oracle.sinkhorn(X, Y, e0, e1, iters)
    cmax = _cmax(X, Y)
    pmax = max(np.abs(F_or).max(), np.abs(G_or).max())
    # Each update is non-expansive in the sup norm of the potentials, so the
    # per-step errors add at most linearly over the 2 * iters updates.
    delta = sum(_step_tol(e, max(N, M), cmax, pmax) for e in emd_oracle.schedule(e0, e1, iters)) * 2
    assert np.max(np.abs(f - F_or)) <= delta and np.max(np.abs(g - G_or)) <= delta
    # Cost: the plan's relative error is at most 2 delta / eps_end (both
    # potentials), plus the float32 plan-pass products and sums.
    tol_c = c_or * (2 * delta / e1 + (max(N, M) + 64) * U32)
    assert np.all(np.abs(cost - c_or) <= tol_c), (cost, c_or, tol_c)
    # Cost from the GPU's own potentials, in float64: tighter.
    own = np.array([(emd_oracle.plan(f[b], g[b], emd_oracle.cost_matrix(X[b], Y[b]), e1)
                     * emd_oracle.cost_matrix(X[b], Y[b])).sum() for b in range(B)])
    assert np.all(np.abs(cost - own) <= own * (cmax / e1 * 2.0 ** -20 + (M + 64) * U32)), (cost, own)
    # Backward with the plan of the GPU's potentials held fixed.
    go = np.array([1.0, 0.5], np.float32)
    gX, gY = cd.emd_backward(Xg, Yg, gc.to_gpu(f), gc.to_gpu(g), e1, gc.to_gpu(go))
    rX, rY = emd_oracle.backward(X, Y, f.astype(np.float64), g.astype(np.float64), e1, go)
    # Each term's weight carries a relative error of about (2^-21 C + 2^-23 |f + g|) / eps
    # in the exponent plus 2^-20 from rsqrt / exp2; terms are bounded by the row mass.
    rel = (2.0 ** -21 * cmax + 2.0 ** -23 * 2 * pmax) / e1 + 2.0 ** -19
    tolX = go[:, None, None] * (rel / N + (M + 16) * U32 / N)
    tolY = go[:, None, None] * (rel / M + (N + 16) * U32 / M)
    assert np.all(np.abs(gc.to_np(gX) - rX) <= tolX), np.max(np.abs(gc.to_np(gX) - rX) - tolX)
    assert np.all(np.abs(gc.to_np(gY) - rY) <= tolY), np.max(np.abs(gc.to_np(gY) - rY) - tolY)


def test_autograd_and_degenerate_inputs():
    X, Y = synth.generate("uniform", 2, 300, 200, 13)
    Xg = gc.to_gpu(X).requires_grad_(True)
    Yg = gc.to_gpu(Y).requires_grad_(True)
    cost = cd.earth_movers_distance(Xg, Yg, 0.5, 0.05, 20)
    cost.sum().backward()
    assert torch.isfinite(Xg.grad).all() and torch.isfinite(Yg.grad).all()
    # Translation invariance of the gradients' sum: sum gX + sum gY = 0.
    tot = Xg.grad.double().sum(1) + Yg.grad.double().sum(1)
    assert torch.all(tot.abs() < 1e-5), tot
    # Identical clouds (zero distances on the diagonal) and a single point.
    Z = gc.to_gpu(X[:, :50])
    c, f, g = cd.emd_forward(Z, Z.clone(), 0.5, 0.01, 60)
    gX, gY = cd.emd_backward(Z, Z, f, g, 0.01, torch.ones(2, device="cuda:0"))
    assert torch.isfinite(c).all() and torch.isfinite(gX).all() and torch.isfinite(gY).all()
    assert torch.all(c < 0.01 * 2 * np.log(50) + 1e-3), c
    c1, _, _ = cd.emd_forward(gc.to_gpu(X[:, :1]), gc.to_gpu(Y[:, :1]), 0.5, 0.05, 3)
    want = np.sqrt(((X[:, 0].astype(np.float64) - Y[:, 0]) ** 2).sum(-1))
    assert np.allclose(gc.to_np(c1), want, rtol=1e-5), (c1, want)


def test_reproducible():
    X, Y = synth.generate("gmm", 2, 2000, 900, 17)
    Xg, Yg = gc.to_gpu(X), gc.to_gpu(Y)
    a = cd.emd_forward(Xg, Yg, 0.5, 0.02, 10)
    b = cd.emd_forward(Xg, Yg, 0.5, 0.02, 10)
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("B,N,M", [(256, 33, 65), (260, 257, 15), (130, 200, 255), (140, 129, 17),
                                   (1, 16, 1), (2, 63, 2049), (3, 65, 16)])
def test_every_split_of_a_half_update_matches_oracle(B, N, M):
    # 4, 2 and 1 queries per lane (as many as leave 256 workgroups and as the
    # item has), 16 waves or 4, targets that leave waves empty, with one target,
    # and with tails.
    eps = 0.05
    print(f"[case] emd split B={B} N={N} M={M}", flush=True)
    X, Y = synth.generate("gmm", B, N, M, 3 * N + M)
    _, f, g = cd.emd_forward(gc.to_gpu(X), gc.to_gpu(Y), eps, eps, 2)
    items = sorted({0, B // 2, B - 1})
    _, F_or, G_or = emd_oracle.sinkhorn(X[items], Y[items], eps, eps, 2)
    pmax = max(np.abs(F_or).max(), np.abs(G_or).max())
    # Four half-updates, each non-expansive in the potentials' sup norm.
    tol = 4 * _step_tol(eps, max(N, M), _cmax(X[items], Y[items]), pmax)
    assert np.max(np.abs(gc.to_np(f)[items] - F_or)) <= tol
    assert np.max(np.abs(gc.to_np(g)[items] - G_or)) <= tol


def test_millions_of_tiny_items_match_oracle():
    # More workgroups than 2^22: a launch holds fewer than 2^32 threads.
    B, N, M, eps = 4_300_000, 2, 3, 0.1
    print(f"[case] emd tiny items B={B} N={N} M={M}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(5)
    X, Y = (torch.rand((B, n, 3), generator=g, device="cuda:0") for n in (N, M))
    cost, f, gp = cd.emd_forward(X, Y, eps, eps, 2)
    items = [0, 1, (1 << 20) - 1, 1 << 20, (1 << 22) - 1, 1 << 22, B - 1]
    Xi, Yi = gc.to_np(X[items]), gc.to_np(Y[items])
    _, F_or, G_or = emd_oracle.sinkhorn(Xi, Yi, eps, eps, 2)
    pmax = max(np.abs(F_or).max(), np.abs(G_or).max())
    tol = 4 * _step_tol(eps, max(N, M), _cmax(Xi, Yi), pmax)
    assert np.max(np.abs(gc.to_np(f[items]) - F_or)) <= tol
    assert np.max(np.abs(gc.to_np(gp[items]) - G_or)) <= tol
    assert bool(torch.isfinite(cost).all())


@pytest.mark.parametrize("N,M", [(64, 100000), (17, 20001), (600, 40000)])
def test_few_queries_against_many_targets(N, M):
    # A few targets at the queries, all others at a distance whose terms are
    # 2^-24.6 of theirs: added one by one to a running sum they would vanish.
    # No partial sum may have more than 512 terms: a batch of 16, at most 256
    # batches, and the merges.
    eps, terms = 1.0 / (24.6 * np.log(2.0)), 512
    print(f"[case] emd few queries N={N} M={M}", flush=True)
    rng = np.random.default_rng(M)
    X = 1e-4 * rng.uniform(-1, 1, (1, N, 3))
    Y = rng.normal(size=(1, M, 3))
    Y /= np.linalg.norm(Y, axis=2, keepdims=True)
    Y[0, ::5000] *= 1e-4
    X, Y = X.astype(np.float32), Y.astype(np.float32)
    g0 = np.zeros((1, M), np.float32)
    _, f, g = cd.emd_forward(gc.to_gpu(X), gc.to_gpu(Y), eps, eps, 1, g_init=gc.to_gpu(g0))
    f, g = gc.to_np(f), gc.to_np(g)
    F_or, _ = emd_oracle.sinkhorn_step(X, Y, g0, eps)
    tol = _step_tol(eps, terms, 1.0, 0.0)
    assert np.max(np.abs(f - F_or)) <= tol, (np.max(np.abs(f - F_or)), tol)
    G_or, _ = emd_oracle.sinkhorn_step(Y, X, f, eps)
    tol_g = _step_tol(eps, min(N, terms), 1.0, np.abs(f).max())
    assert np.max(np.abs(g - G_or)) <= tol_g, (np.max(np.abs(g - G_or)), tol_g)


@pytest.mark.parametrize("B,N,M", [(1, 64, 1537), (1, 65, 20001), (2, 513, 4097), (1, 4097, 300),
                                   (300, 70, 64), (256, 129, 65), (1, 7, 65537)])
def test_split_targets_match_oracle(B, N, M):
    # Few queries: the targets are split over workgroups, with remainders in
    # the last block and in its waves; up to 64 targets: four waves.
    eps = 0.05
    print(f"[case] emd target split B={B} N={N} M={M}", flush=True)
    X, Y = synth.generate("gmm", B, N, M, N + 3 * M)
    _, f, g = cd.emd_forward(gc.to_gpu(X), gc.to_gpu(Y), eps, eps, 2)
    items = sorted({0, B // 2, B - 1})
    _, F_or, G_or = emd_oracle.sinkhorn(X[items], Y[items], eps, eps, 2)
    pmax = max(np.abs(F_or).max(), np.abs(G_or).max())
    # Four half-updates, each non-expansive; sums of at most 512 terms.
    tol = 4 * _step_tol(eps, 512, _cmax(X[items], Y[items]), pmax)
    assert np.max(np.abs(gc.to_np(f)[items] - F_or)) <= tol
    assert np.max(np.abs(gc.to_np(g)[items] - G_or)) <= tol


def test_tens_of_millions_of_single_points():
    # More than 2^24 workgroups of 256 threads in the plan passes.  With one
    # point each the plan is 1, the cost the distance, the gradients its unit vectors.
    B = 17_000_000
    print(f"[case] emd single points B={B}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    X, Y = (torch.rand((B, 1, 3), generator=gen, device="cuda:0") + k for k in (0.0, 1.0))
    cost, f, g = cd.emd_forward(X, Y, 0.1, 0.1, 1)
    d = (X - Y)[:, 0].double()
    want = d.norm(dim=1)
    # f + g = C to a few roundings of it, which the plan's exponent takes over eps.
    assert float((cost / want - 1.0).abs().max()) <= 2.0 ** -17
    go = torch.ones(B, device="cuda:0")
    gX, gY = cd.emd_backward(X, Y, f, g, 0.1, go)
    unit = d / want[:, None]
    for got, ref in ((gX, unit), (gY, -unit)):
        assert float((got[:, 0] - ref).abs().max()) <= 2.0 ** -17
