"""The pruned nearest-neighbour search (cd_forward with the larger workspace)
against the all-pairs search of the same call, bitwise: distances and indices
of both directions.  Sizes around the sort's chunks, ranges and nodes, clouds
that strain it (equal points, outliers, lines, ties, one cloud far from the
other), the static-workspace entry point, and a captured call."""
import ctypes

import numpy as np
import pytest
import torch

import gpu_checks as gc
import oracle
import paper_1911_05063_amd as cd
import synth

pytestmark = pytest.mark.gpu


def _call(X, Y, ws_bytes):
    B, N, M = X.shape[0], X.shape[1], Y.shape[1]
    lib = cd.library()
    # Workspace and outputs start as garbage that would show: small distances.
    ws = torch.zeros(ws_bytes, dtype=torch.uint8, device=X.device)
    out = [torch.full((B, n), -1, dtype=t, device=X.device)
           for n in (N, M) for t in (torch.float32, torch.int32)]
    st = lib.cd_forward(B, N, M, *[ctypes.c_void_p(t.data_ptr()) for t in [X, Y] + out],
                        ctypes.c_void_p(ws.data_ptr()), ws_bytes,
                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0, lib.cd_last_error()
    return out


def _compare(X, Y, what):
    B, N, M = X.shape[0], X.shape[1], Y.shape[1]
    need, best = cd.workspace_bytes(B, N, M), cd.workspace_bytes_best(B, N, M)
    assert best > need, f"{what}: not a shape of the pruned search"
    print(f"[tree] {what} B={B} N={N} M={M}", flush=True)
    ref, got = _call(X, Y, need), _call(X, Y, best)
    for name, a, b in zip(("dist_xy", "idx_xy", "dist_yx", "idx_yx"), got, ref):
        assert torch.equal(a, b), f"{what} {name}: {int((a != b).sum())} differ"
    return got


# One range (<= 4096 points) against many, chunk and node remainders, B that
# does and does not divide the 8 XCDs, more than 64 nodes.
@pytest.mark.parametrize("kind,B,N,M", [
    ("uniform", 1, 27000, 27001), ("sphere", 3, 16384, 16385), ("mesh", 16, 8193, 8191),
    ("gmm", 2, 2049, 190000), ("grid_dup", 5, 40961, 4097), ("mesh", 64, 4096, 4095),
    ("uniform", 1, 262145, 3071), ("gmm", 7, 10240, 12289)])
def test_sizes_match_all_pairs(kind, B, N, M):
    X, Y = synth.generate(kind, B, N, M, 7 * N + M)
    _compare(gc.to_gpu(X), gc.to_gpu(Y), kind)


def _strain(name):
    rng = np.random.default_rng(11)
    N, M = 30011, 28000
    X, Y = rng.uniform(-1, 1, (1, N, 3)), rng.uniform(-1, 1, (1, M, 3))
    if name == "all_equal":           # every target ties: the lowest index wins
        X[:] = 0.25
    elif name == "both_equal":
        X[:], Y[:] = 0.25, -0.5
    elif name == "few_places":        # thousands of copies of 40 points, zero distances
        p = rng.uniform(-1, 1, (40, 3))
        X[0], Y[0] = p[rng.integers(0, 40, N)], p[rng.integers(0, 40, M)]
    elif name == "outliers":          # a thousandth of the points far away
        X[0, ::1000] *= 1e4
        Y[0, 500::1000] *= -1e6
    elif name == "line":              # two coordinates constant
        X[..., 1:], Y[..., 1:] = 0.0, 1e-3
    elif name == "far_apart":         # all targets about as far
        Y += 50.0
    elif name == "shell":             # queries inside a sphere of targets
        X = 0.3 * X
        Y /= np.linalg.norm(Y, axis=2, keepdims=True)
    elif name == "lattice":           # exact ties everywhere
        X, Y = np.round(X * 16) / 16, np.round(Y * 16) / 16 + 1 / 32
    elif name == "tiny":              # distances in float32's subnormal range
        X, Y = X * 1e-21, Y * 1e-21
    elif name == "huge":              # squared distances near float32's largest
        X, Y = X * 3e18, Y * 3e18
    elif name in ("at_3e38", "at_max"):   # one coordinate huge and the same: targets around queries
        Y /= np.linalg.norm(Y[..., 1:], axis=2, keepdims=True)
        X[..., 0] = Y[..., 0] = 3.0e38 if name == "at_3e38" else -np.finfo(np.float32).max
        X[..., 1:] *= 0.3
    return X.astype(np.float32), Y.astype(np.float32)


@pytest.mark.parametrize("name", ["all_equal", "both_equal", "few_places", "outliers", "line",
                                  "far_apart", "shell", "lattice", "tiny", "huge", "at_3e38",
                                  "at_max"])
def test_strained_clouds_match_all_pairs(name):
    X, Y = _strain(name)
    _compare(gc.to_gpu(X), gc.to_gpu(Y), name)


def _without(X, Y, fx, fy):
    """All pairs of the points fx, fy of one item, as the call on all points
    should give it: +inf and -1 for the others."""
    ref = _call(X[:, fx].contiguous(), Y[:, fy].contiguous(),
                cd.workspace_bytes(1, int(fx.sum()), int(fy.sum())))
    out = []
    for mine, other, d, i in ((fx, fy, ref[0], ref[1]), (fy, fx, ref[2], ref[3])):
        dist = torch.full((1, len(mine)), float("inf"), device=X.device)
        idx = torch.full((1, len(mine)), -1, dtype=torch.int32, device=X.device)
        dist[:, mine] = d
        idx[:, mine] = torch.nonzero(other)[:, 0].int()[i.long()]
        out += [dist, idx]
    return out


# Whole leaves and ranges of points with a NaN, single ones between others
# (one range and several), of either sign, in each coordinate.
@pytest.mark.parametrize("N,M", [(30011, 28000), (4001, 180001)])
@pytest.mark.parametrize("name", ["scattered", "runs", "most", "all_x"])
def test_nan_points_have_no_neighbour_and_are_none(name, N, M):
    g = torch.Generator(device="cuda:0").manual_seed(N)
    X, Y = (2 * torch.rand((1, n, 3), generator=g, device="cuda:0") - 1 for n in (N, M))
    for P in (X, Y):
        n = P.shape[1]
        k = {"scattered": torch.arange(0, n, 37), "runs": torch.arange(n // 3, n // 2),
             "most": torch.arange(5, n), "all_x": torch.arange(0, n if P is X else 0)}[name]
        k = k.to(P.device)
        P[0, k, k % 3] = torch.where(k % 2 == 0, float("nan"), -float("nan"))
    need, best = cd.workspace_bytes(1, N, M), cd.workspace_bytes_best(1, N, M)
    assert best > need
    print(f"[tree] nan {name} N={N} M={M}", flush=True)
    got = _call(X, Y, best)
    fx, fy = (torch.isfinite(P[0]).all(dim=1) for P in (X, Y))
    if name == "all_x":
        ref = [t for n in (N, M) for t in (torch.full((1, n), float("inf"), device=X.device),
                                           torch.full((1, n), -1, dtype=torch.int32, device=X.device))]
    else:
        ref = _without(X, Y, fx, fy)
    for what, a, b in zip(("dist_xy", "idx_xy", "dist_yx", "idx_yx"), got, ref):
        assert torch.equal(a, b), f"{name} {what}: {int((a != b).sum())} differ"


# Points with an infinite coordinate (their own results are not defined) and with
# far ones whose squared distances overflow: all others as without them.
@pytest.mark.parametrize("N,M", [(30011, 28000), (4001, 180001)])
@pytest.mark.parametrize("name", ["ends", "scattered", "overflow"])
def test_infinite_points_do_not_disturb_others(name, N, M):
    g = torch.Generator(device="cuda:0").manual_seed(N + 1)
    X, Y = (2 * torch.rand((1, n, 3), generator=g, device="cuda:0") - 1 for n in (N, M))
    for P in (X, Y):
        n = P.shape[1]
        k = torch.tensor([0, n - 1]) if name == "ends" else torch.arange(5, n, 41)
        k = k.to(P.device)
        far = 3e25 if name == "overflow" else float("inf")
        P[0, k, k % 3] = torch.where(k % 2 == 0, far, -far)
    need, best = cd.workspace_bytes(1, N, M), cd.workspace_bytes_best(1, N, M)
    assert best > need
    print(f"[tree] infinite {name} N={N} M={M}", flush=True)
    got = _call(X, Y, best)
    fx, fy = ((P[0].abs() < 1e25).all(dim=1) for P in (X, Y))
    ref = _without(X, Y, fx, fy)
    for what, a, b, mine in zip(("dist_xy", "idx_xy", "dist_yx", "idx_yx"), got, ref, (fx, fx, fy, fy)):
        assert torch.equal(a[:, mine], b[:, mine]), f"{name} {what}"
    for i, n in ((got[1], M), (got[3], N)):
        assert bool(((i >= -1) & (i < n)).all())


def test_entry_points_take_the_same_path_and_bits():
    # Through the binding (default workspace), the static workspace and a graph.
    X_np, Y_np = synth.generate("mesh", 2, 20000, 18001, 5)
    X, Y = gc.to_gpu(X_np), gc.to_gpu(Y_np)
    ref = _compare(X, Y, "entry points")
    rows = np.stack([np.arange(64) % 2, np.arange(64) * 281], axis=1)
    rd, ri = gc.sample_nn(X_np, Y_np, rows)
    assert np.array_equal(gc.to_np(ref[0])[rows[:, 0], rows[:, 1]], rd)
    assert np.array_equal(gc.to_np(ref[1])[rows[:, 0], rows[:, 1]], ri)
    ws = torch.empty(cd.workspace_bytes_best(2, 20000, 18001), dtype=torch.uint8, device="cuda:0")
    small = torch.empty(cd.workspace_bytes(2, 20000, 18001), dtype=torch.uint8, device="cuda:0")
    for got in (cd.nn_distance(X, Y), cd.nn_distance(X, Y, ws), cd.nn_distance(X, Y, small),
                cd.nn_distance_noalloc(X, Y)):
        assert all(torch.equal(a, b) for a, b in zip(got, ref))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        cd.nn_distance(X, Y, ws)
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = cd.nn_distance(X, Y, ws)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref))
        cd.nn_distance(Y, X)          # eager work in between
        torch.cuda.synchronize()


def test_many_clouds_on_two_streams():
    # Each call has its own workspace: interleaved calls give each one's bits.
    clouds = [tuple(gc.to_gpu(a) for a in synth.generate(k, B, N, M, 3))
              for k, B, N, M in (("gmm", 4, 16000, 15000), ("sphere", 48, 4500, 4000))]
    ref = [cd.nn_distance(X, Y) for X, Y in clouds]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    out = []
    for _ in range(3):
        for k, (X, Y) in enumerate(clouds):
            with torch.cuda.stream(streams[k]):
                out.append((k, cd.nn_distance(X, Y)))
    torch.cuda.synchronize()
    for k, got in out:
        assert all(torch.equal(a, b) for a, b in zip(got, ref[k]))


@pytest.mark.parametrize("B,N,M", [(1, 30000, 25001), (32, 8192, 8192)])
def test_distances_match_the_oracle(B, N, M):
    X, Y = synth.generate("mesh", B, N, M, 9)
    got = _compare(gc.to_gpu(X), gc.to_gpu(Y), "oracle")
    ref = oracle.nn(X[:2], Y[:2], fused=True)
    gc.assert_nn_bitwise(tuple(gc.to_np(t)[:2] for t in got), ref, "tree")


def _time(X, Y, ws_bytes):
    B, N, M = X.shape[0], X.shape[1], Y.shape[1]
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=X.device)
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            cd.nn_distance(X, Y, ws)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / 5)
    return float(np.median(times[1:]))


# Every query about as far from every target: the search takes all of them.
@pytest.mark.parametrize("B,N,M", [(1, 30001, 25003), (7, 10240, 12289), (64, 4000, 4001)])
@pytest.mark.parametrize("name", ["cluster", "sphere"])
def test_queries_as_far_from_all_targets(name, B, N, M):
    X, Y = (gc.to_gpu(a) for a in synth.generate("gmm", B, N, M, 5))
    X = 0.8 * X / X.norm(dim=2, keepdim=True)
    Y = 0.01 * Y if name == "cluster" else Y / Y.norm(dim=2, keepdim=True) * 0.1
    if name == "sphere":
        X[:, 7] = float("nan")          # has no neighbour, and is none
        X, Y = Y.contiguous(), X.contiguous()
    X, Y = X.contiguous(), Y.contiguous()
    got = _compare(X, Y, name) if name == "cluster" else None
    if got is None:
        keep = torch.arange(Y.shape[1], device=Y.device) != 7
        ref = _call(X, Y[:, keep].contiguous(), cd.workspace_bytes(B, M, N - 1))
        assert cd.workspace_bytes_best(B, M, N) > cd.workspace_bytes(B, M, N)
        got = _call(X, Y, cd.workspace_bytes_best(B, M, N))
        at = torch.nonzero(keep)[:, 0].int()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], at[ref[1].long()])
        assert torch.equal(got[2][:, keep], ref[2]) and torch.equal(got[3][:, keep], ref[3])
        assert bool(torch.isinf(got[2][:, 7]).all()) and bool((got[3][:, 7] == -1).all())
        return
    pruned, pairs = (_time(X, Y, f(B, N, M)) for f in (cd.workspace_bytes_best, cd.workspace_bytes))
    # 2.3 to 3.2 times all pairs; each query searching by itself 5 to 9 times.
    assert pruned <= 4.0 * pairs, (name, pruned, pairs)


# Clouds that a regular grid over their box does not resolve, in one range of
# the sort and in several: a point far from all others (the first, the last,
# one between), padding at a place of its own, two scenes far apart, outliers.
@pytest.mark.parametrize("B,N,M", [(16, 16384, 16384), (64, 4000, 4000)])
@pytest.mark.parametrize("name", ["first", "last", "between", "padding", "two_scenes", "outliers"])
def test_far_points_do_not_undo_the_pruning(name, B, N, M):
    X, Y = (gc.to_gpu(a) for a in synth.generate("mesh", B, N, M, 3))
    for P, sign in ((X, 1.0), (Y, -1.0)):
        n = P.shape[1]
        if name == "padding":
            P[:, 7 * n // 10:] = sign * 1e6
        elif name == "two_scenes":
            P[:, ::2] += 2e4
        elif name == "outliers":
            P[:, 500::1000] *= sign * 1e4
        else:
            P[:, {"first": 0, "last": n - 1, "between": n // 3}[name]] += 1e5
    _compare(X, Y, name)
    pruned, pairs = (_time(X, Y, f(B, N, M)) for f in (cd.workspace_bytes_best, cd.workspace_bytes))
    # 0.3 to 0.9 of all pairs' time; without a grid of quantiles 3 to 12 times.
    assert pruned <= 1.5 * pairs, (name, pruned, pairs)
