"""The pruned point-to-surface search (large meshes) against all pairs, bitwise.
All pairs: the same call on runs of fewer faces than the pruned search takes,
merged by distance, then face index.  Shapes at its limits and with remainders
in every tile, and meshes that strain its bounds: needles, flat and invalid
faces, equal faces, far and equal points, extreme scales."""
import numpy as np
import pytest
import torch

import gpu_checks as gc
import paper_1911_05063_amd as cd
import synth

pytestmark = pytest.mark.gpu

FEWER = 2047    # faces below which every shape takes all pairs


def _all_pairs(P, V, F):
    dist = torch.full(P.shape[:2], float("inf"), device=P.device)
    face = torch.full(P.shape[:2], -1, dtype=torch.int32, device=P.device)
    for f0 in range(0, F.shape[1], FEWER):
        d, f = cd.p2s_forward(P, V, F[:, f0:f0 + FEWER].contiguous())
        new = d < dist
        dist = torch.where(new, d, dist)
        face = torch.where(new, f + f0, face)
    return dist, face


def _compare(P, V, F, what):
    print(f"[p2s tree] {what} B={P.shape[0]} S={P.shape[1]} nf={F.shape[1]}", flush=True)
    assert P.shape[0] * P.shape[1] * F.shape[1] >= 1.5e8 and F.shape[1] >= 2048, what
    P, V, F = (gc.to_gpu(a) for a in (P, V, F))
    shape = P.shape[0], P.shape[1], V.shape[1], F.shape[1]
    lib = cd.library()
    assert lib.cd_p2s_workspace_bytes_best(*shape) > lib.cd_p2s_workspace_bytes(*shape)
    ref, got = _all_pairs(P, V, F), cd.p2s_forward(P, V, F)
    assert torch.equal(got[0], ref[0]), f"{what} dist: {int((got[0] != ref[0]).sum())} differ"
    assert torch.equal(got[1], ref[1]), f"{what} face: {int((got[1] != ref[1]).sum())} differ"
    return got


@pytest.mark.parametrize("B,S,n", [(16, 4601, 33), (1, 73243, 34), (3, 16385, 65), (40, 1024, 63),
                                   (2, 12289, 100)])
def test_sizes_match_all_pairs(B, S, n):
    # n x n height fields: 2 (n - 1)^2 faces (2048, 2178, 7688, 8192, 19602).
    V, F = synth.grid_mesh(B, n, n)
    rng = np.random.default_rng(S)
    P = np.concatenate([rng.uniform(-1.1, 1.1, (B, S, 2)), rng.normal(0, 0.2, (B, S, 1))], axis=2)
    _compare(P.astype(np.float32), V, F, "grid")


def test_icospheres_match_all_pairs():
    _compare(*synth.p2s_workload(B=8, S=5001, level=4, seed=3), "icosphere")


def _strain(name, nf=3001, S=60007):
    rng = np.random.default_rng(5)
    c = rng.uniform(-1, 1, (1, nf, 1, 3))
    tri = c + 0.03 * rng.normal(size=(1, nf, 3, 3))
    P = rng.uniform(-1.2, 1.2, (1, S, 3))
    if name == "needles":            # two corners next to each other, the third far
        tri[:, ::2, 1] = tri[:, ::2, 0] + 1e-5 * rng.normal(size=tri[:, ::2, 0].shape)
        tri[:, ::2, 2] = tri[:, ::2, 0] + 2.0 * rng.normal(size=tri[:, ::2, 0].shape)
    elif name == "slivers":          # nearly collinear at every aspect ratio
        w = 10.0 ** rng.uniform(-9, 0, (1, nf, 1))
        tri[:, :, 2] = 0.5 * (tri[:, :, 0] + tri[:, :, 1]) + w * 0.1 * rng.normal(size=(1, nf, 3))
    elif name == "flat":             # points and segments among the faces
        tri[:, ::3, 1] = tri[:, ::3, 0]
        tri[:, ::5, 2] = tri[:, ::5, 1]
    elif name == "equal_faces":      # exact ties: the lowest index
        tri[:] = tri[:, :1]
    elif name == "equal_points":
        P[:] = 0.1
    elif name == "far_points":
        P += 300.0
    elif name == "outliers":
        tri[:, ::500] += 1e4
        P[:, ::1000] *= 1e5
    elif name == "tiny":
        tri, P = tri * 1e-17, P * 1e-17
    elif name == "huge":
        tri, P = tri * 1e15, P * 1e15
    elif name == "nan_points":       # single ones, and whole leaves of them
        P[:, ::41, 1] = np.nan
        P[:, 20000:30000, 0] = -np.nan
    elif name == "nan_vertices":     # a corner, so that an edge may be left, or a face
        tri[:, ::3, 1, 2] = np.nan
        tri[:, 1::7] = np.nan
    elif name == "overflow":         # no finite distance: no face
        P[:, ::50] *= 1e25
    V = tri.reshape(1, -1, 3).astype(np.float32)
    F = np.arange(3 * nf, dtype=np.int32).reshape(1, nf, 3)
    if name == "invalid":
        F[:, ::3, 1] = 3 * nf + 7
        F[:, 1::7, 2] = -1
    elif name == "all_invalid":
        F[:] = -1
    return P.astype(np.float32), V, F


@pytest.mark.parametrize("name", ["plain", "needles", "slivers", "flat", "equal_faces",
                                  "equal_points", "far_points", "outliers", "tiny", "huge",
                                  "invalid", "all_invalid", "nan_points", "nan_vertices",
                                  "overflow"])
def test_strained_meshes_match_all_pairs(name):
    got = _compare(*_strain(name), name)
    if name == "all_invalid":
        assert bool(torch.isinf(got[0]).all()) and bool((got[1] == -1).all())


# Few points: four waves share the faces of a leaf of points.
@pytest.mark.parametrize("name", ["plain", "needles", "flat", "equal_faces", "equal_points",
                                  "outliers", "invalid", "all_invalid", "nan_points",
                                  "nan_vertices", "overflow"])
def test_few_points_match_all_pairs(name):
    _compare(*_strain(name, 13001, 13007), name)


@pytest.mark.parametrize("B,S,n", [(1, 27999, 54), (1, 1024, 272), (20, 1100, 84)])
def test_few_points_sizes_match_all_pairs(B, S, n):
    V, F = synth.grid_mesh(B, n, n)
    rng = np.random.default_rng(S)
    P = np.concatenate([rng.uniform(-1.1, 1.1, (B, S, 2)), rng.normal(0, 0.2, (B, S, 1))], axis=2)
    _compare(P.astype(np.float32), V, F, "grid")
