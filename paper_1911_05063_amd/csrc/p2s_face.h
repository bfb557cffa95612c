// Face records of the point-to-surface searches and the distance they give.
#pragma once

#include <cmath>

#include "cd_internal.h"
#include "mesh_common.h"

namespace cdk {

constexpr int kRec = 32;          // floats per face record (31 used)
// Corner of a face with a vertex index out of range: every distance to such a
// record overflows to +inf (no inf - inf anywhere), so it is never chosen.
constexpr float kFar = 3.0e38f;

// The record r of the face (A, B, C), evaluated in double: the corner a, the
// dual basis g0, g1 of the edges e0 = b - a, e1 = c - a in the face's plane, the
// unit normal, an inside threshold (0, or +inf for a face without interior),
// and each edge with its direction over its squared length.
// Returns (|g0| + |g1|) (|e0| + |e1|), 0 without interior: how far the triangle's
// corners move, relative to a shift of its edges.
__device__ __forceinline__ double face_record(const double A[3], const double Bv[3],
                                              const double C[3], float r[kRec])
{
    double e0[3], e1[3], e2[3], n[3];
    for (int i = 0; i < 3; ++i) {
        e0[i] = Bv[i] - A[i];
        e1[i] = C[i] - A[i];
        e2[i] = C[i] - Bv[i];
    }
    n[0] = e0[1] * e1[2] - e0[2] * e1[1];
    n[1] = e0[2] * e1[0] - e0[0] * e1[2];
    n[2] = e0[0] * e1[1] - e0[1] * e1[0];
    const double nn = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
    // Dual basis: g0 = (e1 x n) / |n|^2, g1 = (n x e0) / |n|^2, so that
    // e0.g0 = e1.g1 = 1 and e1.g0 = e0.g1 = n.g0 = n.g1 = 0.
    double g0[3] = {0, 0, 0}, g1[3] = {0, 0, 0}, nh[3] = {0, 0, 0};
    const bool flat = !(nn > 0.0) || !std::isfinite(nn);
    // One reciprocal per denominator (double divisions are long instruction
    // sequences); the record is rounded to float32 afterwards.
    if (!flat) {
        const double rn = 1.0 / nn;
        g0[0] = (e1[1] * n[2] - e1[2] * n[1]) * rn;
        g0[1] = (e1[2] * n[0] - e1[0] * n[2]) * rn;
        g0[2] = (e1[0] * n[1] - e1[1] * n[0]) * rn;
        g1[0] = (n[1] * e0[2] - n[2] * e0[1]) * rn;
        g1[1] = (n[2] * e0[0] - n[0] * e0[2]) * rn;
        g1[2] = (n[0] * e0[1] - n[1] * e0[0]) * rn;
        const double inv = 1.0 / sqrt(nn);
        for (int i = 0; i < 3; ++i) nh[i] = n[i] * inv;
    }
    const double l0 = e0[0] * e0[0] + e0[1] * e0[1] + e0[2] * e0[2];
    const double l1 = e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2];
    const double l2 = e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2];
    const double r0 = l0 > 0.0 ? 1.0 / l0 : 0.0;
    const double r1 = l1 > 0.0 ? 1.0 / l1 : 0.0;
    const double r2 = l2 > 0.0 ? 1.0 / l2 : 0.0;
    for (int i = 0; i < 3; ++i) {
        r[0 + i] = static_cast<float>(A[i]);
        r[3 + i] = static_cast<float>(g0[i]);
        r[6 + i] = static_cast<float>(g1[i]);
        r[9 + i] = static_cast<float>(nh[i]);
        r[13 + i] = static_cast<float>(e0[i]);
        r[16 + i] = static_cast<float>(e0[i] * r0);
        r[19 + i] = static_cast<float>(e1[i]);
        r[22 + i] = static_cast<float>(e1[i] * r1);
        r[25 + i] = static_cast<float>(e2[i]);
        r[28 + i] = static_cast<float>(e2[i] * r2);
    }
    r[12] = flat ? __builtin_inff() : 0.0f;
    r[31] = 0.0f;
    return flat ? 0.0
                : (sqrt(g0[0] * g0[0] + g0[1] * g0[1] + g0[2] * g0[2]) +
                   sqrt(g1[0] * g1[0] + g1[1] * g1[1] + g1[2] * g1[2])) * (sqrt(l0) + sqrt(l1));
}

__device__ __forceinline__ void far_record(float r[kRec])
{
    for (int i = 0; i < kRec; ++i) r[i] = 0.0f;
    r[0] = r[1] = r[2] = kFar;
    r[12] = __builtin_inff();
}

__device__ __forceinline__ float fmaf_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

__device__ __forceinline__ float dot3(float x, float y, float z, float a, float b, float c)
{
    return fmaf_(z, c, fmaf_(y, b, x * a));
}

// Squared distance from v (relative to the segment's origin) to the segment
// {sigma e : sigma in [0, 1]}, en = e / |e|^2.
__device__ __forceinline__ float seg2(float vx, float vy, float vz, float ex, float ey, float ez,
                                      float nx, float ny, float nz)
{
    const float sg = __builtin_amdgcn_fmed3f(dot3(vx, vy, vz, nx, ny, nz), 0.0f, 1.0f);
    const float wx = fmaf_(-sg, ex, vx), wy = fmaf_(-sg, ey, vy), wz = fmaf_(-sg, ez, vz);
    return dot3(wx, wy, wz, wx, wy, wz);
}

// Squared distance from (px, py, pz) to the face of record (A0 .. A7).
__device__ __forceinline__ float face_dist(float px, float py, float pz, const float4 (&A)[8])
{
    const float ax = A[0].x, ay = A[0].y, az = A[0].z;
    const float g0x = A[0].w, g0y = A[1].x, g0z = A[1].y;
    const float g1x = A[1].z, g1y = A[1].w, g1z = A[2].x;
    const float nx = A[2].y, ny = A[2].z, nz = A[2].w, cin = A[3].x;
    const float e0x = A[3].y, e0y = A[3].z, e0z = A[3].w, n0x = A[4].x, n0y = A[4].y, n0z = A[4].z;
    const float e1x = A[4].w, e1y = A[5].x, e1z = A[5].y, n1x = A[5].z, n1y = A[5].w, n1z = A[6].x;
    const float e2x = A[6].y, e2y = A[6].z, e2z = A[6].w, n2x = A[7].x, n2y = A[7].y, n2z = A[7].z;
    const float vx = px - ax, vy = py - ay, vz = pz - az;
    const float s = dot3(vx, vy, vz, g0x, g0y, g0z);
    const float t = dot3(vx, vy, vz, g1x, g1y, g1z);
    const float h = dot3(vx, vy, vz, nx, ny, nz);
    const float u = (1.0f - s) - t;
    const bool inside = __builtin_fminf(__builtin_fminf(s, t), u) >= cin;
    const float dab = seg2(vx, vy, vz, e0x, e0y, e0z, n0x, n0y, n0z);
    const float dca = seg2(vx, vy, vz, e1x, e1y, e1z, n1x, n1y, n1z);
    const float dbc = seg2(vx - e0x, vy - e0y, vz - e0z, e2x, e2y, e2z, n2x, n2y, n2z);
    const float edge = __builtin_fminf(__builtin_fminf(dab, dca), dbc);
    return inside ? h * h : edge;
}

}  // namespace cdk
