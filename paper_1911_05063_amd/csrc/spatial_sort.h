// Points sorted along a space-filling curve, in leaves and nodes with bounding
// boxes: what the exact pruned searches (nn_tree.hip) walk instead of every
// pair.
//
// Two launches sort all clouds of a call:
//  * bucket (clouds of more than one range): a workgroup takes a chunk of
//    kSortChunk points and groups them by range, a run of cells of a Hilbert
//    curve.  kSortSamples points spread over the cloud, the same for all its
//    chunks, give the curve's box and the runs, so that ranges hold about
//    equally many points wherever those lie, and no launch is spent on it.
//    (Points outside that box belong to border cells.)
//  * sort: a workgroup gathers one range of one cloud from all chunks (or a
//    small cloud as it is) and counting-sorts it by the leading bits of the
//    points' indices along the same curve, from the range's lowest index on.
// A regular grid does not resolve every cloud: one point a thousand extents
// away, or padding at a place of its own, puts all others into one cell, and
// leaves of points in no order are boxes around the whole cloud (16 x 16384^2
// samples of meshes with one far point each: 6600 us, all pairs 525).  So where a
// cell is crowded, the cloud (bucket) or the range (sort) takes a grid between
// the quantiles of 64 of its points instead (142 us).
// The order of points within one cell is whatever the LDS atomics give: the
// searches take minima of (distance, original index), which no order changes.
//
// Records (x, y, z, index) of range w start at slot
// align(points in lower ranges, kNode) + w kNode, so that every node (kNode
// slots) belongs to one range; slots behind a range's last point up to the
// next multiple of kTile hold the index ~0 (no point), those behind it are not
// written.  A leaf is kLeaf slots, a node kNodeLeaves leaves.  Boxes hold the
// smallest index of their points too; a box without points is empty
// (lo = +inf, hi = -inf).
//
// A point with a NaN coordinate has no distance to anything.  Its slot holds no
// point (so it is in no box, and no target), but kNanMark as y and its index as
// z, and its leaf's box says so: the searches answer it at once (nan_query).
#pragma once

#include <algorithm>

#include "cd_internal.h"
#include "fixed_point.h"

namespace cdk {

constexpr int kLeaf = 16;
constexpr int kNodeLeaves = 64;
constexpr int kNode = kLeaf * kNodeLeaves;
constexpr int kTile = 64;                        // slots are written up to a multiple of this
constexpr uint32_t kNoPoint = 0xffffffffu;       // index of a slot without a point
// Its x: every squared distance to it is +inf, or NaN from an infinite coordinate
// (a large finite one would be near points as far out).
constexpr float kFarAway = __builtin_inff();
constexpr float kNanMark = 1.0f;                 // its y if it stands for a point with a NaN

struct alignas(32) Box {
    float lx, ly, lz;
    uint32_t first;     // smallest index of a point in the box
    float hx, hy, hz;
    uint32_t nans;      // of a leaf: whether it has points with a NaN coordinate
};

// How one cloud of n points is sorted and stored.
struct SortShape {
    int32_t n;
    int32_t ranges;
    int32_t log_c;      // log2(cells per range)
    int32_t chunks;     // of the bucket pass
    int32_t nodes;      // nodes stored (slots / kNode)
};

// The sorted clouds of a batch in a workspace (byte offsets from its start).
struct SortPlan {
    SortShape s;
    int64_t B;
    size_t entries, offs, curve, rec, leaf, node;
};

// A batch of clouds to sort, and where to.
struct SortJob {
    const float *P;         // [B, n, 3]
    float4 *rec;            // [B, nodes kNode] records
    Box *leaf, *node;       // [B, nodes kNodeLeaves], [B, nodes]
    float4 *entries;        // bucket pass: [B, chunks, points of a chunk],
    uint32_t *offs;         // [B, chunks, ranges + 1],
    struct Curve *curve;    // [B]
    SortShape s;
};

// Clouds of at most this many points can be sorted.
constexpr int64_t kSortMaxPoints = int64_t{1} << 21;

// Lays the sorted clouds out from byte `at` on, which it moves past them.
SortPlan plan_sort(int64_t B, int64_t n, size_t &at);
SortJob sort_job(const SortPlan &p, const float *P, char *ws);
// Sorts two batches of B clouds in the same launches and zeroes n words.
hipError_t launch_sort(int64_t B, const SortJob &a, const SortJob &b, uint32_t *zero, uint32_t n,
                       hipStream_t stream);

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return static_cast<uint32_t>(
        __builtin_amdgcn_mov_dpp(static_cast<int>(v), kCtrl, 0xF, 0xF, true));
}

// Minimum over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ uint32_t row_min_u32(uint32_t m)
{
    m = min(m, dpp_u32<0xB1>(m));
    m = min(m, dpp_u32<0x4E>(m));
    m = min(m, dpp_u32<0x141>(m));
    return min(m, dpp_u32<0x140>(m));
}

__device__ __forceinline__ uint32_t row_max_u32(uint32_t m)
{
    m = max(m, dpp_u32<0xB1>(m));
    m = max(m, dpp_u32<0x4E>(m));
    m = max(m, dpp_u32<0x141>(m));
    return max(m, dpp_u32<0x140>(m));
}

// Minimum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t m)
{
    m = row_min_u32(m);
    const auto r16 = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    m = min(r16[0], r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return min(r32[0], r32[1]);
}

// Whether slot q, of a leaf whose box ends with `hi`, stands for a point with a
// NaN coordinate (the slots of a leaf without any may be unwritten).
__device__ __forceinline__ bool nan_query(const float4 &q, const float4 &hi)
{
    return __float_as_uint(hi.w) != 0u && __float_as_uint(q.w) == kNoPoint && q.y == kNanMark;
}

constexpr uint32_t kXcds = 8;       // accelerator complex dies of an MI355X

// Consecutive workgroups on one XCD (they are dealt out round-robin): the
// ranges and tiles of one item share one L2.
__device__ __forceinline__ uint32_t xcd_block()
{
    const uint32_t i = blockIdx.x, per = gridDim.x / kXcds;
    return i < kXcds * per ? (i % kXcds) * per + i / kXcds : i;
}

__device__ __forceinline__ double pack(float d, uint32_t i)
{
    return __hiloint2double(__float_as_int(d), static_cast<int>(i));
}

__device__ __forceinline__ unsigned long long as_bits(double k)
{
    return static_cast<unsigned long long>(__double_as_longlong(k));
}

__device__ __forceinline__ double as_key(unsigned long long k)
{
    return __longlong_as_double(static_cast<long long>(k));
}

// The smaller key.  The sign is dropped: that of a NaN distance (from infinite
// coordinates) may be set, and its key is to be above every other.
__device__ __forceinline__ double min_key(double a, double b)
{
    double r;
    asm("v_min_f64 %0, |%1|, |%2|" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Smallest distance, per axis, from an interval to another (0 if they meet).
__device__ __forceinline__ float gap(float alo, float ahi, float blo, float bhi)
{
    float r;
    const float u = blo - ahi, v = alo - bhi;
    asm("v_max3_f32 %0, %1, %2, 0" : "=v"(r) : "v"(u), "v"(v));
    return r;
}

__device__ __forceinline__ float sum_sq(float x, float y, float z)
{
    return __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
}

__device__ __forceinline__ float bound(const float4 &alo, const float4 &ahi, const float4 &blo,
                                       const float4 &bhi)
{
    return sum_sq(gap(alo.x, ahi.x, blo.x, bhi.x), gap(alo.y, ahi.y, blo.y, bhi.y),
                  gap(alo.z, ahi.z, blo.z, bhi.z));
}

__device__ __forceinline__ float4 middle(const float4 &lo, const float4 &hi)
{
    return make_float4(0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z), 0.0f);
}

// The value lane U of each row of 16 holds, in all its lanes.
template <int U>
__device__ __forceinline__ float row_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + U, 0xF, 0xF, true));
}

template <int U>
__device__ __forceinline__ void leaf_keys(const float4 &q, const float4 &r, double (&k)[kLeaf])
{
    if constexpr (U < kLeaf) {
        const float dx = row_lane<U>(r.x) - q.x;
        const float dy = row_lane<U>(r.y) - q.y;
        const float dz = row_lane<U>(r.z) - q.z;
        k[U] = pack(sum_sq(dx, dy, dz), __float_as_uint(row_lane<U>(r.w)));
        leaf_keys<U + 1>(q, r, k);
    }
}

__device__ __forceinline__ float high(double k) { return __int_as_float(__double2hiint(k)); }

// Minimum with the lanes 16 and 32 apart: over the four rows.
__device__ __forceinline__ double rows_min(double k)
{
    auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(k), __double2loint(k), false, false);
    auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(k), __double2hiint(k), false, false);
    k = min_key(__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1]));
    lo = __builtin_amdgcn_permlane32_swap(__double2loint(k), __double2loint(k), false, false);
    hi = __builtin_amdgcn_permlane32_swap(__double2hiint(k), __double2hiint(k), false, false);
    return min_key(__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1]));
}

template <int kCtrl>
__device__ __forceinline__ double dpp_key(double k)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(k), kCtrl, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(k), kCtrl, 0xF, 0xF, true));
}

__device__ __forceinline__ float row_max(float w)
{
    w = fmaxf(w, dpp_f<0xB1>(w));
    w = fmaxf(w, dpp_f<0x4E>(w));
    w = fmaxf(w, dpp_f<0x141>(w));
    return fmaxf(w, dpp_f<0x140>(w));
}

// A sorted cloud to search: its leaf and node boxes (two float4 each).
struct Targets {
    const float4 *leaf, *node;
    uint32_t nodes;
};

constexpr int kNear = 4;    // nodes looked at for the first bounds (2: 118 -> 133 us on meshes)

// The four leaves nearest to the box [qlo, qhi] (each the nearest of one
// lane's) in the kNear nearest nodes; ~0: every distance overflows.  Order:
// box distance, then that of the centres (boxes that meet are all at 0).
// nlo, nhi: box of node min(lane, nodes - 1).
__device__ __forceinline__ void nearest_leaves(const Targets &j, const float4 &qlo, const float4 &qhi,
                                               const float4 &nlo, const float4 &nhi, uint32_t lane,
                                               uint32_t near_leaf[4])
{
    const float4 mid = middle(qlo, qhi);
    const auto order = [&](const float4 &lo, const float4 &hi) {
        const float4 m = middle(lo, hi);
        return __float_as_uint(__builtin_fmaf(0.01f, sum_sq(mid.x - m.x, mid.y - m.y, mid.z - m.z),
                                              bound(qlo, qhi, lo, hi)));
    };
    uint32_t near = order(nlo, nhi), near_at = min(lane, j.nodes - 1);
    for (uint32_t from = kWave; from < j.nodes; from += kWave) {
        const uint32_t i = min(from + lane, j.nodes - 1);
        const uint32_t k = order(j.node[2 * i], j.node[2 * i + 1]);
        near_at = k < near ? i : near_at;
        near = min(near, k);
    }
    near = (near & ~63u) | lane;
    uint32_t nodes[kNear];
#pragma unroll
    for (int v = 0; v < kNear; ++v) {
        const uint32_t m = __builtin_amdgcn_readfirstlane(wave_min_u32(near));
        nodes[v] = v == 0 || m < 0x7f800000u ? __builtin_amdgcn_readlane(near_at, m & 63u) : nodes[0];
        near = lane == (m & 63u) ? kNoPoint : near;
    }
    uint32_t key = kNoPoint, key_at = 0u;
#pragma unroll
    for (int v = 0; v < kNear; ++v) {
        const uint32_t at = nodes[v] * kNodeLeaves + lane;
        const uint32_t k = order(j.leaf[at * 2], j.leaf[at * 2 + 1]);
        key_at = k < key ? at : key_at;
        key = min(key, k);
    }
    key = (key & ~63u) | lane;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const uint32_t m = __builtin_amdgcn_readfirstlane(wave_min_u32(key));
        near_leaf[v] = m < 0x7f800000u ? __builtin_amdgcn_readlane(key_at, m & 63u)
                                       : v > 0 ? near_leaf[0] : kNoPoint;
        key = lane == (m & 63u) ? kNoPoint : key;
    }
}

// What lanes of a wave wrote to LDS before this, others may read after it.  (A
// wave's LDS operations execute in order; the fence keeps the compiler from
// moving them, or from taking accesses of other types for unrelated.)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Appends v of the lanes that take it to a list of n values in LDS.
__device__ __forceinline__ void append(uint32_t *list, uint32_t &n, bool take, uint32_t v)
{
    const uint64_t taken = __ballot(take);
    if (take)
        list[__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(taken >> 32),
            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(taken), n))] = v;
    n += __popcll(taken);
}

// Queues the leaves, other than the four done, that takes(lo, hi) of their box
// (and of their node's) lets pass.  full() is called when more than `limit` are
// queued and ends the walk by returning false; it may empty the queue and
// tighten what takes() lets pass.  mine: whether the wave takes this lane's leaf
// of each node.
template <class Takes, class Full>
__device__ __forceinline__ void gather(const Targets &j, const float4 &nlo, const float4 &nhi,
                                       uint32_t lane, const uint32_t done[4], uint32_t *queue,
                                       uint32_t &queued, uint32_t limit, bool mine,
                                       const Takes &takes, const Full &full)
{
    for (uint32_t from = 0; from < j.nodes; from += kWave) {
        float4 lo = nlo, hi = nhi;
        if (from > 0u) {
            const uint32_t i = min(from + lane, j.nodes - 1);
            lo = j.node[2 * i];
            hi = j.node[2 * i + 1];
        }
        uint64_t left = __ballot(from + lane < j.nodes && takes(lo, hi));
        if (left == 0ull) continue;
        // The next node's boxes are on their way while one's are looked at (16 x
        // 16384^2 mesh samples 133 -> 126 us, a template of 26645 points against a
        // surface 131 -> 124).
        uint32_t node = __builtin_ctzll(left);
        const auto leaf_of = [&](uint32_t n) { return (from + n) * kNodeLeaves + lane; };
        float4 llo = j.leaf[leaf_of(node) * 2], lhi = j.leaf[leaf_of(node) * 2 + 1];
        while (left != 0ull) {
            left &= left - 1ull;
            const uint32_t at = leaf_of(node), ahead = left != 0ull ? __builtin_ctzll(left) : node;
            const float4 alo = j.leaf[leaf_of(ahead) * 2], ahi = j.leaf[leaf_of(ahead) * 2 + 1];
            bool take = mine && takes(llo, lhi);
#pragma unroll
            for (int v = 0; v < 4; ++v) take = take && done[v] != at;
            append(queue, queued, take, at);
            node = ahead;
            llo = alo;
            lhi = ahi;
            if (queued <= limit) continue;
            if (!full()) return;
            left &= __ballot(takes(lo, hi));
            if (left != 0ull && static_cast<uint32_t>(__builtin_ctzll(left)) != node) {
                node = __builtin_ctzll(left);
                llo = j.leaf[leaf_of(node) * 2];
                lhi = j.leaf[leaf_of(node) * 2 + 1];
            }
        }
    }
}

}  // namespace cdk
