// Nearest neighbours in both directions by an exact pruned search over sorted
// clouds: cd_forward's path for large problems.  Its results are bitwise those
// of the all-pairs search (nn_search.hip): the same distance arithmetic, the
// lowest index among equal distances.
//
// The all-pairs search is bound by the FP32 VALU (B N M distances); a query
// needs only the few targets near it.  Here the clouds are sorted along a
// space-filling curve into leaves of 16 points with bounding boxes, 64 leaves
// to a node (spatial_sort.h), and a leaf is skipped when the distance to its
// box exceeds what a query already has.  The skip is exact, not approximate: a
// box's bound is evaluated like a distance, with the gap to the box in place
// of each coordinate difference; subtraction, product and FMA round
// monotonically, so it is at most the computed distance of every point in the
// box.  A leaf at exactly a query's distance is visited only if it holds an
// index below the query's.
//
//  * leaf_search_kernel: a wave takes the 16 queries of one leaf (they are
//    neighbours), the four rows of 16 lanes each another leaf of targets.  A
//    lane has a query and reads its row's targets by DPP row broadcasts; keys
//    (distance bits << 32 | index) are positive doubles, so that one v_min_f64
//    keeps the smallest distance and, among equal ones, the lowest index.
//    First bounds come from the four leaves nearest to the queries' box
//    (ordered by box distance plus a hundredth of the centres': boxes that meet
//    the queries' are all at 0, and in that order bounds were found in half the
//    visits).  Then the leaves within the bounds of the queries' box are queued,
//    each query lists those within its own, and a row visits one query's list,
//    a target per lane: 4.5 leaves per query on the mesh workload.
//  * query_search_kernel: where more than kSplit leaves are within the box's
//    bounds (queries far apart: outliers, or targets all about as far away), a
//    wave would take many times the others' time at the end of the launch (a
//    tenth of a millisecond, more than all the rest).  Such leaves of queries
//    go to a list, and a second launch searches for each of their queries in a
//    wave of its own.  Measured with a wave per four of them: slower on
//    outliers (245 against 157 us on the Gaussian mixtures), since their
//    common box is the problem.
//
// Bound by instruction issue and latency (about 1600 VALU instructions per 16
// queries on the mesh workload against 15000 for all pairs).  cd_forward, all
// pairs -> this (us, one box): 16 x 16384^2 mesh samples 496 -> 118; 4 x 100000 x
// 10000 mixture 480 -> 155; 8 x 65536^2 grid points 3660 -> 169; 1 x 30000 x 25001
// 102 -> 53; 1 x 200000^2 uniform 4500 -> 110.
#include "cd_internal.h"
#include "fixed_point.h"
#include "spatial_sort.h"

#include <algorithm>

namespace cdk {
namespace {

struct TreeSide {
    const float *P;         // [B, n, 3] the cloud
    float4 *entries;        // [B, chunks kSortChunk]
    Curve *curve;           // [B]
    uint32_t *offs;         // [B, chunks, ranges + 1]
    float4 *rec;            // [B, slots] sorted records
    Box *leaf, *node;       // [B, slots / kLeaf], [B, nodes]
    SortShape s;
};

struct TreeArgs {
    TreeSide side[2];
    uint32_t *list;         // counter and leaves of heavy queries
};

constexpr uint32_t kXcds = 8;
// The rule for this path.  Sorting and three to four dependent launches cost
// about 45 us whatever the size, the time of 3.5e8 pairs of the all-pairs
// search; measured, uniform clouds and mixtures gain from 4e8 pairs on (4 x
// 10000^2: 70 -> 50 us) but a sphere against a surface inside it, where each
// query is about as far from many targets, only from 2e9 (1e9: 135 -> 155 us, 2e9:
// 263 -> 258).  With a cloud of few points there is nothing to skip (17 x
// 100000: 47 us either way).
constexpr double kMinPairs = 7e8;
constexpr int64_t kMinCloud = 1800;
constexpr size_t kMaxTreeBytes = size_t{4} << 30;
constexpr uint32_t kQueryWaves = 8192;   // of the search for heavy queries
constexpr int kNear = 4;            // nodes looked at for the first bounds (2: 118 -> 133 us on meshes)
constexpr uint32_t kQueue = 192;    // leaves queued at most
constexpr uint32_t kDrain = 32;     // leaves a single query queues before it visits them
constexpr uint32_t kSplit = 128;    // and above this the queries are split
static_assert(kSplit + kWave <= kQueue && kDrain + kWave <= kQueue, "a node's leaves fit the queue");
constexpr uint32_t kList = 48;      // leaves listed per query

// Consecutive workgroups on one XCD (they are dealt out round-robin): the
// ranges and tiles of one item share one L2.
__device__ __forceinline__ uint32_t xcd_block()
{
    const uint32_t i = blockIdx.x, per = gridDim.x / kXcds;
    return i < kXcds * per ? (i % kXcds) * per + i / kXcds : i;
}

__global__ __launch_bounds__(kBucketThreads) void bucket_kernel(TreeArgs a)
{
    const uint32_t wg = xcd_block();
    const uint32_t c0 = a.side[0].s.chunks, c1 = a.side[1].s.chunks;
    const int64_t b = wg / (c0 + c1);
    const uint32_t c = wg % (c0 + c1);
    const TreeSide &t = a.side[c < c0 ? 0 : 1];
    if (t.s.ranges == 1) return;     // sorted straight from the cloud
    bucket_chunk(reinterpret_cast<const P3f *>(t.P) + b * t.s.n, t.s,
                 static_cast<int>(c < c0 ? c : c - c0),
                 t.entries + b * t.s.chunks * kSortChunk,
                 t.offs + b * t.s.chunks * (t.s.ranges + 1), t.curve + b);
}

__global__ __launch_bounds__(kSortThreads) void sort_kernel(TreeArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.list = 0u;
    const uint32_t wg = xcd_block();
    const uint32_t w0 = a.side[0].s.ranges, w1 = a.side[1].s.ranges;
    const int64_t b = wg / (w0 + w1);
    const uint32_t w = wg % (w0 + w1);
    const TreeSide &t = a.side[w < w0 ? 0 : 1];
    sort_range(reinterpret_cast<const P3f *>(t.P) + b * t.s.n, t.s,
               static_cast<int>(w < w0 ? w : w - w0), t.entries + b * t.s.chunks * kSortChunk,
               t.offs + b * t.s.chunks * (t.s.ranges + 1), t.curve + b,
               t.rec + b * t.s.nodes * kNode, t.leaf + b * t.s.nodes * kNodeLeaves,
               t.node + b * t.s.nodes);
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

__device__ __forceinline__ double min_key(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
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

// The two directions of a call: queries of cloud k against the other cloud.
struct SearchArgs {
    const float4 *rec[2], *leaf[2], *node[2];
    float *dist[2];
    int32_t *idx[2];
    uint32_t *list;         // [0]: heavy leaves of queries, [1..]: which
    SortShape s[2];
    int64_t B;
};

// A leaf of queries (numbered over items, directions and leaves) and the cloud
// they search.
struct Job {
    const float4 *qrec, *qleaf;                 // its records, its box
    const float4 *rec, *leaf, *node;            // the other cloud's
    float *dist;
    int32_t *idx;
    uint32_t nodes;
};

__device__ __forceinline__ Job job_of(const SearchArgs &a, uint32_t n)
{
    const uint32_t t0 = a.s[0].nodes * kNodeLeaves, t1 = a.s[1].nodes * kNodeLeaves;
    const int64_t b = n / (t0 + t1);
    uint32_t tile = n % (t0 + t1);
    const int k = tile < t0 ? 0 : 1;
    tile -= k == 0 ? 0u : t0;
    const int64_t nq = a.s[k].nodes, nt = a.s[1 - k].nodes;
    Job j;
    j.qrec = (k == 0 ? a.rec[0] : a.rec[1]) + b * nq * kNode + tile * kLeaf;
    j.qleaf = (k == 0 ? a.leaf[0] : a.leaf[1]) + (b * nq * kNodeLeaves + tile) * 2;
    j.rec = (k == 0 ? a.rec[1] : a.rec[0]) + b * nt * kNode;
    j.leaf = (k == 0 ? a.leaf[1] : a.leaf[0]) + b * nt * kNodeLeaves * 2;
    j.node = (k == 0 ? a.node[1] : a.node[0]) + b * nt * 2;
    j.dist = (k == 0 ? a.dist[0] : a.dist[1]) + b * a.s[k].n;
    j.idx = (k == 0 ? a.idx[0] : a.idx[1]) + b * a.s[k].n;
    j.nodes = static_cast<uint32_t>(nt);
    return j;
}

// The four leaves nearest to the box [qlo, qhi] (each the nearest of one
// lane's) in the kNear nearest nodes; ~0: every distance overflows.  Order:
// box distance, then that of the centres (boxes that meet are all at 0).
// nlo, nhi: box of node min(lane, nodes - 1).
__device__ __forceinline__ void nearest_leaves(const Job &j, const float4 &qlo, const float4 &qhi,
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

// Appends v of the lanes that take it to a list of n values in LDS.
__device__ __forceinline__ void append(uint32_t *list, uint32_t &n, bool take, uint32_t v)
{
    const uint64_t taken = __ballot(take);
    if (take)
        list[__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(taken >> 32),
            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(taken), n))] = v;
    n += __popcll(taken);
}

// Queues the leaves, other than the four done, within the bound `worst` of the
// box [qlo, qhi] (of those at that very distance, the ones with an index below
// `last`).  full() is called when more than `limit` are queued and ends the
// walk by returning false; it may empty the queue and tighten the bounds.
template <class Full>
__device__ __forceinline__ void gather(const Job &j, const float4 &qlo, const float4 &qhi,
                                       const float4 &nlo, const float4 &nhi, uint32_t lane,
                                       const uint32_t done[4], const float &worst,
                                       const uint32_t &last, uint32_t *queue, uint32_t &queued,
                                       uint32_t limit, const Full &full)
{
    const auto within = [&](float d, uint32_t first) {
        return d < worst || (d == worst && first < last);
    };
    for (uint32_t from = 0; from < j.nodes; from += kWave) {
        float4 lo = nlo, hi = nhi;
        if (from > 0u) {
            const uint32_t i = min(from + lane, j.nodes - 1);
            lo = j.node[2 * i];
            hi = j.node[2 * i + 1];
        }
        const float d = bound(qlo, qhi, lo, hi);
        const uint32_t first = from + lane < j.nodes && lo.x <= hi.x ? __float_as_uint(lo.w) : kNoPoint;
        uint64_t left = ~0ull;
        for (;;) {
            left &= __ballot(first != kNoPoint && within(d, first));
            if (left == 0ull) break;
            const uint32_t at = (from + __builtin_ctzll(left)) * kNodeLeaves + lane;
            left &= left - 1ull;
            const float4 llo = j.leaf[at * 2], lhi = j.leaf[at * 2 + 1];
            bool take = within(bound(qlo, qhi, llo, lhi), __float_as_uint(llo.w)) && llo.x <= lhi.x;
#pragma unroll
            for (int v = 0; v < 4; ++v) take = take && done[v] != at;
            append(queue, queued, take, at);
            if (queued > limit && !full()) return;
        }
    }
}

// One wave: the 16 queries of a leaf.
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(7, 8)))
void leaf_search_kernel(SearchArgs a)
{
    __shared__ float4 query[kLeaf];
    __shared__ unsigned long long found[kLeaf];     // best key of each query
    __shared__ __attribute__((aligned(16))) uint32_t lists[kLeaf][kList];
    __shared__ uint32_t queue[kQueue];
    const uint32_t lane = threadIdx.x, sub = lane & 15u, row = lane >> 4;
    const uint32_t n = xcd_block();
    const Job j = job_of(a, n);
    const float4 qlo = j.qleaf[0], qhi = j.qleaf[1];
    const uint32_t n0 = min(lane, j.nodes - 1);
    const float4 nlo = j.node[2 * n0], nhi = j.node[2 * n0 + 1];
    const float4 q = j.qrec[sub];
    if (!(qlo.x <= qhi.x)) return;
    const uint32_t id = __float_as_uint(q.w);

    // 1. Bounds: all queries visit the four leaves nearest to their box, one
    // per row.
    uint32_t done[4], mine = 0u;
    nearest_leaves(j, qlo, qhi, nlo, nhi, lane, done);
    // A slot without a point beats everything.
    double best = id != kNoPoint ? pack(__builtin_inff(), kNoPoint) : 0.0;
    if (done[0] != kNoPoint) {
#pragma unroll
        for (int v = 0; v < 4; ++v) mine = row == static_cast<uint32_t>(v) ? done[v] : mine;
        double k[kLeaf];
        leaf_keys<0>(q, j.rec[mine * kLeaf + sub], k);
#pragma unroll
        for (int s = kLeaf / 2; s > 0; s >>= 1)
#pragma unroll
            for (int u = 0; u < s; ++u) k[u] = min_key(k[u], k[u + s]);
        best = rows_min(min_key(best, k[0]));
    }
    const float worst = row_max(high(best));
    const uint32_t last = row_max_u32(static_cast<uint32_t>(__double2loint(best)));
    if (lane < kLeaf) {
        query[sub] = q;
        found[sub] = as_bits(best);
    }

    const uint32_t leaf0 = done[0] != kNoPoint ? done[0] : 0u;   // fills up a list

    // 2. The other leaves within the bounds of the box are queued.  Too many
    // (queries far apart, or as far from all targets): a wave each.
    uint32_t queued = 0u;
    bool heavy = false;
    gather(j, qlo, qhi, nlo, nhi, lane, done, worst, last, queue, queued, kSplit,
           [&] { heavy = true; return false; });
    if (heavy) {
        if (lane == 0u) a.list[1u + atomicAdd(a.list, 1u)] = n;
        return;
    }
    // Each query takes those within its own bound to its list; row r visits
    // the lists of queries r, 4 + r, 8 + r and 12 + r, a target per lane.
    __builtin_amdgcn_wave_barrier();
    uint32_t listed[kLeaf / 4];
#pragma unroll
    for (uint32_t p = 0; p < kLeaf / 4; ++p) listed[p] = 0u;
    for (uint32_t c = 0u; c < queued; c += kLeaf) {
        const uint32_t leaf = queue[min(c + sub, queued - 1u)];
        const float4 lo = j.leaf[leaf * 2], hi = j.leaf[leaf * 2 + 1];
        bool full = c + kLeaf >= queued;
#pragma unroll
        for (uint32_t p = 0; p < kLeaf / 4; ++p) {
            const uint32_t i = p * 4 + row;
            const float4 u = query[i];
            const float d = sum_sq(gap(u.x, u.x, lo.x, hi.x), gap(u.y, u.y, lo.y, hi.y),
                                   gap(u.z, u.z, lo.z, hi.z));
            const bool take = c + sub < queued && pack(d, __float_as_uint(lo.w)) < as_key(found[i]);
            const uint32_t taken = static_cast<uint32_t>(__ballot(take) >> (row * 16u)) & 0xffffu;
            if (take) lists[i][listed[p] + __popc(taken & ((1u << sub) - 1u))] = leaf;
            listed[p] += __popc(taken);
            full |= listed[p] > kList - kLeaf;
        }
        if (__ballot(full) == 0ull) continue;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (uint32_t p = 0; p < kLeaf / 4; ++p) {
            const uint32_t i = p * 4 + row;
            const float4 u = query[i];
            double k = as_key(found[i]);
            for (uint32_t s = 0u; __ballot(s < listed[p]) != 0ull; s += 4u) {
                const uint4 l = *reinterpret_cast<const uint4 *>(&lists[i][s]);
                float4 t[4];
                t[0] = j.rec[(s < listed[p] ? l.x : leaf0) * kLeaf + sub];
                t[1] = j.rec[(s + 1u < listed[p] ? l.y : leaf0) * kLeaf + sub];
                t[2] = j.rec[(s + 2u < listed[p] ? l.z : leaf0) * kLeaf + sub];
                t[3] = j.rec[(s + 3u < listed[p] ? l.w : leaf0) * kLeaf + sub];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    k = min_key(k, pack(sum_sq(t[v].x - u.x, t[v].y - u.y, t[v].z - u.z),
                                        __float_as_uint(t[v].w)));
            }
            k = min_key(k, dpp_key<0xB1>(k));
            k = min_key(k, dpp_key<0x4E>(k));
            k = min_key(k, dpp_key<0x141>(k));
            k = min_key(k, dpp_key<0x140>(k));
            if (sub == 0u) found[i] = as_bits(k);
            listed[p] = 0u;
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (id != kNoPoint && row == 0u) {
        best = as_key(found[sub]);
        j.dist[id] = high(best);
        j.idx[id] = __double2loint(best);
    }
}

// One wave: one query of a listed leaf at a time.
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(8, 8)))
void query_search_kernel(SearchArgs a)
{
    __shared__ uint32_t queue[kQueue];
    const uint32_t lane = threadIdx.x, sub = lane & 15u, row = lane >> 4;
    const uint32_t items = a.list[0] * kLeaf;
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        const Job j = job_of(a, a.list[1u + item / kLeaf]);
        const float4 q = j.qrec[item % kLeaf];
        const uint32_t n0 = min(lane, j.nodes - 1);
        const float4 nlo = j.node[2 * n0], nhi = j.node[2 * n0 + 1];
        const uint32_t id = __float_as_uint(q.w);
        if (id == kNoPoint) continue;
        double best = pack(__builtin_inff(), kNoPoint);
        float worst = __builtin_inff();
        uint32_t last = kNoPoint;
        const auto visit = [&](const float4 &t) {
            best = min_key(best, pack(sum_sq(t.x - q.x, t.y - q.y, t.z - q.z), __float_as_uint(t.w)));
        };
        const auto settle = [&] {
            best = min_key(best, dpp_key<0xB1>(best));
            best = min_key(best, dpp_key<0x4E>(best));
            best = min_key(best, dpp_key<0x141>(best));
            best = rows_min(min_key(best, dpp_key<0x140>(best)));
            worst = high(best);
            last = static_cast<uint32_t>(__double2loint(best));
        };
        uint32_t done[4];
        nearest_leaves(j, q, q, nlo, nhi, lane, done);
        if (done[0] != kNoPoint) {
            uint32_t mine = done[0];
#pragma unroll
            for (int v = 1; v < 4; ++v) mine = row == static_cast<uint32_t>(v) ? done[v] : mine;
            visit(j.rec[mine * kLeaf + sub]);
            settle();
        }
        uint32_t queued = 0u;
        const auto drain = [&] {
            __builtin_amdgcn_wave_barrier();
            for (uint32_t c = 0u; c < queued; c += 16u) {
                float4 t[4];
#pragma unroll
                for (uint32_t v = 0u; v < 4u; ++v)
                    t[v] = j.rec[queue[min(c + 4u * v + row, queued - 1u)] * kLeaf + sub];
#pragma unroll
                for (uint32_t v = 0u; v < 4u; ++v) visit(t[v]);
            }
            if (queued > 0u) settle();
            queued = 0u;
            __builtin_amdgcn_wave_barrier();
            return true;
        };
        gather(j, q, q, nlo, nhi, lane, done, worst, last, queue, queued, kDrain, drain);
        drain();
        if (lane == 0u) {
            j.dist[id] = high(best);
            j.idx[id] = __double2loint(best);
        }
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

int ceil_log2(int64_t x)
{
    int l = 0;
    while ((int64_t{1} << l) < x) ++l;
    return l;
}

}  // namespace

TreePlan plan_tree(int64_t B, int64_t N, int64_t M)
{
    TreePlan p{};
    p.B = B;
    const int64_t n[2] = {N, M};
    if (std::max(N, M) > static_cast<int64_t>(kMaxChunks) * kSortChunk) return p;
    size_t at = 0;
    for (int k = 0; k < 2; ++k) {
        p.chunks[k] = static_cast<int32_t>(ceil_div(n[k], kSortChunk));
        p.ranges[k] = n[k] <= kOneRange ? 1 : static_cast<int32_t>(std::min<int64_t>(
                                                  ceil_div(n[k], kRangePoints), kMaxRanges));
        p.log_c[k] = std::min(std::max(ceil_log2(n[k]) + 2, 9), kLogCells);
        p.nodes[k] = static_cast<int32_t>(ceil_div(n[k], kNode) + p.ranges[k]);
    }
    p.bucket = p.ranges[0] > 1 || p.ranges[1] > 1;
    for (int k = 0; k < 2; ++k) {
        p.entries[k] = at;
        if (p.bucket) at += align256(static_cast<size_t>(B) * p.chunks[k] * kSortChunk * sizeof(float4));
        p.offs[k] = at;
        if (p.bucket) at += align256(static_cast<size_t>(B) * p.chunks[k] * (p.ranges[k] + 1) * 4);
        p.curve[k] = at;
        at += align256(static_cast<size_t>(B) * sizeof(Curve));
        p.rec[k] = at;
        at += align256(static_cast<size_t>(B) * p.nodes[k] * kNode * sizeof(float4));
        p.leaf[k] = at;
        at += align256(static_cast<size_t>(B) * p.nodes[k] * kNodeLeaves * sizeof(Box));
        p.node[k] = at;
        at += align256(static_cast<size_t>(B) * p.nodes[k] * sizeof(Box));
    }
    p.list = at;
    at += align256(4 * (1 + static_cast<size_t>(B) * (p.nodes[0] + p.nodes[1]) * kNodeLeaves));
    p.bytes = at;
    // Where the pairs take longer than the sort and its launches (see above).
    p.use = static_cast<double>(B) * N * M >= kMinPairs && std::min(N, M) >= kMinCloud &&
            p.bytes <= kMaxTreeBytes;
    return p;
}

hipError_t launch_tree(const TreePlan &p, int64_t N, int64_t M, const FwdArgs &f, hipStream_t stream)
{
    TreeArgs a{};
    char *base = static_cast<char *>(f.ws);
    for (int k = 0; k < 2; ++k) {
        TreeSide &t = a.side[k];
        t.P = k == 0 ? f.X : f.Y;
        t.entries = reinterpret_cast<float4 *>(base + p.entries[k]);
        t.offs = reinterpret_cast<uint32_t *>(base + p.offs[k]);
        t.curve = reinterpret_cast<Curve *>(base + p.curve[k]);
        t.rec = reinterpret_cast<float4 *>(base + p.rec[k]);
        t.leaf = reinterpret_cast<Box *>(base + p.leaf[k]);
        t.node = reinterpret_cast<Box *>(base + p.node[k]);
        t.s.n = static_cast<int32_t>(k == 0 ? N : M);
        t.s.ranges = p.ranges[k];
        t.s.log_c = p.log_c[k];
        t.s.chunks = p.chunks[k];
        t.s.nodes = p.nodes[k];
    }
    a.list = reinterpret_cast<uint32_t *>(base + p.list);
    if (p.bucket)
        bucket_kernel<<<static_cast<uint32_t>(p.B * (p.chunks[0] + p.chunks[1])), kBucketThreads, 0,
                        stream>>>(a);
    sort_kernel<<<static_cast<uint32_t>(p.B * (static_cast<int64_t>(p.ranges[0]) + p.ranges[1])), kSortThreads,
                  0, stream>>>(a);
    SearchArgs s{};
    for (int k = 0; k < 2; ++k) {
        s.rec[k] = a.side[k].rec;
        s.leaf[k] = reinterpret_cast<const float4 *>(a.side[k].leaf);
        s.node[k] = reinterpret_cast<const float4 *>(a.side[k].node);
        s.s[k] = a.side[k].s;
    }
    s.dist[0] = f.dist_xy;
    s.dist[1] = f.dist_yx;
    s.idx[0] = f.idx_xy;
    s.idx[1] = f.idx_yx;
    s.list = a.list;
    s.B = p.B;
    const uint32_t leaves = static_cast<uint32_t>(p.B * (static_cast<int64_t>(p.nodes[0]) + p.nodes[1]) * kNodeLeaves);
    leaf_search_kernel<<<leaves, kWave, 0, stream>>>(s);
    query_search_kernel<<<std::min<uint32_t>(leaves * kLeaf, kQueryWaves), kWave, 0, stream>>>(s);
    return hipGetLastError();
}

}  // namespace cdk
