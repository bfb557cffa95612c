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
//    common box is the problem; with a workgroup per leaf and its 16 queries
//    sharing the targets' loads: 173 -> 192 us there, 4 x 60000 x 3001 90 -> 144, for
//    131 -> 123 on a template.  Where nearly every query would visit nearly all
//    targets, it takes all of them, from the clouds as they are.
//
// Bound by instruction issue and latency (about 1600 VALU instructions per 16
// queries on the mesh workload against 15000 for all pairs).  cd_forward, all
// pairs -> this (us, calls back to back): 16 x 16384^2 mesh samples 525 -> 126; 4 x
// 100000 x 10000 mixture 505 -> 174; 8 x 65536^2 grid points 3660 -> 200; 1 x 30000 x
// 25001 110 -> 57; 1 x 200000^2 uniform 4600 -> 184.
#include "cd_internal.h"
#include "fixed_point.h"
#include "spatial_sort.h"

#include <algorithm>

namespace cdk {
namespace {

// The rule for this path.  Sorting and three to four dependent launches cost
// about 45 us whatever the size, the time of 3.5e8 pairs of the all-pairs
// search.  Measured, all pairs -> this (us), and a template (a sphere against a
// surface inside it, where each query is about as far from many targets), the
// worst of the kinds looked at that are not all of that sort:
//                       template    mesh       uniform    sphere     mixture
//   1 x 26645^2 (7.1e8)  113 128    113  56    107  43    106  49    115  58
//   16 x 6661^2 (7.1e8)  123 129    124  78    128  70    124  58    128  70
//   4 x 60000 x 3001     115 161    113  90    113  87    113  79    114  95
//   1 x 31622^2 (1e9)    142 147    144  61    145  49    145  57    144  56
//   8 x 3001 x 40000     169 127    174 100    172  83    172  70    180  83
//   16 x 11180^2 (2e9)   283 240    281  98    281  81    280  75    285  90
//   16 x 15811^2 (4e9)   505 385    517 117    513 102    514  94    513 118
// The line is where every other kind gains at least a fifth, most of them twice;
// templates lose up to 14% below 1.2e9 pairs, and up to 40% where a small cloud is
// set against a large one.  Clouds where every query is as far from all targets
// (a sphere around its centre) lose at any size, up to 3 times (kAllShare).  With
// a cloud of few points there is nothing to skip (17 x 100000: 47 us either way).
constexpr double kMinPairs = 7e8;
constexpr int64_t kMinCloud = 1800;
constexpr size_t kMaxTreeBytes = size_t{4} << 30;
constexpr int kQueryWaves = 4;           // of a workgroup of the search for heavy queries
constexpr int kQueryThreads = kQueryWaves * kWave;
constexpr uint32_t kQueryGroups = 2048;  // workgroups of it at most
constexpr int kBatch = 32;               // targets per batch where it takes all
constexpr uint32_t kQueue = 192;    // leaves queued at most
constexpr uint32_t kDrain = 32;     // leaves a single query queues before it visits them
constexpr uint32_t kSplit = 128;    // and above this the queries are split
static_assert(kSplit + kWave <= kQueue && kDrain + kWave <= kQueue, "a node's leaves fit the queue");
// Where more than this share of all leaves of queries is heavy, and clouds are
// not so large that kSplit leaves of targets are few, all targets are taken
// instead (search_all).  Measured, share: us with the tree, with all targets, and of
// the all-pairs search, which shares its distances between the directions:
// template 16 x 15811^2 0.22: 385, -, 505; lognormal radii 64 x 4000^2 0.58: 374, -, 153;
// a sphere of 30000 points around 25001 0.81: 500, 330, 105, 16 x 16384^2 0.84: 3190,
// 1290, 505; around a cluster 1.0: 3740, 1280, 510.  (Lognormal radii 16 x 16384^2,
// 0.82, take 1320 for 700.)  Handing such calls back to the all-pairs kernels
// (650 us) costs two launches that mostly do nothing, 5 us of every call; a
// count of the nodes in the bounds of each heavy leaf, for large clouds too, 3 us.
constexpr double kAllShare = 0.75;
constexpr double kAllMostPairs = 1.7e9;  // of an item (1 x 200000^2 lognormal, 0.58: 1260, all pairs 4800)
constexpr uint32_t kList = 48;      // leaves listed per query

// The two directions of a call: queries of cloud k against the other cloud.
struct SearchArgs {
    const float4 *rec[2], *leaf[2], *node[2];
    float *dist[2];
    int32_t *idx[2];
    uint32_t *list;         // heavy leaves of queries (below)
    uint32_t leaves, items; // leaves of queries, over items and directions; items
    const float *cloud[2];  // [B, n, 3]
    uint32_t most_heavy;    // leaves; with more all targets are taken
    SortShape s[2];
};

// The list of heavy leaves: kStripes lists, leaf n in list n % kStripes, so that
// the waves that add to them seldom meet at one counter (10 ns each time; 32768
// heavy leaves with one counter: 380 us).  Their lengths, kStride words apart, then
// their entries.
constexpr uint32_t kStripes = kWave;
constexpr uint32_t kStride = 32;

__host__ __device__ __forceinline__ uint32_t stripe_room(uint32_t leaves)
{
    return (leaves + kStripes - 1) / kStripes;
}

// A leaf of queries (numbered over items, directions and leaves) and the cloud
// they search.
struct Job {
    const float4 *qrec, *qleaf;                 // its records, its box
    const float4 *rec;                          // the other cloud's
    Targets t;
    float *dist;
    int32_t *idx;
    uint32_t nq, nt;                            // points of the two clouds

    // Query i's neighbour.  Records, leaf numbers and indices are read from
    // the workspace, which calls that overlap share (cd_forward_noalloc): each is
    // bounded before it is an address, and an index that leaves the call is
    // one of a target or -1.
    __device__ __forceinline__ void store(uint32_t i, float d, uint32_t target) const
    {
        if (i >= nq) return;
        dist[i] = d;
        idx[i] = target < nt ? static_cast<int32_t>(target) : -1;
    }
};

// Whether a box can hold something nearer than `worst` to the box [qlo, qhi],
// or as near with an index below `last`.
__device__ __forceinline__ bool within(const float4 &qlo, const float4 &qhi, const float4 &lo,
                                       const float4 &hi, float worst, uint32_t last)
{
    const float d = bound(qlo, qhi, lo, hi);
    return lo.x <= hi.x && (d < worst || (d == worst && __float_as_uint(lo.w) < last));
}

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
    j.t.leaf = (k == 0 ? a.leaf[1] : a.leaf[0]) + b * nt * kNodeLeaves * 2;
    j.t.node = (k == 0 ? a.node[1] : a.node[0]) + b * nt * 2;
    j.dist = (k == 0 ? a.dist[0] : a.dist[1]) + b * a.s[k].n;
    j.idx = (k == 0 ? a.idx[0] : a.idx[1]) + b * a.s[k].n;
    j.t.nodes = static_cast<uint32_t>(nt);
    j.nq = static_cast<uint32_t>(a.s[k].n);
    j.nt = static_cast<uint32_t>(a.s[1 - k].n);
    return j;
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
    const uint32_t n0 = min(lane, j.t.nodes - 1);
    const float4 nlo = j.t.node[2 * n0], nhi = j.t.node[2 * n0 + 1];
    const float4 q = j.qrec[sub];
    if (nan_query(q, qhi) && row == 0u)     // nothing is near it
        j.store(__float_as_uint(q.z), __builtin_inff(), kNoPoint);
    if (!(qlo.x <= qhi.x)) return;
    const uint32_t id = __float_as_uint(q.w);

    // 1. Bounds: all queries visit the four leaves nearest to their box, one
    // per row.
    uint32_t done[4], mine = 0u;
    nearest_leaves(j.t, qlo, qhi, nlo, nhi, lane, done);
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

    // 2. The other leaves within the bounds of the box are queued.  Too many
    // (queries far apart, or as far from all targets): a wave each.
    uint32_t queued = 0u;
    bool heavy = false;
    gather(j.t, nlo, nhi, lane, done, queue, queued, kSplit, true,
           [&](const float4 &lo, const float4 &hi) { return within(qlo, qhi, lo, hi, worst, last); },
           [&] { heavy = true; return false; });
    if (heavy) {
        if (lane == 0u) {
            const uint32_t s = n % kStripes, room = stripe_room(a.leaves);
            const uint32_t at = atomicAdd(a.list + s * kStride, 1u);
            if (at < room) a.list[kStripes * kStride + s * room + at] = n;
        }
        return;
    }
    wave_sync();
    // Each query takes those within its own bound to its list; row r visits
    // the lists of queries r, 4 + r, 8 + r and 12 + r, a target per lane.
    const uint32_t fill = queued > 0u ? queue[0] : 0u;   // a leaf with points, to fill a list up
    uint32_t listed[kLeaf / 4];
#pragma unroll
    for (uint32_t p = 0; p < kLeaf / 4; ++p) listed[p] = 0u;
    for (uint32_t c = 0u; c < queued; c += kLeaf) {
        const uint32_t leaf = queue[min(c + sub, queued - 1u)];
        const float4 lo = j.t.leaf[leaf * 2], hi = j.t.leaf[leaf * 2 + 1];
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
        wave_sync();
#pragma unroll
        for (uint32_t p = 0; p < kLeaf / 4; ++p) {
            const uint32_t i = p * 4 + row;
            const float4 u = query[i];
            double k = as_key(found[i]);
            for (uint32_t s = 0u; __ballot(s < listed[p]) != 0ull; s += 4u) {
                const uint4 l = *reinterpret_cast<const uint4 *>(&lists[i][s]);
                float4 t[4];
                t[0] = j.rec[(s < listed[p] ? l.x : fill) * kLeaf + sub];
                t[1] = j.rec[(s + 1u < listed[p] ? l.y : fill) * kLeaf + sub];
                t[2] = j.rec[(s + 2u < listed[p] ? l.z : fill) * kLeaf + sub];
                t[3] = j.rec[(s + 3u < listed[p] ? l.w : fill) * kLeaf + sub];
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
        wave_sync();
    }
    if (id != kNoPoint && row == 0u) {
        best = as_key(found[sub]);
        j.store(id, high(best), static_cast<uint32_t>(__double2loint(best)));
    }
}

using Constant = __attribute__((address_space(4))) float;

// All targets for 64 queries of a cloud, those numbered `group` over items and
// directions: a query per lane, a share of the targets per wave.  As in the
// all-pairs search, the index of the minimum is looked for in the batch of
// targets that last lowered it.
__device__ __forceinline__ void search_all(const SearchArgs &a, uint32_t group, uint32_t wave,
                                           uint32_t lane, double (&part)[kQueryWaves][kWave])
{
    const uint32_t g0 = (a.s[0].n + kWave - 1) / kWave, g1 = (a.s[1].n + kWave - 1) / kWave;
    const int64_t b = group / (g0 + g1);
    uint32_t g = group % (g0 + g1);
    const int k = g < g0 ? 0 : 1;
    g -= k == 0 ? 0u : g0;
    const int nq = k == 0 ? a.s[0].n : a.s[1].n, nt = k == 0 ? a.s[1].n : a.s[0].n;
    const int64_t q = b * nq + min(static_cast<int>(g * kWave + lane), nq - 1);
    const float *Q = (k == 0 ? a.cloud[0] : a.cloud[1]) + 3 * q;
    // Memory that the launch does not write: scalar loads, although the results of
    // the workgroup's last queries were stored.
    const Constant *T = reinterpret_cast<const Constant *>(
        reinterpret_cast<uintptr_t>((k == 0 ? a.cloud[1] : a.cloud[0]) + 3 * b * nt));
    const float qx = Q[0], qy = Q[1], qz = Q[2];
    const auto dist = [&](const Constant *t) { return sum_sq(t[0] - qx, t[1] - qy, t[2] - qz); };
    const int per = (nt + kQueryWaves * kBatch - 1) / (kQueryWaves * kBatch) * kBatch;
    const int t0 = min(static_cast<int>(wave) * per, nt), t1 = min(t0 + per, nt);
    float best = __builtin_inff();
    int from = t0, t = t0;
    for (; t + kBatch <= t1; t += kBatch) {
        const Constant *p = T + 3 * t;      // the same in all lanes
        float m = __builtin_inff();
#pragma unroll
        for (int u = 0; u < kBatch; u += 2) {
            const float d0 = dist(p + 3 * u), d1 = dist(p + 3 * u + 3);
            asm("v_min3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(m), "v"(d0), "v"(d1));
        }
        from = m < best ? t : from;
        best = m < best ? m : best;
    }
#pragma unroll 1
    for (int u = t; u < t1; ++u) {
        const float d = dist(T + 3 * u);
        from = d < best ? t : from;
        best = d < best ? d : best;
    }
    uint32_t at = kNoPoint;
    if (best < __builtin_inff())
#pragma unroll 1
        for (int u = min(from + kBatch, t1) - 1; u >= from; --u)
            at = dist(T + 3 * u) == best ? u : at;
    part[wave][lane] = pack(best, at);
    __syncthreads();
    if (wave == 0u && g * kWave + lane < static_cast<uint32_t>(nq)) {
        double key = part[0][lane];
#pragma unroll
        for (int w = 1; w < kQueryWaves; ++w) key = min_key(key, part[w][lane]);
        (k == 0 ? a.dist[0] : a.dist[1])[q] = high(key);
        (k == 0 ? a.idx[0] : a.idx[1])[q] = __double2loint(key);
    }
    __syncthreads();
}

// A wave takes one query of a listed leaf at a time; or, where those are expected
// to visit too many leaves, a workgroup all targets for 64 queries.
__global__ __launch_bounds__(kQueryThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
void query_search_kernel(SearchArgs a)
{
    __shared__ uint32_t queues[kQueryWaves][kQueue];
    __shared__ double part[kQueryWaves][kWave];
    const uint32_t lane = threadIdx.x % kWave, sub = lane & 15u, row = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t *queue = queues[wave];
    // Lane l: the entries of lists 0 to l.
    const uint32_t room = stripe_room(a.leaves);
    uint32_t upto = min(a.list[lane * kStride], room);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(upto, d, kWave);
        upto += lane >= static_cast<uint32_t>(d) ? o : 0u;
    }
    const uint32_t heavy = __builtin_amdgcn_readlane(upto, kWave - 1), items = heavy * kLeaf;
    if (heavy > a.most_heavy) {
        const uint32_t groups = a.items * ((a.s[0].n + kWave - 1) / kWave + (a.s[1].n + kWave - 1) / kWave);
        for (uint32_t g = blockIdx.x; g < groups; g += gridDim.x) search_all(a, g, wave, lane, part);
        return;
    }
    for (uint32_t item = blockIdx.x * kQueryWaves + wave; item < items; item += gridDim.x * kQueryWaves) {
        const uint32_t s = __popcll(__ballot(upto <= item / kLeaf));
        const uint32_t at = item / kLeaf - (s > 0u ? __builtin_amdgcn_readlane(upto, s - 1u) : 0u);
        const Job j = job_of(a, min(a.list[kStripes * kStride + s * room + at], a.leaves - 1u));
        const float4 q = j.qrec[item % kLeaf];
        const uint32_t n0 = min(lane, j.t.nodes - 1);
        const float4 nlo = j.t.node[2 * n0], nhi = j.t.node[2 * n0 + 1];
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
        nearest_leaves(j.t, q, q, nlo, nhi, lane, done);
        if (done[0] != kNoPoint) {
            uint32_t mine = done[0];
#pragma unroll
            for (int v = 1; v < 4; ++v) mine = row == static_cast<uint32_t>(v) ? done[v] : mine;
            visit(j.rec[mine * kLeaf + sub]);
            settle();
        }
        uint32_t queued = 0u;
        const auto drain = [&] {
            wave_sync();
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
            wave_sync();
            return true;
        };
        gather(j.t, nlo, nhi, lane, done, queue, queued, kDrain, true,
               [&](const float4 &lo, const float4 &hi) { return within(q, q, lo, hi, worst, last); },
               drain);
        drain();
        if (lane == 0u) j.store(id, high(best), static_cast<uint32_t>(__double2loint(best)));
    }
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct TreeLayout {
    SortPlan sort[2];
    size_t list, bytes;
};

TreeLayout layout(int64_t B, int64_t N, int64_t M)
{
    TreeLayout l{};
    size_t at = 0;
    l.sort[0] = plan_sort(B, N, at);
    l.sort[1] = plan_sort(B, M, at);
    l.list = at;
    const size_t leaves = static_cast<size_t>(B) * (l.sort[0].s.nodes + l.sort[1].s.nodes) * kNodeLeaves;
    l.bytes = at + align256(4 * kStripes * (kStride + (leaves + kStripes - 1) / kStripes));
    return l;
}

}  // namespace

size_t tree_workspace_bytes(int64_t B, int64_t N, int64_t M)
{
    // Where the pairs take longer than the sort and its launches (see above).
    if (static_cast<double>(B) * N * M < kMinPairs || std::min(N, M) < kMinCloud ||
        std::max(N, M) > kSortMaxPoints)
        return 0;
    const size_t bytes = layout(B, N, M).bytes;
    return bytes <= kMaxTreeBytes ? bytes : 0;
}

hipError_t launch_tree(int64_t B, int64_t N, int64_t M, const FwdArgs &f, hipStream_t stream)
{
    const TreeLayout l = layout(B, N, M);
    char *base = static_cast<char *>(f.ws);
    const SortJob job[2] = {sort_job(l.sort[0], f.X, base), sort_job(l.sort[1], f.Y, base)};
    SearchArgs s{};
    s.list = reinterpret_cast<uint32_t *>(base + l.list);
    const hipError_t e = launch_sort(B, job[0], job[1], s.list, kStripes * kStride, stream);
    if (e != hipSuccess) return e;
    for (int k = 0; k < 2; ++k) {
        s.rec[k] = job[k].rec;
        s.leaf[k] = reinterpret_cast<const float4 *>(job[k].leaf);
        s.node[k] = reinterpret_cast<const float4 *>(job[k].node);
        s.s[k] = job[k].s;
    }
    s.dist[0] = f.dist_xy;
    s.dist[1] = f.dist_yx;
    s.idx[0] = f.idx_xy;
    s.idx[1] = f.idx_yx;
    const uint32_t leaves = static_cast<uint32_t>(
        B * (static_cast<int64_t>(s.s[0].nodes) + s.s[1].nodes) * kNodeLeaves);
    s.leaves = leaves;
    leaf_search_kernel<<<leaves, kWave, 0, stream>>>(s);
    s.most_heavy = static_cast<double>(N) * M <= kAllMostPairs
                       ? static_cast<uint32_t>(kAllShare * static_cast<double>(B) * (N + M) / kLeaf)
                       : leaves;
    s.items = static_cast<uint32_t>(B);
    s.cloud[0] = f.X;
    s.cloud[1] = f.Y;
    query_search_kernel<<<std::min((leaves * kLeaf + kQueryWaves - 1) / kQueryWaves, kQueryGroups),
                          kQueryThreads, 0, stream>>>(s);
    return hipGetLastError();
}

}  // namespace cdk
