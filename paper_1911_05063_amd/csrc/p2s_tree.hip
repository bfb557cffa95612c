// Point-to-surface distances by an exact pruned search over sorted points and
// faces: cd_p2s_forward's path for large meshes.  The results are bitwise those
// of the all-pairs search (p2s.hip): the same distance of every (point, face)
// visited, the lowest face index among equal distances.
//
// The all-pairs search is bound by the FP32 VALU (52 instructions a pair).
// Here points, and faces by their centroids, are sorted (spatial_sort.h) into
// leaves of 16, and a leaf of faces is skipped when no computed distance to one
// of its faces can be as small as what a point already has.
//
// That needs a bound on the computed distances, not the true ones.  With R the
// largest distance from the point to a corner of the face, h and the segment
// residuals carry at most 8 2^-24 R of rounding each.  The barycentric s, t
// carry 8 2^-24 R |g0|, |g1|, so a point just outside may be taken for one
// inside, at the distance of the plane: its projection then lies within the
// triangle of the shifted edges, whose corners are at most
// 16 2^-24 R (|g0| + |g1|) (|e0| + |e1|) (and 8 2^-24 R for 1 - s - t) from the
// face's.  So computed distance >= true distance - m R with
// m = (64 + 32 (|g0| + |g1|) (|e0| + |e1|)) 2^-24, twice those sums; a needle has a
// large m and is never skipped.  A leaf keeps the largest m of its faces and m
// times its diagonal D; R is at most the distance d to its box plus D, hence
// it is skipped only if (d - m d - m D)^2 exceeds the point's distance.
//
//  * centroid_kernel, the sort's launches, then face_leaf_kernel: a node of 1024
//    sorted faces per workgroup, records and boxes.
//  * face_search_kernel: a wave takes the 16 points of a leaf; its rows of 16
//    lanes take four leaves of faces, a face per lane, whose records stay in
//    VGPRs while the points that need any of the four are evaluated one after
//    the other (coordinates in SGPRs): one load of a record serves up to 16
//    points, and no lane exchange is needed until the end but for the bounds.
//    The four leaves nearest to the points come first, then the others within
//    the bounds of the points' box.
//
// Measured (us, all pairs -> this): 16 x 16384 points against 5120 faces 1266 ->
// 148, 16 x 11284 against 7200 1347 -> 154.
// The search itself takes 109 us of the first: about 4500 VALU instructions per
// 16 points, issue bound at three waves per SIMD (163 VGPRs; four waves spill
// and take 10 us more).
#include <algorithm>

#include "p2s_face.h"
#include "spatial_sort.h"

namespace cdk {
namespace {

// The rule for this path.  The sort and the records cost about 45 us, the time
// of 5e7 pairs of the all-pairs search; from 1.5e8 pairs on surfaces gain twice
// that and more.  Boxes around few, large triangles skip little, and meshes below
// 2048 faces keep all pairs (2000 random triangles 566 -> 602 us, 1000 137 -> 193);
// a height field of 1922 faces would gain (3 x 50001 points 341 -> 76).  Large
// triangles in any number, and points near the centre of a closed surface, are
// about as far from all faces, and lose: 15 to 40% where there are many points,
// up to twice where the sort is a large part.  Measured (us, all pairs -> this):
//                        icosphere  grid       small soup  large soup  points inside
//   1.6e8 pairs, 1 item   189  58    188  78    208  84     177 354     175 328
//   1.6e8, 8 items        192  70    255  84    189  79     178 252     176 281
//   5e8, 8 items          510  89    582 101    552 130     543 690     474 675
//   1.3e9, 16 items      1270 148   1347 154   1243 192    1230 1525   1210 1370
// (soups: random triangles of the size of the cloud, or a tenth of it.)
constexpr double kMinPairs = 1.5e8;
constexpr int64_t kMinPoints = 1024, kMinFaces = 2048;
constexpr size_t kMaxTreeBytes = size_t{4} << 30;
constexpr uint32_t kQueue = 192;    // leaves queued at most
constexpr uint32_t kFull = kQueue - kWave;
// Waves per leaf of points: one, or four where the points fill only about half of
// the chip's wave slots.  Measured (us, all pairs, one wave, four): 1 x 8000
// points against 20000 faces (small triangles) 208 128 84, large triangles 198 837
// 379; 8 x 2777 against 7200 (height fields) 255 119 83; 1 x 22222 188 86 78; but 1 x
// 31250 against 5120 (icospheres) 189 57 77.
constexpr int64_t kFewPoints = 28000;
constexpr int kSplitWaves = 4;
constexpr int kThreads = 256;

// A face's centroid, to sort by (vertex 0 for a face with a vertex index out
// of range, 0 for a NaN: such a face may have an edge without one).
__global__ __launch_bounds__(kThreads) void centroid_kernel(int64_t B, int64_t nv, int64_t nf,
                                                            const float *V, const int32_t *F, float *C)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (k >= B * nf) return;
    const int32_t t[3] = {F[3 * k], F[3 * k + 1], F[3 * k + 2]};
    const bool ok = face_ok_nb(t, nv);
    const float *Vb = V + k / nf * nv * 3;
    float v[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < 3; ++i) v[j][i] = Vb[3 * static_cast<int64_t>(ok ? t[j] : 0) + i];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float c = v[0][i] * (1.0f / 3.0f) + v[1][i] * (1.0f / 3.0f) + v[2][i] * (1.0f / 3.0f);
        C[3 * k + i] = c == c ? c : 0.0f;
    }
}

// One node of sorted faces per workgroup, a face per thread: records (eight
// float4 per face, the 16 faces of a leaf side by side; the last float holds the
// face's index) and the boxes of leaves and node.  Box words 3 and 7: margins.
__global__ __launch_bounds__(kNode) void face_leaf_kernel(int64_t nv, int64_t nf, int nodes,
                                                          const float *V, const int32_t *F,
                                                          const float4 *sorted, Box *leaf, Box *node,
                                                          float4 *rec)
{
    __shared__ float part[kNodeLeaves][8];
    const int64_t nd = blockIdx.x, b = nd / nodes;
    const uint32_t lf = threadIdx.x / kLeaf, sub = threadIdx.x % kLeaf;
    const bool empty = !(leaf[nd * kNodeLeaves + lf].lx <= leaf[nd * kNodeLeaves + lf].hx);
    // (Read from the workspace: bounded before it is an address.)
    const uint32_t id = empty ? kNoPoint : __float_as_uint(sorted[nd * kNode + threadIdx.x].w);
    const bool face = id < static_cast<uint32_t>(nf);
    const int32_t *t3 = F + (b * nf + (face ? id : 0u)) * 3;
    const int32_t t[3] = {t3[0], t3[1], t3[2]};
    const bool ok = face && face_ok_nb(t, nv);
    const float *Vb = V + b * nv * 3;
    double A[3], Bv[3], C[3];
    float lo[3], hi[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float x = Vb[3 * static_cast<int64_t>(ok ? t[0] : 0) + i];
        const float y = Vb[3 * static_cast<int64_t>(ok ? t[1] : 0) + i];
        const float z = Vb[3 * static_cast<int64_t>(ok ? t[2] : 0) + i];
        A[i] = x;
        Bv[i] = y;
        C[i] = z;
        lo[i] = ok ? fminf(x, fminf(y, z)) : __builtin_inff();
        hi[i] = ok ? fmaxf(x, fmaxf(y, z)) : -__builtin_inff();
    }
    float r[kRec];
    double spread = 0.0;
    if (ok)
        spread = face_record(A, Bv, C, r);
    else
        far_record(r);
    r[31] = __uint_as_float(ok ? id : kNoPoint);
    // Relative margin of this face's computed distances.
    float m = ok ? static_cast<float>((64.0 + 32.0 * spread) * 0x1p-24) : 0.0f;
    if (!(m < 0.5f)) m = __builtin_inff();
    if (!empty) {
        float4 *out = rec + (nd * kNodeLeaves + lf) * (8 * kLeaf) + sub;
#pragma unroll
        for (int c = 0; c < 8; ++c)
            out[c * kLeaf] = make_float4(r[4 * c], r[4 * c + 1], r[4 * c + 2], r[4 * c + 3]);
    }
    float v[7] = {-lo[0], -lo[1], -lo[2], hi[0], hi[1], hi[2], m};
#pragma unroll
    for (int c = 0; c < 7; ++c) v[c] = row_max(v[c]);
    const float dx = v[3] + v[0], dy = v[4] + v[1], dz = v[5] + v[2];
    // (An empty leaf: no margin, box empty.)
    const float md = v[3] >= -v[0] ? v[6] * sqrtf(sum_sq(dx, dy, dz)) * 1.001f : 0.0f;
    __syncthreads();
    if (sub == 0) {
        leaf[nd * kNodeLeaves + lf] = Box{-v[0], -v[1], -v[2], __float_as_uint(v[6]),
                                          v[3], v[4], v[5], __float_as_uint(md)};
#pragma unroll
        for (int c = 0; c < 7; ++c) part[lf][c] = v[c];
        part[lf][7] = md;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        float w[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) w[c] = wave_max(part[threadIdx.x][c]);
        if (threadIdx.x == 0)
            node[nd] = Box{-w[0], -w[1], -w[2], __float_as_uint(w[6]), w[3], w[4], w[5],
                           __float_as_uint(w[7])};
    }
}

struct SearchArgs {
    const float4 *points, *pleaf;       // sorted points and their leaves' boxes
    const float4 *rec, *leaf, *node;    // sorted faces
    float *dist;
    int32_t *fidx;
    SortShape p, f;
};

// Whether a computed distance from within the box [qlo, qhi] to a face of the
// box (lo, hi) can be at most `worst`.
__device__ __forceinline__ bool reaches(const float4 &qlo, const float4 &qhi, const float4 &lo,
                                        const float4 &hi, float worst)
{
    const float d = __builtin_amdgcn_sqrtf(bound(qlo, qhi, lo, hi));
    const float t = fmaxf(__builtin_fmaf(-lo.w, d, d) - hi.w, 0.0f);   // (NaN: 0)
    return lo.x <= hi.x && !(__builtin_fmaf(t, t * (1.0f - 0x1p-20f), -1e-37f) > worst);
}

// A leaf of points per workgroup; each of its kWaves waves takes a share of the
// leaves of faces.
template <int kWaves>
__global__ __launch_bounds__(kWaves * kWave) __attribute__((amdgpu_waves_per_eu(3, 8)))
void face_search_kernel(SearchArgs a)
{
    __shared__ uint32_t queues[kWaves][kQueue];
    __shared__ double part[kWaves][kLeaf];
    const uint32_t lane = threadIdx.x % kWave, sub = lane & 15u, row = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t *queue = queues[wave];
    const uint32_t n = xcd_block();
    const uint32_t tiles = a.p.nodes * kNodeLeaves;
    const int64_t b = n / tiles;
    const float4 *pl = a.pleaf + static_cast<int64_t>(n) * 2;
    const float4 qlo = pl[0], qhi = pl[1];
    Targets t;
    t.leaf = a.leaf + b * a.f.nodes * kNodeLeaves * 2;
    t.node = a.node + b * a.f.nodes * 2;
    t.nodes = a.f.nodes;
    const float4 *rec = a.rec + b * a.f.nodes * kNode * 8;
    const uint32_t n0 = min(lane, t.nodes - 1);
    const float4 nlo = t.node[2 * n0], nhi = t.node[2 * n0 + 1];
    const float4 q = a.points[static_cast<int64_t>(n) * kLeaf + sub];
    const uint32_t np = static_cast<uint32_t>(a.p.n), nf = static_cast<uint32_t>(a.f.n);
    if (nan_query(q, qhi) && threadIdx.x < kLeaf && __float_as_uint(q.z) < np) {   // no face is near it
        a.dist[b * np + __float_as_uint(q.z)] = __builtin_inff();
        a.fidx[b * np + __float_as_uint(q.z)] = -1;
    }
    if (!(qlo.x <= qhi.x)) return;
    const uint32_t id = __float_as_uint(q.w);
    const uint32_t active = static_cast<uint32_t>(__ballot(id != kNoPoint)) & 0xffffu;

    float px[kLeaf], py[kLeaf], pz[kLeaf];
    double best[kLeaf];
#pragma unroll
    for (int i = 0; i < kLeaf; ++i) {
        px[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.x), i));
        py[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.y), i));
        pz[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.z), i));
        best[i] = pack(__builtin_inff(), kNoPoint);
    }
    float mine = __builtin_inff(), worst = __builtin_inff();   // bounds of query `sub`, of all
    // Each row a leaf, a face per lane, against the queries of `mask`.
    const auto visit = [&](uint32_t leaf, uint32_t mask) __attribute__((always_inline)) {
        float4 R[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) R[c] = rec[(leaf * 8u + c) * kLeaf + sub];
#pragma unroll
        for (int i = 0; i < kLeaf; ++i) {
            if ((mask >> i & 1u) == 0u) continue;
            const float d = __builtin_fminf(face_dist(px[i], py[i], pz[i], R), __builtin_inff());
            best[i] = min_key(best[i], pack(d, __float_as_uint(R[7].w)));
        }
    };
    const auto settle = [&]() __attribute__((always_inline)) {
        uint32_t w = 0u;
#pragma unroll
        for (int i = 0; i < kLeaf; ++i) {
            const uint32_t v = row_min_u32(__float_as_uint(high(best[i])));
            w = sub == static_cast<uint32_t>(i) ? v : w;
        }
        const auto r16 = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        w = min(r16[0], r16[1]);
        const auto r32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
        mine = id != kNoPoint ? __uint_as_float(min(r32[0], r32[1])) : -1.0f;
        worst = row_max(mine);
    };
    uint32_t done[4];
    nearest_leaves(t, qlo, qhi, nlo, nhi, lane, done);
    if (lane < 4u)
        queue[lane] = done[0] == kNoPoint ? 0u : lane == 0u ? done[0] : lane == 1u ? done[1]
                      : lane == 2u        ? done[2] : done[3];
    uint32_t queued = done[0] != kNoPoint ? 4u : 0u;
    const auto drain = [&]() __attribute__((always_inline)) {
        wave_sync();
        for (uint32_t c = 0u; c < queued; c += 4u) {
            const uint32_t leaf = queue[min(c + row, queued - 1u)];
            const float4 lo = t.leaf[leaf * 2], hi = t.leaf[leaf * 2 + 1];
            const uint64_t need = __ballot(reaches(q, q, lo, hi, mine));
            const uint32_t both = static_cast<uint32_t>(need) | static_cast<uint32_t>(need >> 32);
            const uint32_t mask = (both | both >> 16) & active;
            if (mask == 0u) continue;
            visit(leaf, mask);
            settle();
        }
        queued = 0u;
        wave_sync();
        return true;
    };
    for (bool first = true;; first = false) {
        drain();
        if (!first) break;
        gather(t, nlo, nhi, lane, done, queue, queued, kFull, lane % kWaves == wave,
               [&](const float4 &lo, const float4 &hi) { return reaches(qlo, qhi, lo, hi, worst); }, drain);
    }
    double out = 0.0;
#pragma unroll
    for (int i = 0; i < kLeaf; ++i) {
        double k = best[i];
        k = min_key(k, dpp_key<0xB1>(k));
        k = min_key(k, dpp_key<0x4E>(k));
        k = min_key(k, dpp_key<0x141>(k));
        k = min_key(k, dpp_key<0x140>(k));
        out = sub == static_cast<uint32_t>(i) ? k : out;
    }
    out = rows_min(out);
    if (kWaves > 1) {
        if (row == 0u) part[wave][sub] = out;
        __syncthreads();
        if (wave > 0u) return;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) out = min_key(out, part[w][sub]);
    }
    if (id < np && row == 0u) {
        const int64_t o = b * np + id;
        const uint32_t face = static_cast<uint32_t>(__double2loint(out));
        a.dist[o] = high(out);
        // As all pairs: a face whose distance overflows is not chosen.
        a.fidx[o] = high(out) < __builtin_inff() && face < nf ? static_cast<int32_t>(face) : -1;
    }
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct TreeLayout {
    SortPlan points, faces;
    size_t centroids, rec, bytes;
};

TreeLayout layout(int64_t B, int64_t S, int64_t nf)
{
    TreeLayout l{};
    size_t at = 0;
    l.points = plan_sort(B, S, at);
    l.faces = plan_sort(B, nf, at);
    l.centroids = at;
    at += align256(static_cast<size_t>(B) * nf * 12);
    l.rec = at;
    at += align256(static_cast<size_t>(B) * l.faces.s.nodes * kNode * kRec * 4);
    l.bytes = at;
    return l;
}

}  // namespace

size_t p2s_tree_bytes(int64_t B, int64_t S, int64_t nf)
{
    if (static_cast<double>(B) * S * nf < kMinPairs || S < kMinPoints || nf < kMinFaces ||
        std::max(S, nf) > kSortMaxPoints)
        return 0;
    const size_t bytes = layout(B, S, nf).bytes;
    return bytes <= kMaxTreeBytes ? bytes : 0;
}

hipError_t launch_p2s_tree(int64_t B, int64_t S, int64_t nv, int64_t nf, const float *P,
                           const float *V, const int32_t *F, float *dist, int32_t *fidx, void *ws,
                           hipStream_t stream)
{
    const TreeLayout l = layout(B, S, nf);
    char *base = static_cast<char *>(ws);
    float *centroids = reinterpret_cast<float *>(base + l.centroids);
    centroid_kernel<<<static_cast<uint32_t>((B * nf + kThreads - 1) / kThreads), kThreads, 0, stream>>>(
        B, nv, nf, V, F, centroids);
    const SortJob pj = sort_job(l.points, P, base), fj = sort_job(l.faces, centroids, base);
    const hipError_t e = launch_sort(B, pj, fj, nullptr, 0u, stream);
    if (e != hipSuccess) return e;
    float4 *rec = reinterpret_cast<float4 *>(base + l.rec);
    face_leaf_kernel<<<static_cast<uint32_t>(B * fj.s.nodes), kNode, 0, stream>>>(
        nv, nf, fj.s.nodes, V, F, fj.rec, fj.leaf, fj.node, rec);
    SearchArgs a{};
    a.points = pj.rec;
    a.pleaf = reinterpret_cast<const float4 *>(pj.leaf);
    a.rec = rec;
    a.leaf = reinterpret_cast<const float4 *>(fj.leaf);
    a.node = reinterpret_cast<const float4 *>(fj.node);
    a.dist = dist;
    a.fidx = fidx;
    a.p = pj.s;
    a.f = fj.s;
    const uint32_t leaves = static_cast<uint32_t>(B * pj.s.nodes * kNodeLeaves);
    if (B * S < kFewPoints)
        face_search_kernel<kSplitWaves><<<leaves, kSplitWaves * kWave, 0, stream>>>(a);
    else
        face_search_kernel<1><<<leaves, kWave, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace cdk
