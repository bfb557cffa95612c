// Approximate Earth-mover's distance between point clouds (Kaolin Sec. 2.5
// names an approximate EMD among its point-cloud metrics, citing Fan et al.): the optimal
// transport problem with uniform masses a = 1/N, b = 1/M and Euclidean cost
// C_ij = |x_i - y_j|, regularised by entropy and solved with log-domain
// Sinkhorn iterations, each touching all N*M pairs.  With a scheduled eps:
//     f_i <- -eps log sum_j b exp((g_j - C_ij) / eps)
//     g_j <- -eps log sum_i a exp((f_i - C_ij) / eps)
// and the plan P_ij = a b exp((f_i + g_j - C_ij) / eps), the cost is
// sum_ij P_ij C_ij; its backward holds P fixed:
//     d cost / d x_i = sum_j P_ij (x_i - y_j) / C_ij,  d cost / d y_j = the opposite sum.
//
//  * lse_kernel: one half-update.  A workgroup of 16 waves holds 64, 128 or 256
//    queries (1, 2 or 4 per lane, the same in every wave) in VGPRs; each wave
//    walks a sixteenth of the targets, whose index is wave-uniform, so that
//    coordinates and scaled potential (one float4, written by the half-update
//    before) arrive by scalar loads.  The log-sum-exp runs in base 2 online over
//    batches of targets: the batch maximum rescales the running sum once, then
//    each pair adds exp2(z - max), z = (g_j - C_ij) log2(e) / eps.  The waves'
//    (max, sum) meet in LDS and the finished potentials are written, so that a
//    half-update is one launch and leaves no partials.  Queries per lane: as
//    many as leave one workgroup per CU; up to 64 targets take 4 waves, since more
//    would be idle.  Where one query per lane still leaves CUs idle (few queries,
//    many targets), the targets are split over workgroups too, and
//    lse_merge_kernel finishes the potentials.  Per half-update (us; all targets
//    split over workgroups and merged by every query group of the next
//    half-update -> no split -> this):
//      32 x 2048^2      60.0  56.9  57.4      1 x 64 x 100000    127   347  19.6
//      2 x 500 x 701    14.0   7.0   7.1      1 x 512 x 100000   193   362  36.8
//      4 x 300 x 3000   20.5  15.0   6.4      1 x 4096^2        36.7  31.1  12.8
//      1 x 3000 x 30000  110   130  51.3      1 x 8192^2        51.8  60.2  35.0
//      1000 x 5 x 7     10.6  10.8   4.0      100000 x 10^2      949  1295   238
//    Bound by instruction issue: 12 instructions a term, two of them
//    transcendental at about 9 cycles each, 62 cycles per 64 terms.  Measured and
//    not kept: targets through LDS (6315 against 5420 us for the 50 iterations
//    of 32 x 2048^2), scalar loads a batch ahead (5693: the compiler moves them to
//    VGPRs), 8 waves (5623), 8 or fewer targets a batch with fewer queries.
//  * plan_kernel: per (query block, target block) tile, either the tile's
//    sum of P_ij C_ij (in double, reduced in a fixed order) or per query
//    the sum of P_ij (q_i - t_j) / C_ij; partial sums over target blocks are
//    added in order by cost_reduce_kernel / grad_merge_kernel.
// Square roots and exponentials use the hardware approximations (v_sqrt_f32,
// v_rsq_f32, v_exp_f32).  Exponents are bounded: after each half-update the
// updated side's sums equal its mass, so every a b exp(z) is at most 1.
#include <algorithm>
#include <cmath>

#include "cd_internal.h"

namespace cdk {
namespace {

constexpr int kEQ = 4;                      // queries per lane
constexpr int kEThreads = 256;              // 4 waves
constexpr int kEGroup = kEQ * kEThreads;    // queries per workgroup
constexpr int kEBatch = 16;                 // targets per batch of a plan pass
constexpr int kEMinTB = 64;                 // targets per block, at least
constexpr int64_t kETargetTiles = 512;
constexpr int kLseWaves = 16;               // waves of a half-update's workgroup
// Workgroups of a launch at most: with 2^22 of 1024 threads, 2^32 threads, only
// some of them run.  (A loop over groups in the kernel: 7.0 -> 8.0 us a
// half-update of 2 x 500 x 701.)
constexpr int64_t kLseGrid = 1 << 21;
constexpr int64_t kPlanGrid = 1 << 23;      // the same for workgroups of 256 threads
constexpr int kLseFew = 4;                  // waves where the targets are few
constexpr int kLseStep = 16;                // targets per wave: a multiple
constexpr int kSplitGain = 64;              // targets per wave that a split has to save
constexpr int kMergeAhead = 16;             // partials loaded together by a merge
constexpr int64_t kCUs = 256;
constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

struct LseArgs {
    const float *Q;         // [B, nq, 3]
    const float4 *T;        // [B, nt] targets: coordinates, potential times k
    float4 *Q4;             // [B, nq] the queries as targets of the next half-update
    float *pq;              // [B, nq] updated potentials of the queries
    int64_t nq, nt;
    float k;                // log2(e) / eps
    float k_next;           // that of the next half-update
    float2 *part;           // [B, nTB, nq] (max, sum) per target block (nTB > 1)
    float out_scale;        // -eps ln 2
    float out_bias;         // eps log(nt)  (= -eps log b)
    int nQG, per;           // query groups per item; targets per wave
    int nTB, TB;            // target blocks; targets per block
    uint32_t first;         // query group of the launch's first workgroup
};

__device__ __forceinline__ float dist2(float qx, float qy, float qz, float tx, float ty, float tz)
{
    const float dx = qx - tx, dy = qy - ty, dz = qz - tz;
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

// One batch of kB targets for kQ queries: running max m and sum s.  The batch
// is summed by itself, so that no sum has more terms than a batch or than a wave
// has batches: one by one, terms below 2^-24 of the running sum would be lost.
template <int kQ, int kB>
__device__ __forceinline__ void lse_batch(const float (&qx)[kQ], const float (&qy)[kQ],
                                          const float (&qz)[kQ], float (&m)[kQ], float (&s)[kQ],
                                          const float4 (&t)[kB], float kk)
{
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        float z[kB];
        float bm = -__builtin_inff();
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const float c = __builtin_amdgcn_sqrtf(dist2(qx[k], qy[k], qz[k], t[u].x, t[u].y, t[u].z));
            z[u] = __builtin_fmaf(-c, kk, t[u].w);
            bm = __builtin_fmaxf(bm, z[u]);
        }
        const float mn = __builtin_fmaxf(m[k], bm);
        // (An FMA at the end in place of the product here: 57 -> 60 us a
        // half-update of 32 x 2048^2, in every order of the terms.)
        const float before = s[k] * __builtin_amdgcn_exp2f(m[k] - mn);
        float acc = 0.0f;
#pragma unroll
        for (int u = 0; u < kB; ++u) acc += __builtin_amdgcn_exp2f(z[u] - mn);
        s[k] = before + acc;
        m[k] = mn;
    }
}

// -eps log(b sum exp(...)) of a query from its (max, sum), M and S.
__device__ __forceinline__ void finish(const LseArgs &a, int64_t at, float M, float S)
{
    const float pot = __builtin_fmaf(a.out_scale, M + __log2f(S), a.out_bias);
    a.pq[at] = pot;
    a.Q4[at].w = pot * a.k_next;
}

// kSplit: the workgroup's targets are one block of nTB, and it leaves (max, sum).
template <int kQ, int kB, int kWaves, bool kSplit>
__global__ __launch_bounds__(kWaves * kWave) void lse_kernel(LseArgs a)
{
    __shared__ float2 part[kWaves][kQ * kWave];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const uint32_t tile = a.first + blockIdx.x;
    const uint32_t tb = kSplit ? tile % static_cast<uint32_t>(a.nTB) : 0u;
    const uint32_t group = kSplit ? tile / static_cast<uint32_t>(a.nTB) : tile;
    const int64_t b = group / static_cast<uint32_t>(a.nQG);
    const int64_t q0 = static_cast<int64_t>(group % static_cast<uint32_t>(a.nQG)) * (kQ * kWave);
    float qx[kQ], qy[kQ], qz[kQ], m[kQ], s[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        const int64_t q = std::min<int64_t>(q0 + k * kWave + lane, a.nq - 1);
        const float *p = a.Q + (b * a.nq + q) * 3;
        qx[k] = p[0];
        qy[k] = p[1];
        qz[k] = p[2];
        m[k] = -__builtin_inff();
        s[k] = 0.0f;
    }
    // This wave's targets; the index is the same for all its lanes, so that
    // they arrive by scalar loads.
    const float4 *Tb = a.T + b * a.nt;
    const float kk = a.k;
    const int t0 = kSplit ? static_cast<int>(tb) * a.TB : 0;
    const int nt = kSplit ? static_cast<int>(std::min<int64_t>(static_cast<int64_t>(t0) + a.TB, a.nt))
                          : static_cast<int>(a.nt);
    int j = __builtin_amdgcn_readfirstlane(
        static_cast<int>(std::min<int64_t>(t0 + static_cast<int64_t>(wave) * a.per, nt)));
    const int j1 = static_cast<int>(std::min<int64_t>(static_cast<int64_t>(j) + a.per, nt));
    for (; j + kB <= j1; j += kB) {
        float4 t[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) t[u] = Tb[j + u];
        lse_batch<kQ, kB>(qx, qy, qz, m, s, t, kk);
    }
    if (j < j1) {
        // The tail: clamped loads, weight 0 past the end.
        float4 t[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            t[u] = Tb[std::min(j + u, j1 - 1)];
            t[u].w = j + u < j1 ? t[u].w : -__builtin_inff();
        }
        lse_batch<kQ, kB>(qx, qy, qz, m, s, t, kk);
    }
#pragma unroll
    for (int k = 0; k < kQ; ++k) part[wave][k * kWave + lane] = make_float2(m[k], s[k]);
    __syncthreads();
    // A thread merges one query's (max, sum) of all waves, in order.
    const int64_t q = q0 + threadIdx.x;
    if (threadIdx.x >= kQ * kWave || q >= a.nq) return;
    float2 v[kWaves];
    float M = -__builtin_inff(), S = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        v[w] = part[w][threadIdx.x];
        M = __builtin_fmaxf(M, v[w].x);
    }
#pragma unroll
    for (int w = 0; w < kWaves; ++w) S += v[w].y * __builtin_amdgcn_exp2f(v[w].x - M);
    if (kSplit)
        a.part[(b * a.nTB + tb) * a.nq + q] = make_float2(M, S);
    else
        finish(a, b * a.nq + q, M, S);
}

// Potentials from the target blocks' (max, sum), in order.
__global__ __launch_bounds__(kWave) void lse_merge_kernel(LseArgs a, int64_t B)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kWave + threadIdx.x;
    if (k >= B * a.nq) return;
    const int64_t b = k / a.nq, q = k - b * a.nq;
    const float2 *p = a.part + b * a.nTB * a.nq + q;
    float M = -__builtin_inff(), S = 0.0f;
    for (int t0 = 0; t0 < a.nTB; t0 += kMergeAhead) {
        // (A block past the last repeats it with weight 0.)
        float2 v[kMergeAhead];
        float m = M;
#pragma unroll
        for (int u = 0; u < kMergeAhead; ++u) {
            v[u] = p[std::min(t0 + u, a.nTB - 1) * a.nq];
            v[u].y = t0 + u < a.nTB ? v[u].y : 0.0f;
            m = __builtin_fmaxf(m, v[u].x);
        }
        S *= __builtin_amdgcn_exp2f(M - m);
#pragma unroll
        for (int u = 0; u < kMergeAhead; ++u) S += v[u].y * __builtin_amdgcn_exp2f(v[u].x - m);
        M = m;
    }
    finish(a, k, M, S);
}

// Both clouds as targets; the y's with their starting potential g (nullptr: 0).
__global__ __launch_bounds__(kThreads) void targets_kernel(int64_t nx, int64_t ny, const float *X,
                                                           const float *Y, const float *g, float k,
                                                           float4 *X4, float4 *Y4)
{
    int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= nx + ny) return;
    const bool y = i >= nx;
    i -= y ? nx : 0;
    const float *p = (y ? Y : X) + 3 * i;
    (y ? Y4 : X4)[i] = make_float4(p[0], p[1], p[2], y && g ? g[i] * k : 0.0f);
}

struct PlanArgs {
    const float *Q, *T;     // [B, nq, 3], [B, nt, 3]
    const float *pq, *pt;   // potentials of queries and targets
    const float *go;        // [B] (gradient mode)
    double *cost_part;      // [B, nQG, nTB] (cost mode)
    float *grad_part;       // [B, nTB, nq, 3] (gradient mode, nTB > 1)
    float *grad;            // [B, nq, 3] (gradient mode, nTB == 1)
    int64_t nq, nt;
    float k;                // log2(e) / eps
    float mass;             // a b = 1 / (nq nt)
    int nQG, nTB, TB;
    uint32_t first;         // tile of the launch's first workgroup
};

template <bool kGrad>
__device__ __forceinline__ void plan_batch(const float (&qx)[kEQ], const float (&qy)[kEQ],
                                           const float (&qz)[kEQ], const float (&qk)[kEQ],
                                           float (&acc)[kEQ], float (&gx)[kEQ], float (&gy)[kEQ],
                                           float (&gz)[kEQ], const float (&tx)[kEBatch],
                                           const float (&ty)[kEBatch], const float (&tz)[kEBatch],
                                           const float (&tk)[kEBatch], float kk)
{
#pragma unroll
    for (int u = 0; u < kEBatch; ++u) {
#pragma unroll
        for (int k = 0; k < kEQ; ++k) {
            const float d2 = dist2(qx[k], qy[k], qz[k], tx[u], ty[u], tz[u]);
            const float r = d2 > 0.0f ? __builtin_amdgcn_rsqf(d2) : 0.0f;
            const float c = d2 * r;
            const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(-c, kk, qk[k] + tk[u]));
            if (kGrad) {
                const float wr = w * r;
                gx[k] = __builtin_fmaf(wr, qx[k] - tx[u], gx[k]);
                gy[k] = __builtin_fmaf(wr, qy[k] - ty[u], gy[k]);
                gz[k] = __builtin_fmaf(wr, qz[k] - tz[u], gz[k]);
            } else {
                acc[k] = __builtin_fmaf(w, c, acc[k]);
            }
        }
    }
}

template <bool kGrad>
__global__ __launch_bounds__(kEThreads) void plan_kernel(PlanArgs a)
{
    __shared__ double red[kEThreads / kWave];
    const int64_t per_item = static_cast<int64_t>(a.nQG) * a.nTB, tile = a.first + blockIdx.x;
    const int64_t b = tile / per_item;
    const int rest = static_cast<int>(tile % per_item);
    const int qg = rest / a.nTB, tb = rest % a.nTB;
    const int64_t q0 = static_cast<int64_t>(qg) * kEGroup;
    float qx[kEQ], qy[kEQ], qz[kEQ], qk[kEQ], acc[kEQ], gx[kEQ], gy[kEQ], gz[kEQ];
#pragma unroll
    for (int k = 0; k < kEQ; ++k) {
        const int64_t q = q0 + k * kEThreads + threadIdx.x;
        const bool in = q < a.nq;
        const int64_t qc = in ? q : 0;
        const float *p = a.Q + (b * a.nq + qc) * 3;
        qx[k] = p[0];
        qy[k] = p[1];
        qz[k] = p[2];
        qk[k] = in ? a.pq[b * a.nq + qc] * a.k : -__builtin_inff();   // outside: weight 0
        acc[k] = gx[k] = gy[k] = gz[k] = 0.0f;
    }
    const int j0 = tb * a.TB;
    const int j1 = static_cast<int>(std::min<int64_t>(static_cast<int64_t>(j0) + a.TB, a.nt));
    const int jfull = j0 + (j1 - j0) / kEBatch * kEBatch;
    const float *Tb = a.T + b * a.nt * 3;
    const float *pb = a.pt + b * a.nt;
    const float kk = a.k;
    for (int jb = j0; jb < jfull; jb += kEBatch) {
        float tx[kEBatch], ty[kEBatch], tz[kEBatch], tk[kEBatch];
#pragma unroll
        for (int u = 0; u < kEBatch; ++u) {
            tx[u] = Tb[3 * (jb + u) + 0];
            ty[u] = Tb[3 * (jb + u) + 1];
            tz[u] = Tb[3 * (jb + u) + 2];
            tk[u] = pb[jb + u] * kk;
        }
        plan_batch<kGrad>(qx, qy, qz, qk, acc, gx, gy, gz, tx, ty, tz, tk, kk);
    }
    if (jfull < j1) {
        float tx[kEBatch], ty[kEBatch], tz[kEBatch], tk[kEBatch];
#pragma unroll
        for (int u = 0; u < kEBatch; ++u) {
            const int j = std::min(jfull + u, j1 - 1);
            tx[u] = Tb[3 * j + 0];
            ty[u] = Tb[3 * j + 1];
            tz[u] = Tb[3 * j + 2];
            tk[u] = jfull + u < j1 ? pb[j] * kk : -__builtin_inff();
        }
        plan_batch<kGrad>(qx, qy, qz, qk, acc, gx, gy, gz, tx, ty, tz, tk, kk);
    }
    if (kGrad) {
        const float sc = a.mass * a.go[b];
#pragma unroll
        for (int k = 0; k < kEQ; ++k) {
            const int64_t q = q0 + k * kEThreads + threadIdx.x;
            if (q >= a.nq) continue;
            float *dst = a.nTB == 1 ? a.grad + (b * a.nq + q) * 3
                                    : a.grad_part + ((b * a.nTB + tb) * a.nq + q) * 3;
            const float sv = a.nTB == 1 ? sc : 1.0f;
            dst[0] = sv * gx[k];
            dst[1] = sv * gy[k];
            dst[2] = sv * gz[k];
        }
        return;
    }
    // Cost mode: the tile's sum, reduced in a fixed order.
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kEQ; ++k) t += static_cast<double>(acc[k]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, kWave);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int w = 0; w < kEThreads / kWave; ++w) sum += red[w];
        a.cost_part[(b * a.nQG + qg) * a.nTB + tb] = sum;
    }
}

__global__ __launch_bounds__(kThreads) void cost_reduce_kernel(const double *part, int64_t tiles,
                                                               float mass, int64_t first, float *cost)
{
    __shared__ double red[kThreads / kWave];
    const int64_t b = first + blockIdx.x;
    double t = 0.0;
    for (int64_t i = threadIdx.x; i < tiles; i += kThreads) t += part[b * tiles + i];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, kWave);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kThreads / kWave; ++w) s += red[w];
        cost[b] = static_cast<float>(s * static_cast<double>(mass));
    }
}

__global__ __launch_bounds__(kThreads) void grad_merge_kernel(PlanArgs a, int64_t B)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (k >= B * a.nq * 3) return;
    const int64_t b = k / (a.nq * 3), e = k - b * a.nq * 3;
    const float *p = a.grad_part + b * a.nTB * a.nq * 3 + e;
    float s = 0.0f;
    for (int t = 0; t < a.nTB; ++t) s += p[static_cast<int64_t>(t) * a.nq * 3];
    a.grad[k] = s * (a.mass * a.go[b]);
}

int64_t ceil_div(int64_t x, int64_t y) { return (x + y - 1) / y; }

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Query groups and target blocks for queries of size nq against nt targets.
struct Tiles {
    int nQG, nTB, TB;
};

Tiles tiles_for(int64_t B, int64_t nq, int64_t nt)
{
    Tiles t;
    t.nQG = static_cast<int>(ceil_div(nq, kEGroup));
    int64_t want = std::max<int64_t>(1, ceil_div(kETargetTiles, B * t.nQG));
    want = std::min(want, std::max<int64_t>(1, ceil_div(nt, kEMinTB)));
    const int64_t tb = ceil_div(ceil_div(nt, want), kEBatch) * kEBatch;
    t.TB = static_cast<int>(tb);
    t.nTB = static_cast<int>(ceil_div(nt, tb));
    return t;
}

// How a half-update is split.
struct LseSplit {
    int q;          // queries per lane
    bool few;       // kLseFew waves a workgroup, not kLseWaves
    int nQG;        // query groups per item
    int nTB, TB;    // target blocks; targets per block
    int per;        // targets per wave
};

// Queries per lane: as many as leave one workgroup per CU and as the item has.
// Few waves: where more would have no targets.  Target blocks: where even one
// query per lane leaves CUs idle, as many as fill them, if the targets that this
// takes from a wave (0.1 us each: four waves on a SIMD, 62 cycles a target) are
// worth the merge's launch (about 5 us).
LseSplit split_for(int64_t B, int64_t nq, int64_t nt)
{
    LseSplit l{};
    const auto groups = [&](int q) { return B * ceil_div(nq, q * kWave); };
    l.q = nq > 2 * kWave && groups(4) >= kCUs ? 4 : nq > kWave && groups(2) >= kCUs ? 2 : 1;
    l.few = nt <= kLseFew * kLseStep;
    l.nQG = static_cast<int>(ceil_div(nq, l.q * kWave));
    const int waves = l.few ? kLseFew : kLseWaves;
    const auto per = [&](int64_t n) { return ceil_div(ceil_div(n, waves), kLseStep) * kLseStep; };
    // (None with two or four queries per lane: those leave a workgroup per CU.)
    const int64_t blocks = std::min(kCUs / groups(l.q), ceil_div(nt, waves * kLseStep));
    l.nTB = 1;
    l.TB = static_cast<int>(nt);
    if (blocks > 1 && per(nt) - per(ceil_div(nt, blocks)) >= kSplitGain) {
        l.TB = static_cast<int>(per(ceil_div(nt, blocks)) * waves);
        l.nTB = static_cast<int>(ceil_div(nt, l.TB));
    }
    l.per = static_cast<int>(per(l.TB));
    return l;
}

struct EmdLayout {
    Tiles xy, yx;               // plan passes: queries X against Y; queries Y against X
    size_t x4_bytes, y4_bytes, part_bytes, cost_bytes, grad_bytes;
};

EmdLayout layout(int64_t B, int64_t N, int64_t M)
{
    EmdLayout L;
    L.xy = tiles_for(B, N, M);
    L.yx = tiles_for(B, M, N);
    L.x4_bytes = align256(static_cast<size_t>(B * N) * sizeof(float4));
    L.y4_bytes = align256(static_cast<size_t>(B * M) * sizeof(float4));
    const auto part = [&](int64_t nq, int64_t nt) {
        const LseSplit l = split_for(B, nq, nt);
        return l.nTB > 1 ? static_cast<size_t>(B * l.nTB * nq) * sizeof(float2) : 0;
    };
    L.part_bytes = align256(std::max(part(N, M), part(M, N)));
    L.cost_bytes = align256(static_cast<size_t>(B * L.xy.nQG * L.xy.nTB) * 8);
    const size_t g1 = L.xy.nTB > 1 ? static_cast<size_t>(B * L.xy.nTB * N) * 12 : 0;
    const size_t g2 = L.yx.nTB > 1 ? static_cast<size_t>(B * L.yx.nTB * M) * 12 : 0;
    L.grad_bytes = align256(std::max(g1, g2));
    return L;
}

// (Targets are split only with one query per lane and more than 64 targets.)
void launch_lse(const LseSplit &l, uint32_t grid, const LseArgs &a, hipStream_t stream)
{
    const int waves = l.few ? kLseFew : kLseWaves;
    const auto run = [&](auto kernel) { kernel<<<grid, waves * kWave, 0, stream>>>(a); };
    if (l.nTB > 1)
        run(lse_kernel<1, 16, kLseWaves, true>);
    else if (l.q == 4)
        run(l.few ? lse_kernel<4, 8, kLseFew, false> : lse_kernel<4, 8, kLseWaves, false>);
    else if (l.q == 2)
        run(l.few ? lse_kernel<2, 16, kLseFew, false> : lse_kernel<2, 16, kLseWaves, false>);
    else
        run(l.few ? lse_kernel<1, 16, kLseFew, false> : lse_kernel<1, 16, kLseWaves, false>);
}

// One half-update of the queries' potentials.
void lse_pass(int64_t B, const float *Q, float4 *Q4, int64_t nq, const float4 *T, int64_t nt,
              float *pq, float eps, float eps_next, float2 *part, hipStream_t stream)
{
    const LseSplit l = split_for(B, nq, nt);
    LseArgs a{};
    a.Q = Q;
    a.T = T;
    a.Q4 = Q4;
    a.pq = pq;
    a.part = part;
    a.nq = nq;
    a.nt = nt;
    a.k = kLog2e / eps;
    a.k_next = kLog2e / eps_next;
    a.out_scale = -eps * 0.6931471805599453f;
    a.out_bias = static_cast<float>(static_cast<double>(eps) * std::log(static_cast<double>(nt)));
    a.per = l.per;
    a.nQG = l.nQG;
    a.nTB = l.nTB;
    a.TB = l.TB;
    const int64_t tiles = B * l.nQG * l.nTB;
    for (int64_t first = 0; first < tiles; first += kLseGrid) {
        a.first = static_cast<uint32_t>(first);
        launch_lse(l, static_cast<uint32_t>(std::min(tiles - first, kLseGrid)), a, stream);
    }
    if (l.nTB > 1)
        lse_merge_kernel<<<static_cast<uint32_t>(ceil_div(B * nq, kWave)), kWave, 0, stream>>>(a, B);
}

hipError_t plan_pass(int64_t B, const float *Q, int64_t nq, const float *T, int64_t nt,
                     const float *pq, const float *pt, float eps, const Tiles &t, bool gradient,
                     const float *go, double *cost_part, float *grad_part, float *grad,
                     hipStream_t stream)
{
    PlanArgs a{};
    a.Q = Q;
    a.T = T;
    a.pq = pq;
    a.pt = pt;
    a.go = go;
    a.cost_part = cost_part;
    a.grad_part = grad_part;
    a.grad = grad;
    a.nq = nq;
    a.nt = nt;
    a.k = kLog2e / eps;
    a.mass = static_cast<float>(1.0 / (static_cast<double>(nq) * static_cast<double>(nt)));
    a.nQG = t.nQG;
    a.nTB = t.nTB;
    a.TB = t.TB;
    const int64_t tiles = B * t.nQG * t.nTB;
    for (int64_t first = 0; first < tiles; first += kPlanGrid) {
        a.first = static_cast<uint32_t>(first);
        const uint32_t grid = static_cast<uint32_t>(std::min(tiles - first, kPlanGrid));
        if (gradient)
            plan_kernel<true><<<grid, kEThreads, 0, stream>>>(a);
        else
            plan_kernel<false><<<grid, kEThreads, 0, stream>>>(a);
    }
    if (gradient && t.nTB > 1)
        grad_merge_kernel<<<static_cast<uint32_t>(ceil_div(B * nq * 3, kThreads)), kThreads, 0,
                            stream>>>(a, B);
    return hipGetLastError();
}

}  // namespace

size_t emd_workspace_bytes(int64_t B, int64_t N, int64_t M)
{
    const EmdLayout L = layout(B, N, M);
    return L.x4_bytes + L.y4_bytes + L.part_bytes + L.cost_bytes + L.grad_bytes;
}

float emd_eps(double eps_start, double eps_end, int n_iters, int t)
{
    if (n_iters <= 1) return static_cast<float>(eps_end);
    const double e = eps_start * std::pow(eps_end / eps_start,
                                          static_cast<double>(t) / static_cast<double>(n_iters - 1));
    return static_cast<float>(e);
}

hipError_t launch_emd_forward(int64_t B, int64_t N, int64_t M, const float *X, const float *Y,
                              double eps_start, double eps_end, int n_iters, bool warm, float *f,
                              float *g, float *cost, void *ws, hipStream_t stream)
{
    const EmdLayout L = layout(B, N, M);
    char *base = static_cast<char *>(ws);
    float4 *X4 = reinterpret_cast<float4 *>(base);
    float4 *Y4 = reinterpret_cast<float4 *>(base + L.x4_bytes);
    float2 *part = reinterpret_cast<float2 *>(base + L.x4_bytes + L.y4_bytes);
    double *cost_part = reinterpret_cast<double *>(base + L.x4_bytes + L.y4_bytes + L.part_bytes);
    targets_kernel<<<static_cast<uint32_t>(ceil_div(B * (N + M), kThreads)), kThreads, 0, stream>>>(
        B * N, B * M, X, Y, warm ? g : nullptr, kLog2e / emd_eps(eps_start, eps_end, n_iters, 0), X4, Y4);
    hipError_t e;
    for (int t = 0; t < n_iters; ++t) {
        const float eps = emd_eps(eps_start, eps_end, n_iters, t);
        const float next = emd_eps(eps_start, eps_end, n_iters, std::min(t + 1, n_iters - 1));
        lse_pass(B, X, X4, N, Y4, M, f, eps, eps, part, stream);
        lse_pass(B, Y, Y4, M, X4, N, g, eps, next, part, stream);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const float eps = emd_eps(eps_start, eps_end, n_iters, n_iters - 1);
    e = plan_pass(B, X, N, Y, M, f, g, eps, L.xy, false, nullptr, cost_part, nullptr,
                             nullptr, stream);
    if (e != hipSuccess) return e;
    for (int64_t first = 0; first < B; first += kPlanGrid)
        cost_reduce_kernel<<<static_cast<uint32_t>(std::min(B - first, kPlanGrid)), kThreads, 0, stream>>>(
            cost_part, static_cast<int64_t>(L.xy.nQG) * L.xy.nTB,
            static_cast<float>(1.0 / (static_cast<double>(N) * static_cast<double>(M))), first, cost);
    return hipGetLastError();
}

hipError_t launch_emd_backward(int64_t B, int64_t N, int64_t M, const float *X, const float *Y,
                               const float *f, const float *g, double eps, const float *go,
                               float *gX, float *gY, void *ws, hipStream_t stream)
{
    const EmdLayout L = layout(B, N, M);
    char *base = static_cast<char *>(ws);
    float *grad_part = reinterpret_cast<float *>(base + L.x4_bytes + L.y4_bytes + L.part_bytes +
                                                 L.cost_bytes);
    const float e32 = static_cast<float>(eps);
    hipError_t e = plan_pass(B, X, N, Y, M, f, g, e32, L.xy, true, go, nullptr, grad_part, gX,
                             stream);
    if (e != hipSuccess) return e;
    return plan_pass(B, Y, M, X, N, g, f, e32, L.yx, true, go, nullptr, grad_part, gY, stream);
}

}  // namespace cdk
