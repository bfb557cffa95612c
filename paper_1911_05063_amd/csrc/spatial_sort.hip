// The sort of spatial_sort.h: kernels and launches.
#include "spatial_sort.h"

namespace cdk {

namespace {

constexpr int kBucketThreads = 256;
constexpr int kBucketHeld = 8;                   // points per thread
constexpr int kSortChunk = kBucketThreads * kBucketHeld;
constexpr int kSortSamples = 4 * kBucketThreads;
constexpr int kRangeLevels = 4;                  // curve levels that tell ranges apart
constexpr int kRangeCells = 1 << (3 * kRangeLevels);
constexpr int kMaxRanges = 512;                  // per cloud
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortHeld = 8;                     // points per thread kept in registers
constexpr int kOneRange = kSortHeld * kSortThreads;   // clouds up to this size: one range
constexpr int kRangePoints = 1536;               // points per range aimed at above that
constexpr int kMaxChunks = 1024;                 // per cloud (LDS segment table)
constexpr int kLogCells = 13;                    // cells per range at most: 32 KB of LDS counters
constexpr int kLevels = 10;                      // curve levels within a range
// A cell with more of a cloud's samples, or with a larger share of a range's
// points (and more of them), is crowded: the grid does not resolve the cloud.
// (From 62 samples on, mixtures of 4 x 100000 x 10000 points took the warp, which
// costs the sort about 13 us, for nothing: 177 -> 213 us.)
constexpr uint32_t kCrowdSamples = kSortSamples / 8;
constexpr uint32_t kCrowdSixteenths = 7, kCrowdPoints = 16 * kLeaf;
static_assert(static_cast<int64_t>(kMaxChunks) * kSortChunk == kSortMaxPoints, "segment table");

struct P3f {
    float x, y, z;
};

// Inclusive prefix sum over the wave in lane order.
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v)
{
    const auto step = [](uint32_t x, int moved) { return x + static_cast<uint32_t>(moved); };
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xA, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xC, 0xF, false));
    return v;
}

// Index along the Hilbert curve of a cell of the 2^kLevels cube (kLevels bits
// per axis), after Skilling, "Programming the Hilbert curve" (2004): the axes
// are turned level by level, then Gray-decoded and interleaved.  Neighbours on
// the curve are neighbours in space, which those of a Z-order curve are not at
// its jumps: the searches visit about half as many leaves.
// (kUnroll 1: a loop, for paths that few clouds take, so that they don't grow
// the usual path's code.)
template <int kLevels, int kUnroll = kLevels>
__device__ __forceinline__ uint32_t hilbert(uint32_t x, uint32_t y, uint32_t z)
{
#pragma unroll kUnroll
    for (int l = kLevels - 1; l > 0; --l) {
        const uint32_t low = (1u << l) - 1u;
        const auto bit = [&](uint32_t v) { return 0u - ((v >> l) & 1u); };   // all ones if set
        // Axis bit set: invert x's lower bits; else swap x's and the axis' lower bits.
        x ^= bit(x) & low;
        uint32_t t = (x ^ y) & low & ~bit(y);
        x ^= t ^ (bit(y) & low);
        y ^= t;
        t = (x ^ z) & low & ~bit(z);
        x ^= t ^ (bit(z) & low);
        z ^= t;
    }
    y ^= x;
    z ^= y;
    uint32_t t = 0u;
#pragma unroll kUnroll
    for (int l = kLevels - 1; l > 0; --l) t ^= ((1u << l) - 1u) & (0u - ((z >> l) & 1u));
    x ^= t;
    y ^= t;
    z ^= t;
    uint32_t code = 0u;
#pragma unroll kUnroll
    for (int l = kLevels - 1; l >= 0; --l)
        code = code << 3 | ((x >> l) & 1u) << 2 | ((y >> l) & 1u) << 1 | ((z >> l) & 1u);
    return code;
}

// A box as maxima: -lo, hi.
struct MaxBox {
    float v[6];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = -__builtin_inff();
    }
    __device__ __forceinline__ void add(float x, float y, float z)
    {
        v[0] = fmaxf(v[0], -x);
        v[1] = fmaxf(v[1], -y);
        v[2] = fmaxf(v[2], -z);
        v[3] = fmaxf(v[3], x);
        v[4] = fmaxf(v[4], y);
        v[5] = fmaxf(v[5], z);
    }
    // Over the workgroup's waves (red: one entry each); ends with a barrier.
    template <int kWaves>
    __device__ __forceinline__ void group(float (*red)[6])
    {
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            v[c] = wave_max(v[c]);
            if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave][c] = v[c];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = wave_max(red[threadIdx.x % kWaves][c]);
    }
};

// A grid of 2^kLevels cells per axis between quantiles of 64 samples: the
// points between one and the next (a sixteenth of them) share 64 equal cells.
// The outermost quantiles reach at most eight times as far as their
// neighbours; points beyond belong to border cells.  For clouds that a regular
// grid does not resolve: a few points far from all others, padding at a place of
// its own, several scales.
constexpr int kKnots = 16;
constexpr int kPerKnot = (1 << kLevels) / kKnots;

struct Warp {
    float knot[3][kKnots], scale[3][kKnots];    // lower ends of the intervals, cells per unit

    __device__ __forceinline__ uint32_t cell(int axis, float p) const
    {
        const float *k = knot[axis];
        int i = p >= k[8] ? 8 : 0;
        i += p >= k[i + 4] ? 4 : 0;
        i += p >= k[i + 2] ? 2 : 0;
        i += p >= k[i + 1] ? 1 : 0;
        return static_cast<uint32_t>(i * kPerKnot) +
               static_cast<uint32_t>(__builtin_amdgcn_fmed3f((p - k[i]) * scale[axis][i], 0.0f,
                                                             static_cast<float>(kPerKnot - 1)));
    }

    // One axis from the wave's 64 samples (one per lane; NaN: past all others).
    __device__ __forceinline__ void set(int axis, float v)
    {
        const int lane = threadIdx.x % kWave;
        v = v == v ? v : __builtin_inff();
#pragma unroll
        for (int k = 2; k <= kWave; k <<= 1)
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                const float o = __shfl_xor(v, j, kWave);
                v = ((lane & j) == 0) == ((lane & k) == 0) ? fminf(v, o) : fmaxf(v, o);
            }
        const auto at = [&](int i) { return __shfl(v, i, kWave); };
        const float least = fmaxf(at(0), at(4) - 8.0f * (at(8) - at(4)));
        const float most = fminf(at(63), at(60) + 8.0f * (at(60) - at(56)));
        const float q = __shfl(v, 4 * (lane % kKnots), kWave);
        const float next = __shfl(v, min(4 * (lane % kKnots) + 4, kWave - 1), kWave);
        const float lo = lane == 0 ? least : q, hi = lane == kKnots - 1 ? most : next;
        if (lane < kKnots) {
            const float width = hi - lo;
            knot[axis][lane] = lo;
            scale[axis][lane] = width > 0.0f ? static_cast<float>(kPerKnot) / width : 0.0f;
        }
    }
};

}  // namespace

// Curve indices in a box, 2^kLevels cells over its longest side, or in a warped
// grid, to any number of levels (fewer levels give the leading bits).  Any
// value, NaN included, gives an index.
struct Curve {
    float lo[3], scale;     // cells per unit at kLevels levels
    uint32_t warped;        // the grid is w instead
    Warp w;
    __device__ __forceinline__ void box(const MaxBox &b)
    {
        lo[0] = -b.v[0];
        lo[1] = -b.v[1];
        lo[2] = -b.v[2];
        const float ext = fmaxf(b.v[3] + b.v[0], fmaxf(b.v[4] + b.v[1], b.v[5] + b.v[2]));
        scale = ext > 0.0f ? static_cast<float>(1 << kLevels) / ext : 0.0f;
    }
};

namespace {

// A curve's box in registers; the warp stays where it is.
struct Grid {
    float lo[3], scale;
    const Warp *w;
    __device__ __forceinline__ explicit Grid(const Curve &c)
        : lo{c.lo[0], c.lo[1], c.lo[2]}, scale(c.scale), w(&c.w)
    {
    }
    template <int kTo>
    __device__ __forceinline__ uint32_t code(float x, float y, float z) const
    {
        const auto cell = [&](float p, float l) {
            return static_cast<uint32_t>(__builtin_amdgcn_fmed3f(
                       (p - l) * scale, 0.0f, static_cast<float>((1 << kLevels) - 1))) >>
                   (kLevels - kTo);
        };
        return hilbert<kTo>(cell(x, lo[0]), cell(y, lo[1]), cell(z, lo[2]));
    }
    template <int kTo>
    __device__ __forceinline__ uint32_t warped(float x, float y, float z) const
    {
        constexpr int kDown = kLevels - kTo;
        return hilbert<kTo, 1>(w->cell(0, x) >> kDown, w->cell(1, y) >> kDown, w->cell(2, z) >> kDown);
    }
};

// How a point (x, y, z, index) is stored: one with a NaN coordinate as a slot
// without a point that keeps its index aside (spatial_sort.h).
__device__ __forceinline__ float4 record(const float4 &q)
{
    const bool nan = __builtin_isnan(q.x) || __builtin_isnan(q.y) || __builtin_isnan(q.z);
    return nan ? make_float4(kFarAway, kNanMark, q.w, __uint_as_float(kNoPoint)) : q;
}

// Exclusive prefix sums over kPer kWave counters per wave of a workgroup of
// kWaves waves, in place (all threads; total: one entry per wave); returns the
// sum of all.  Starts and ends with a barrier.
template <int kWaves, int kPer>
__device__ __forceinline__ uint32_t scan_counters(uint32_t *cells, uint32_t *total)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint32_t *mine = cells + wave * kPer * kWave + lane;
    __syncthreads();
    uint32_t v[kPer], carry = 0u;
#pragma unroll
    for (int k = 0; k < kPer; ++k) v[k] = mine[k * kWave];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t incl = wave_scan_u32(v[k]);
        v[k] = carry + incl - v[k];
        carry += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (lane == 0) total[wave] = carry;
    __syncthreads();
    uint32_t before = 0u, all = 0u;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const uint32_t t = total[k];
        before += k < wave ? t : 0u;
        all += t;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) mine[k * kWave] = v[k] + before;
    __syncthreads();
    return all;
}

template <int kWaves>
__device__ __forceinline__ uint32_t scan_counters(uint32_t *cells, int n, uint32_t *total)
{
    constexpr int kGroup = kWaves * kWave;
    if (n <= kGroup) return scan_counters<kWaves, 1>(cells, total);
    if (n <= 2 * kGroup) return scan_counters<kWaves, 2>(cells, total);
    if (n <= 4 * kGroup) return scan_counters<kWaves, 4>(cells, total);
    if (n <= 8 * kGroup) return scan_counters<kWaves, 8>(cells, total);
    return scan_counters<kWaves, 16>(cells, total);
}

// Where sample k of kSortSamples is in a cloud that ends with point `last`.
__device__ __forceinline__ uint64_t sample_at(int k, int last)
{
    return static_cast<uint64_t>(k) * static_cast<uint32_t>(last) / (kSortSamples - 1);
}

// Points of one chunk grouped by range: entries (x, y, z, index) and, per
// range, the first of its entries (one more offset ends the last range).
__device__ __forceinline__ void bucket_chunk(const P3f *__restrict__ pts, const SortShape &s,
                                             int chunk, float4 *__restrict__ entries,
                                             uint32_t *__restrict__ offs,
                                             Curve *__restrict__ shared_curve)
{
    constexpr int kPerThread = kSortSamples / kBucketThreads;
    __shared__ uint32_t share[kRangeCells];      // samples per cell, then its range
    __shared__ uint32_t hist[kMaxRanges];
    __shared__ float red[kBucketThreads / kWave][6];
    __shared__ uint32_t total[kBucketThreads / kWave];
    __shared__ Curve curve;
    __shared__ uint32_t crowded;
    __shared__ uint16_t codes[kBucketHeld][kBucketThreads];      // of a warped curve
    const int tid = threadIdx.x;
    const int first = chunk * kSortChunk, last = s.n - 1;
    P3f p[kBucketHeld], sample[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
        sample[k] = pts[sample_at(k * kBucketThreads + tid, last)];
#pragma unroll
    for (int k = 0; k < kBucketHeld; ++k) p[k] = pts[min(first + k * kBucketThreads + tid, last)];
    for (int r = tid; r < kMaxRanges; r += kBucketThreads) hist[r] = 0u;
    for (int r = tid; r < kRangeCells; r += kBucketThreads) share[r] = 0u;
    MaxBox box;
    box.clear();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) box.add(sample[k].x, sample[k].y, sample[k].z);
    if (tid == 0) crowded = 0u;
    box.group<kBucketThreads / kWave>(red);
    if (tid == 0) {
        curve.box(box);
        curve.warped = 0u;
    }
    __syncthreads();
    const Grid grid(curve);
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
        if (atomicAdd(&share[grid.code<kRangeLevels>(sample[k].x, sample[k].y, sample[k].z)], 1u) >= kCrowdSamples)
            crowded = 1u;
    __syncthreads();
    const bool warped = __builtin_amdgcn_readfirstlane(crowded) != 0u;
    if (warped) {
        if (tid < 3 * kWave)
            curve.w.set(tid / kWave, reinterpret_cast<const float *>(
                                         pts + static_cast<uint64_t>(tid % kWave) * static_cast<uint32_t>(last) /
                                                   (kWave - 1))[tid / kWave]);
        if (tid == 0) curve.warped = 1u;
        for (int r = tid; r < kRangeCells; r += kBucketThreads) share[r] = 0u;
        __syncthreads();
        // (Loops that are not unrolled, on reloaded points: the code of the
        // usual path stays small.)
#pragma unroll 1
        for (int k = 0; k < kPerThread; ++k) {
            const P3f q = pts[sample_at(k * kBucketThreads + tid, last)];
            atomicAdd(&share[grid.warped<kRangeLevels>(q.x, q.y, q.z)], 1u);
        }
#pragma unroll 1
        for (int k = 0; k < kBucketHeld; ++k) {
            const P3f q = pts[min(first + k * kBucketThreads + tid, last)];
            codes[k][tid] = static_cast<uint16_t>(grid.warped<kRangeLevels>(q.x, q.y, q.z));
        }
    }
    if (chunk == 0)
        for (uint32_t k = tid; k < sizeof(Curve) / 4; k += kBucketThreads)
            reinterpret_cast<uint32_t *>(shared_curve)[k] = reinterpret_cast<const uint32_t *>(&curve)[k];
    scan_counters<kBucketThreads / kWave>(share, kRangeCells, total);
    // A cell whose samples follow t others belongs to range t ranges / samples.
    // A cell of four ranges' worth of samples or more (in a warped grid one and a
    // half: many equal points) is dealt out by index.
    const uint32_t deal = warped ? 3 * kSortSamples / 2 : 4 * kSortSamples;
    uint32_t range[kBucketHeld], rank[kBucketHeld];
#pragma unroll
    for (int k = 0; k < kBucketHeld; ++k) {
        const int i = first + k * kBucketThreads + tid;
        const uint32_t c = warped ? codes[k][tid] : grid.code<kRangeLevels>(p[k].x, p[k].y, p[k].z);
        const uint32_t t = share[c], own = (c + 1 < kRangeCells ? share[c + 1] : kSortSamples) - t;
        const uint32_t dealt = own * s.ranges >= deal
                                   ? (static_cast<uint32_t>(i) * 2654435761u >> 16) * own >> 16 : 0u;
        range[k] = min((t + dealt) * s.ranges / kSortSamples, static_cast<uint32_t>(s.ranges) - 1u);
        if (i <= last) rank[k] = atomicAdd(&hist[range[k]], 1u);
    }
    scan_counters<kBucketThreads / kWave>(hist, s.ranges, total);
    const uint32_t count = static_cast<uint32_t>(min(kSortChunk, s.n - first));
#pragma unroll
    for (int k = 0; k < kBucketHeld; ++k) {
        const int i = first + k * kBucketThreads + tid;
        if (i <= last)
            entries[first + hist[range[k]] + rank[k]] =
                make_float4(p[k].x, p[k].y, p[k].z, __uint_as_float(static_cast<uint32_t>(i)));
    }
    uint32_t *o = offs + static_cast<size_t>(chunk) * (s.ranges + 1);
    for (int r = tid; r < s.ranges; r += kBucketThreads) o[r] = hist[r];
    if (tid == 0) o[s.ranges] = count;
}

// Range w of one cloud.  What it reads back from the workspace (segments,
// points) is bounded before it is an address: a call that shares the workspace
// with another may get wrong results, but writes within its own arrays.
__device__ __forceinline__ void sort_range(const P3f *__restrict__ pts, const SortShape &s, int w,
                                           const float4 *__restrict__ entries,
                                           const uint32_t *__restrict__ offs,
                                           const Curve *__restrict__ shared_curve,
                                           float4 *__restrict__ rec, Box *__restrict__ leaf,
                                           Box *__restrict__ node)
{
    __shared__ uint32_t cells[1 << kLogCells];
    __shared__ uint32_t pre[kMaxChunks + 1], seg[kMaxChunks];
    __shared__ float red[kSortWaves][6];
    __shared__ uint32_t total[kSortWaves], below_total[kSortWaves], ends[kSortWaves][2];
    __shared__ Curve curve;
    __shared__ uint32_t crowded;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int ncell = 1 << s.log_c, ranges = s.ranges;
    const bool one = ranges == 1;
    uint32_t count = static_cast<uint32_t>(s.n), below = 0u;
    const int scanned = max(ncell, kSortThreads);
    for (int c = tid; c < scanned; c += kSortThreads) cells[c] = 0u;
    if (!one) {
        // The range's segment of every chunk (two chunks per thread), the
        // points before each, and the points of lower ranges.
        uint32_t len[2], lower = 0u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int c = 2 * tid + k;
            const uint32_t *o = offs + static_cast<size_t>(min(c, s.chunks - 1)) * (ranges + 1) + w;
            const uint32_t held = static_cast<uint32_t>(min(kSortChunk, s.n - min(c, s.chunks - 1) * kSortChunk));
            const uint32_t a = min(o[0], held), e = min(max(o[1], a), held);
            len[k] = c < s.chunks ? e - a : 0u;
            lower += c < s.chunks ? a : 0u;
            if (c < s.chunks) seg[c] = a;
        }
        const uint32_t incl = wave_scan_u32(len[0] + len[1]), li = wave_scan_u32(lower);
        if (lane == kWave - 1) {
            total[wave] = incl;
            below_total[wave] = li;
        }
        __syncthreads();
        uint32_t before = incl - len[0] - len[1];
        count = 0u;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            const uint32_t t = total[k];
            before += k < wave ? t : 0u;
            count += t;
            below += below_total[k];
        }
        count = min(count, static_cast<uint32_t>(s.n) - min(below, static_cast<uint32_t>(s.n)));
        if (2 * tid < s.chunks) pre[2 * tid] = before;
        if (2 * tid + 1 < s.chunks) pre[2 * tid + 1] = before + len[0];
        if (tid == 0) pre[s.chunks] = count;
        __syncthreads();
    }
    // Point i of the range.
    const auto fetch = [&](uint32_t i) -> float4 {
        if (one) {
            const P3f p = pts[i];
            return make_float4(p.x, p.y, p.z, __uint_as_float(i));
        }
        int lo = 0, hi = s.chunks;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= i) lo = mid; else hi = mid;
        }
        return entries[static_cast<uint32_t>(lo) * kSortChunk + seg[lo] + (i - pre[lo])];
    };
    const uint32_t start = (below + kNode - 1) / kNode * kNode + static_cast<uint32_t>(w) * kNode;
    const uint32_t next = (below + count + kNode - 1) / kNode * kNode + static_cast<uint32_t>(w + 1) * kNode;
    float4 *out = rec + start;
    if (count > 0u) {
        const bool held = count <= kSortHeld * kSortThreads;
        float4 p[kSortHeld];
        if (held) {
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k)
                if (static_cast<uint32_t>(k * kSortThreads) < count)
                    p[k] = fetch(min(static_cast<uint32_t>(k * kSortThreads + tid), count - 1));
                else
                    p[k] = p[0];
        }
        if (one) {
            MaxBox box;
            box.clear();
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k) box.add(p[k].x, p[k].y, p[k].z);
            box.group<kSortWaves>(red);
            if (tid == 0) {
                curve.box(box);
                curve.warped = 0u;
            }
        } else if (tid < static_cast<int>(sizeof(Curve) / 4)) {
            reinterpret_cast<uint32_t *>(&curve)[tid] = reinterpret_cast<const uint32_t *>(shared_curve)[tid];
        }
        if (tid == 0) crowded = 0u;
        __syncthreads();
        const Grid grid(curve);
        bool warped = __builtin_amdgcn_readfirstlane(curve.warped) != 0u;
        // The range's codes from the lowest on, in as many cells as there are.
        uint32_t code[kSortHeld], rank[kSortHeld], low = kNoPoint, high = 0u;
        int down = 0;
        const auto code_of = [&](const float4 &q) {
            return warped ? grid.warped<kLevels>(q.x, q.y, q.z) : grid.code<kLevels>(q.x, q.y, q.z);
        };
        const auto cell = [&](const float4 &q) {
            return min((code_of(q) - low) >> down, static_cast<uint32_t>(ncell) - 1u);
        };
        const auto span = [&] {     // low, high of the workgroup
            low = wave_min_u32(low);
            high = ~wave_min_u32(~high);
            if (lane == 0) {
                ends[wave][0] = low;
                ends[wave][1] = ~high;
            }
            __syncthreads();
            low = wave_min_u32(ends[lane % kSortWaves][0]);
            high = ~wave_min_u32(ends[lane % kSortWaves][1]);
            down = max(32 - __builtin_clz((high - low) | 1u) - s.log_c, 0);
        };
        const uint32_t crowd = max(count * kCrowdSixteenths / 16u, kCrowdPoints);
        const auto rank_held = [&] {    // codes -> ranks within cells; notes a crowded one
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k)
                if (static_cast<uint32_t>(k * kSortThreads) < count) {
                    low = min(low, code[k]);
                    high = max(high, code[k]);
                }
            span();
            bool full = false;
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k)
                if (static_cast<uint32_t>(k * kSortThreads + tid) < count) {
                    rank[k] = atomicAdd(&cells[(code[k] - low) >> down], 1u);
                    full |= rank[k] >= crowd;
                }
            if (full) crowded = 1u;
            __syncthreads();
        };
        bool done = false;
        if (held && !warped) {
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k)
                if (static_cast<uint32_t>(k * kSortThreads) < count)
                    code[k] = grid.code<kLevels>(p[k].x, p[k].y, p[k].z);
            rank_held();
            done = __builtin_amdgcn_readfirstlane(crowded) == 0u;
        }
        // Otherwise: many points, a warped curve, or a crowded cell, which takes
        // the range's own quantiles.  (Apart from the usual path, which a loop
        // around both made 8 us slower.)
        for (bool own = false; !done;) {
            if (!own && __builtin_amdgcn_readfirstlane(crowded) != 0u) {
                own = warped = true;
                if (wave < 3) {
                    const float4 q = fetch(static_cast<uint32_t>(lane) * (count - 1u) / (kWave - 1u));
                    curve.w.set(wave, wave == 0 ? q.x : wave == 1 ? q.y : q.z);
                }
                for (int c = tid; c < scanned; c += kSortThreads) cells[c] = 0u;
                __syncthreads();
            }
            low = kNoPoint;
            high = 0u;
            if (held) {
#pragma unroll
                for (int k = 0; k < kSortHeld; ++k)
                    if (static_cast<uint32_t>(k * kSortThreads) < count)
                        code[k] = grid.warped<kLevels>(p[k].x, p[k].y, p[k].z);
                rank_held();
            } else {
                for (uint32_t i = tid; i < count; i += kSortThreads) {
                    const uint32_t c = code_of(fetch(i));
                    low = min(low, c);
                    high = max(high, c);
                }
                span();
                bool full = false;
                for (uint32_t i = tid; i < count; i += kSortThreads)
                    full |= atomicAdd(&cells[cell(fetch(i))], 1u) >= crowd;
                if (full) crowded = 1u;
                __syncthreads();
            }
            done = own || __builtin_amdgcn_readfirstlane(crowded) == 0u;
        }
        scan_counters<kSortWaves>(cells, scanned, total);
        if (held) {
#pragma unroll
            for (int k = 0; k < kSortHeld; ++k)
                if (static_cast<uint32_t>(k * kSortThreads + tid) < count)
                    out[cells[(code[k] - low) >> down] + rank[k]] = record(p[k]);
        } else {
            for (uint32_t i = tid; i < count; i += kSortThreads) {
                const float4 q = fetch(i);
                out[min(atomicAdd(&cells[cell(q)], 1u), count - 1u)] = record(q);
            }
        }
        const uint32_t filled = (count + kTile - 1) / kTile * kTile;
        for (uint32_t t = count + tid; t < filled; t += kSortThreads)
            out[t] = make_float4(kFarAway, 0.0f, 0.0f, __uint_as_float(kNoPoint));
        __syncthreads();
    }
    // Boxes: a wave takes a node, a lane a leaf.
    for (uint32_t nd = start / kNode + wave; nd < next / kNode; nd += kSortWaves) {
        const uint32_t r0 = nd * kNode + lane * kLeaf - start;   // first record of the leaf
        MaxBox b;
        b.clear();
        uint32_t first = kNoPoint, nans = 0u;
        if (r0 < count) {
            const uint32_t m = min(static_cast<uint32_t>(kLeaf), count - r0);
            const float4 *src = out + r0;
#pragma unroll
            for (uint32_t u = 0; u < kLeaf; ++u) {
                const float4 q = src[min(u, m - 1)];
                const bool point = __float_as_uint(q.w) != kNoPoint;
                if (point) b.add(q.x, q.y, q.z);
                first = min(first, __float_as_uint(q.w));
                nans |= point ? 0u : 1u;
            }
        }
        leaf[static_cast<size_t>(nd) * kNodeLeaves + lane] =
            Box{-b.v[0], -b.v[1], -b.v[2], first, b.v[3], b.v[4], b.v[5], nans};
#pragma unroll
        for (int c = 0; c < 6; ++c) b.v[c] = wave_max(b.v[c]);
        first = wave_min_u32(first);
        if (lane == 0) node[nd] = Box{-b.v[0], -b.v[1], -b.v[2], first, b.v[3], b.v[4], b.v[5], 0u};
    }
}

struct SortArgs {
    SortJob job[2];
    uint32_t *zero;
    uint32_t n;
};

__global__ __launch_bounds__(kBucketThreads) void bucket_kernel(SortArgs a)
{
    const uint32_t wg = xcd_block();
    const uint32_t c0 = a.job[0].s.chunks, c1 = a.job[1].s.chunks;
    const int64_t b = wg / (c0 + c1);
    const uint32_t c = wg % (c0 + c1);
    const SortJob &t = a.job[c < c0 ? 0 : 1];
    if (t.s.ranges == 1) return;     // sorted straight from the cloud
    bucket_chunk(reinterpret_cast<const P3f *>(t.P) + b * t.s.n, t.s,
                 static_cast<int>(c < c0 ? c : c - c0),
                 t.entries + b * t.s.chunks * kSortChunk,
                 t.offs + b * t.s.chunks * (t.s.ranges + 1), t.curve + b);
}

__global__ __launch_bounds__(kSortThreads) void sort_kernel(SortArgs a)
{
    if (blockIdx.x == 0)
        for (uint32_t k = threadIdx.x; k < a.n; k += kSortThreads) a.zero[k] = 0u;
    const uint32_t wg = xcd_block();
    const uint32_t w0 = a.job[0].s.ranges, w1 = a.job[1].s.ranges;
    const int64_t b = wg / (w0 + w1);
    const uint32_t w = wg % (w0 + w1);
    const SortJob &t = a.job[w < w0 ? 0 : 1];
    sort_range(reinterpret_cast<const P3f *>(t.P) + b * t.s.n, t.s,
               static_cast<int>(w < w0 ? w : w - w0), t.entries + b * t.s.chunks * kSortChunk,
               t.offs + b * t.s.chunks * (t.s.ranges + 1), t.curve + b,
               t.rec + b * t.s.nodes * kNode, t.leaf + b * t.s.nodes * kNodeLeaves,
               t.node + b * t.s.nodes);
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

SortPlan plan_sort(int64_t B, int64_t n, size_t &at)
{
    SortPlan p{};
    p.B = B;
    p.s.n = static_cast<int32_t>(n);
    p.s.chunks = static_cast<int32_t>(ceil_div(n, kSortChunk));
    p.s.ranges = n <= kOneRange ? 1 : static_cast<int32_t>(std::min<int64_t>(ceil_div(n, kRangePoints), kMaxRanges));
    p.s.log_c = std::min(std::max(ceil_log2(n) + 2, 9), kLogCells);
    p.s.nodes = static_cast<int32_t>(ceil_div(n, kNode) + p.s.ranges);
    const size_t b = static_cast<size_t>(B);
    const auto place = [&](size_t &where, size_t bytes) {
        where = at;
        at += align256(bytes);
    };
    place(p.entries, p.s.ranges > 1 ? b * p.s.chunks * kSortChunk * sizeof(float4) : 0);
    place(p.offs, p.s.ranges > 1 ? b * p.s.chunks * (p.s.ranges + 1) * 4 : 0);
    place(p.curve, b * sizeof(Curve));
    place(p.rec, b * p.s.nodes * kNode * sizeof(float4));
    place(p.leaf, b * p.s.nodes * kNodeLeaves * sizeof(Box));
    place(p.node, b * p.s.nodes * sizeof(Box));
    return p;
}

SortJob sort_job(const SortPlan &p, const float *P, char *ws)
{
    SortJob j{};
    j.P = P;
    j.rec = reinterpret_cast<float4 *>(ws + p.rec);
    j.leaf = reinterpret_cast<Box *>(ws + p.leaf);
    j.node = reinterpret_cast<Box *>(ws + p.node);
    j.entries = reinterpret_cast<float4 *>(ws + p.entries);
    j.offs = reinterpret_cast<uint32_t *>(ws + p.offs);
    j.curve = reinterpret_cast<Curve *>(ws + p.curve);
    j.s = p.s;
    return j;
}

hipError_t launch_sort(int64_t B, const SortJob &a, const SortJob &b, uint32_t *zero, uint32_t n,
                       hipStream_t stream)
{
    const SortArgs args{{a, b}, zero, n};
    if (a.s.ranges > 1 || b.s.ranges > 1)
        bucket_kernel<<<static_cast<uint32_t>(B * (static_cast<int64_t>(a.s.chunks) + b.s.chunks)),
                        kBucketThreads, 0, stream>>>(args);
    sort_kernel<<<static_cast<uint32_t>(B * (static_cast<int64_t>(a.s.ranges) + b.s.ranges)),
                  kSortThreads, 0, stream>>>(args);
    return hipGetLastError();
}

}  // namespace cdk
