// Image comparison measures of Sec. 5.2 (Tables 3 and 4) on the device.
//
// Both images are divided by their largest pixel.  Over pixels: RMSE of the
// difference and Pearson's r.  Radially: the normalised images averaged over
// annuli one pixel wide around (cx, cy) out to r_max (annulus k holds
// k <= rho < k + 1, rho from the pixel centre (j + 0.5, i + 0.5), computed
// from rho^2, exact for such centres), zones by theta = 180 deg (k + 0.5) /
// r_max (< 30, 30..120, > 120 deg) with the RMSE of the two profiles in each,
// Pearson's r of the profiles, and, given a third image c, the share of
// annuli where a is closer to b than c is.
//
// Two kernels: block maxima; then pixel sums per block and annulus sums in
// int64 fixed point (2^38 per unit, so their totals do not depend on the order
// of the atomics), with the totals, profiles and measures taken by the block
// that finishes last.  Blocks of the second kernel own whole tiles of 64 x 64
// pixels (of as many in a flat image), which touch few annuli, so few annulus sums leave a block, and a wave
// takes patches of 8 x 8 of them: about 8 of its lanes meet in one annulus, where
// a row of 64 pixels can lie in a single one.  Every sum over pixels or annuli is
// a fixed partition and tree, whatever block is last.
//
// At 512 x 512 with a third image the call reads 6.3 MB, 1.3 us at the copy
// rate; it is bound by latency, each kernel being a few dependent trips to
// memory.  One lane that walked over the blocks' sums and the annuli took 200
// of the 263 us the call took; now the kernels take 4.7 and 18.6 us (about 5 of
// them the annulus adds in LDS, 6 the last block's part) and the call 48, the
// rest of which is launches and the wait.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "common.hpp"
#include "wave.hpp"

namespace mcmie {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxGrid = 256;
constexpr int kTileBits = 6;                   // tiles are 2^6 columns wide (fewer for narrow images, more for flat ones)
constexpr int kTileRows = 4;                   // pixels of a tile per lane
constexpr double kRadFix = 274877906944.0;     // 2^38
constexpr int kPix = 6;                        // pixel sums per block: x, y, xx, yy, xy, (x - y)^2

struct MetricsArgs {
    const double *a, *b, *c;
    int nx, ny;
    double cx, cy, r_max;
    int n_r;
    uint64_t n_pix, per_block;
    uint32_t tile_bits, tiles_x, tiles, tiles_per_block;   // tiles of 2^tile_bits columns, four pixels per lane
    double *blk_max;                 // grid x 3
    double *blk_sum;                 // grid x kPix
    unsigned long long *rad;         // n_r x 4: pixels, a, b, c (fixed point)
    unsigned long long *done;        // blocks that have finished their sums (the word of out[11], written last)
    double *out;                     // MC_METRICS_N (device)
    double *result;                  // where the measures go: out, or pinned host memory
    double *profiles;                // optional: 4 x n_r (a, b, c profiles, pixel counts)
};

// op over N <= kWaves values of every lane of the block, in a fixed order: over
// the rows of each wave without touching LDS, then wave i over the 64 rows of
// value i.  Every lane gets the results.  `s` holds N x 65 doubles.  (Exchanges
// through LDS, ds_bpermute, took 0.9 us a value with 16 waves at it.)
template <int N, class Op>
__device__ __forceinline__ void block_reduce(double (&v)[N], double *s, Op op)
{
    static_assert(N <= kWaves, "a wave per value");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = row_reduce(v[i], op);
    if ((lane & 15) == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) s[i * 64 + wave * 4 + (lane >> 4)] = v[i];
    __syncthreads();
    if (wave < N) {
        const double r = row_reduce(s[wave * 64 + lane], op);
        const int2 x = __builtin_bit_cast(int2, r);
        double row[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            row[i] = __builtin_bit_cast(double, int2{__builtin_amdgcn_readlane(x.x, 16 * i),
                                                     __builtin_amdgcn_readlane(x.y, 16 * i)});
        if (lane == 0) s[N * 64 + wave] = op(op(row[0], row[1]), op(row[2], row[3]));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s[N * 64 + i];
    __syncthreads();
}
template <int N>
__device__ __forceinline__ void block_max(double (&v)[N], double *s)
{
    block_reduce(v, s, [](double x, double y) { return fmax(x, y); });
}
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double *s)
{
    block_reduce(v, s, [](double x, double y) { return x + y; });
}

__global__ __launch_bounds__(kThreads) void metrics_max(MetricsArgs m)
{
    __shared__ double s[3 * 65];
    const uint64_t lo = (uint64_t)blockIdx.x * m.per_block;
    const uint64_t hi = lo + m.per_block < m.n_pix ? lo + m.per_block : m.n_pix;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
    for (uint64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
        v[0] = fmax(v[0], m.a[i]);
        v[1] = fmax(v[1], m.b[i]);
        if (m.c) v[2] = fmax(v[2], m.c[i]);
    }
    // Clear the annulus sums and the block count for the next kernel.
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < 4 * m.n_r; i += gridDim.x * kThreads) m.rad[i] = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) *m.done = 0ull;
    block_max(v, s);
    if (threadIdx.x < 3) m.blk_max[3 * blockIdx.x + threadIdx.x] = v[threadIdx.x == 0 ? 0 : (threadIdx.x == 1 ? 1 : 2)];
}

// The totals, profiles and measures, by all lanes of one block.
__device__ void metrics_final(const MetricsArgs &m, const double (&top)[3], double *s, double *s_prof)
{
    const int tid = threadIdx.x;
    // Radial profiles and the measures over non-empty annuli: squared errors
    // and annuli of the zones, annuli used, profile sums, annuli where a is
    // closer than c.
    // And the pixel sums over the blocks (10..15).
    double q[10 + kPix] = {};
    for (int g = tid; g < (int)gridDim.x; g += kThreads)
        for (int j = 0; j < kPix; ++j) q[10 + j] += m.blk_sum[kPix * g + j];
    for (int k = tid; k < m.n_r; k += kThreads) {
        const double cnt = (double)m.rad[4 * k + 0];
        const double pa = cnt > 0 ? (double)m.rad[4 * k + 1] * (1.0 / kRadFix) / cnt : 0.0;
        const double pb = cnt > 0 ? (double)m.rad[4 * k + 2] * (1.0 / kRadFix) / cnt : 0.0;
        const double pc = cnt > 0 ? (double)m.rad[4 * k + 3] * (1.0 / kRadFix) / cnt : 0.0;
        if (m.profiles) {
            m.profiles[k] = pa;
            m.profiles[m.n_r + k] = pb;
            m.profiles[2 * m.n_r + k] = pc;
            m.profiles[3 * m.n_r + k] = cnt;
        }
        s_prof[2 * k] = cnt > 0 ? pa : -1.0;     // (a profile is never negative)
        s_prof[2 * k + 1] = pb;
        if (cnt > 0) {
            const double theta = 180.0 * (k + 0.5) / m.r_max;
            const int z = theta < 30.0 ? 0 : (theta <= 120.0 ? 1 : 2);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                q[i] += z == i ? (pa - pb) * (pa - pb) : 0.0;
                q[3 + i] += z == i ? 1.0 : 0.0;
            }
            q[6] += 1.0;
            q[7] += pa;
            q[8] += pb;
            if (m.c && fabs(pa - pb) < fabs(pc - pb)) q[9] += 1.0;
        }
    }
    block_sum(q, s);
    const double *t = q + 10;
    const double used = q[6], ma = used > 0 ? q[7] / used : 0.0, mb = used > 0 ? q[8] / used : 0.0;
    double c[3] = {0, 0, 0};
    for (int k = tid; k < m.n_r; k += kThreads) {
        if (s_prof[2 * k] < 0.0) continue;
        const double pa = s_prof[2 * k] - ma, pb = s_prof[2 * k + 1] - mb;
        c[0] += pa * pb;
        c[1] += pa * pa;
        c[2] += pb * pb;
    }
    block_sum(c, s);
    if (tid != 0) return;
    const double n = (double)m.n_pix;
    m.result[0] = sqrt(t[5] / n);
    const double cov = t[4] - t[0] * t[1] / n, vx = t[2] - t[0] * t[0] / n, vy = t[3] - t[1] * t[1] / n;
    const double den = sqrt(vx * vy);
    m.result[1] = den > 0.0 ? cov / den : NAN;
#pragma unroll
    for (int z = 0; z < 3; ++z) m.result[2 + z] = q[3 + z] > 0 ? sqrt(q[z] / q[3 + z]) : 0.0;
    const double rden = sqrt(c[1] * c[2]);
    m.result[5] = rden > 0.0 ? c[0] / rden : NAN;
    m.result[6] = (double)m.n_r;
    for (int i = 0; i < 3; ++i) m.result[7 + i] = top[i];
    m.result[10] = m.c ? (used > 0 ? q[9] / used : NAN) : NAN;
    m.result[11] = n;
}

__global__ __launch_bounds__(kThreads) void metrics_sums(MetricsArgs m)
{
    extern __shared__ __attribute__((aligned(16))) unsigned long long s_rad[];   // 4 x n_r
    __shared__ double s[kWaves * 65];
    __shared__ uint32_t s_last;
    const int tid = threadIdx.x;
    double top[3] = {0.0, 0.0, 0.0};
    for (int g = tid; g < (int)gridDim.x; g += kThreads)
        for (int j = 0; j < 3; ++j) top[j] = fmax(top[j], m.blk_max[3 * g + j]);
    for (int i = tid; i < 4 * m.n_r; i += kThreads) s_rad[i] = 0ull;
    block_max(top, s);   // (also the barrier after the clearing)
    const double ia = top[0] > 0.0 ? 1.0 / top[0] : 0.0, ib = top[1] > 0.0 ? 1.0 / top[1] : 0.0;
    const double ic = top[2] > 0.0 ? 1.0 / top[2] : 0.0;
    double acc[kPix] = {};
    const double r2max = m.r_max * m.r_max;
    const uint32_t t0 = blockIdx.x * m.tiles_per_block, t1 = min(t0 + m.tiles_per_block, m.tiles);
    for (uint32_t t = t0; t < t1; ++t) {
        const int tb = (int)m.tile_bits, sb = max(min(tb, 3), tb - 6), lane = tid & 63;
        const int col0 = (int)((t % m.tiles_x) << tb) + (lane & ((1 << sb) - 1));
        const int row0 = (int)(t / m.tiles_x) * ((kTileRows * kThreads) >> tb) + (lane >> sb);
        double va[kTileRows], vb[kTileRows], vc[kTileRows];
        int row[kTileRows], col[kTileRows];
#pragma unroll
        for (int u = 0; u < kTileRows; ++u) {
            const int patch = (tid >> 6) + u * kWaves;
            col[u] = col0 + ((patch & ((1 << (tb - sb)) - 1)) << sb);
            row[u] = row0 + ((patch >> (tb - sb)) << (6 - sb));
            const uint64_t i = (uint64_t)row[u] * (uint64_t)m.nx + (uint64_t)col[u];
            const bool in = col[u] < m.nx && row[u] < m.ny;
            va[u] = in ? m.a[i] : 0.0;
            vb[u] = in ? m.b[i] : 0.0;
            vc[u] = in && m.c ? m.c[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kTileRows; ++u) {
            if (!(col[u] < m.nx && row[u] < m.ny)) continue;
            // Normalised by the largest pixel (a zero image stays zero).
            const double x = va[u] * ia, y = vb[u] * ib;
            acc[0] += x;
            acc[1] += y;
            acc[2] += x * x;
            acc[3] += y * y;
            acc[4] += x * y;
            acc[5] += (x - y) * (x - y);
            const double dx = (col[u] + 0.5) - m.cx, dy = (row[u] + 0.5) - m.cy;
            const double r2 = dx * dx + dy * dy;
            if (r2 < r2max) {
                const int k = min((int)floor(sqrt(r2)), m.n_r - 1);
                atomicAdd(&s_rad[4 * k + 0], 1ull);
                atomicAdd(&s_rad[4 * k + 1], (unsigned long long)llrint(x * kRadFix));
                atomicAdd(&s_rad[4 * k + 2], (unsigned long long)llrint(y * kRadFix));
                if (m.c) atomicAdd(&s_rad[4 * k + 3], (unsigned long long)llrint(vc[u] * ic * kRadFix));
            }
        }
    }
    block_sum(acc, s);   // (also the barrier after the annulus sums)
    if (tid == 0)
        for (int j = 0; j < kPix; ++j) m.blk_sum[kPix * blockIdx.x + j] = acc[j];
    for (int i = tid; i < 4 * m.n_r; i += kThreads)
        if (s_rad[i]) atomicAdd(&m.rad[i], s_rad[i]);
    // The block that finishes last sees every block's sums: each wave waits for its
    // own annulus adds (a barrier does not: on this GPU it orders LDS only, and the
    // adds, whose results nobody reads, would still be under way), then one lane
    // makes the block's pixel sums visible to the device and counts the block as
    // done.  The adds are device-scope and need no write-back of the L2 (a fence by
    // each wave wrote it back once per wave).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        s_last = atomicAdd(m.done, 1ull) == gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    metrics_final(m, top, s, (double *)s_rad);
}

uint64_t grid_for(uint64_t n_pix)
{
    // Four pixels per lane, at most one block per compute unit.
    const uint64_t g = (n_pix + kThreads * 4 - 1) / (kThreads * 4);
    return g < 1 ? 1 : (g > kMaxGrid ? kMaxGrid : g);
}

uint64_t metrics_work_words(uint64_t n_pix, int n_r)
{
    const uint64_t g = grid_for(n_pix);
    return g * 3 + g * (kPix + 1) + 4ull * n_r + MC_METRICS_N;   // (a word per block to spare)
}

int annuli(const mc_radial_t &r) { return (int)std::ceil(r.r_max); }

}  // namespace
}  // namespace mcmie

extern "C" uint64_t mc_metrics_work_bytes(int32_t nx, int32_t ny, const mc_radial_t *radial)
{
    using namespace mcmie;
    if (nx < 1 || ny < 1 || !radial || !(radial->r_max > 0.0) || annuli(*radial) > MC_MAX_ANNULI) return 0;
    return metrics_work_words((uint64_t)nx * ny, annuli(*radial)) * 8;
}

extern "C" int mc_image_metrics(const double *a, const double *b, const double *c, int32_t nx, int32_t ny,
                                const mc_radial_t *radial, double *profiles, void *work, uint64_t work_bytes,
                                double out[MC_METRICS_N], void *stream)
{
    using namespace mcmie;
    clear_error();
    if (!a || !b || !radial || !work || !out) return fail(MC_EINVAL, "mc_image_metrics: null argument");
    if (nx < 1 || ny < 1 || (uint64_t)nx * ny > (1ull << 24))
        return fail(MC_EINVAL, "mc_image_metrics: image of %d x %d outside 1 .. 2^24 pixels", nx, ny);
    const mc_radial_t r = *radial;
    if (!std::isfinite(r.cx) || !std::isfinite(r.cy) || !(r.r_max > 0.0) || !std::isfinite(r.r_max) ||
        annuli(r) > MC_MAX_ANNULI)
        return fail(MC_EINVAL, "mc_image_metrics: need a finite centre and 0 < r_max <= %d", MC_MAX_ANNULI);
    const uint64_t n_pix = (uint64_t)nx * ny;
    const int n_r = annuli(r);
    if (((uintptr_t)work & 7) || work_bytes < metrics_work_words(n_pix, n_r) * 8)
        return fail(MC_EINVAL, "mc_image_metrics: work needs %llu bytes, 8-byte aligned",
                    (unsigned long long)(metrics_work_words(n_pix, n_r) * 8));
    const uint64_t g = grid_for(n_pix);
    MetricsArgs m{};
    m.a = a; m.b = b; m.c = c;
    m.nx = nx; m.ny = ny;
    m.cx = r.cx; m.cy = r.cy; m.r_max = r.r_max;
    m.n_r = n_r;
    m.n_pix = n_pix;
    m.per_block = (n_pix + g - 1) / g;
    double *w = (double *)work;
    m.blk_max = w;
    m.blk_sum = w + 3 * g;
    m.rad = (unsigned long long *)(w + 3 * g + kPix * g);
    m.out = w + 3 * g + kPix * g + 4ull * n_r;
    m.done = (unsigned long long *)(m.out + 11);
    HostResult host;
    m.result = host ? host.data() : m.out;
    m.profiles = profiles;
    // Tiles of 4096 pixels: 64 columns and rows, fewer columns than that only where the
    // image has fewer, and more where it has fewer rows (always 64 rows a tile: the
    // call took 799 us for 2^24 x 1 pixels and 73.9 for 1e5 x 1, with flat tiles 181 and 35.8).
    while (m.tile_bits < (uint32_t)kTileBits && (1 << m.tile_bits) < nx) ++m.tile_bits;
    constexpr uint32_t kPixBits = 12;
    static_assert(kTileRows * kThreads == 1 << kPixBits, "pixels of a tile");
    while (m.tile_bits < kPixBits && (1 << m.tile_bits) < nx && (1 << (kPixBits - 1 - m.tile_bits)) >= ny) ++m.tile_bits;
    const uint32_t tile_h = 1u << (kPixBits - m.tile_bits);
    m.tiles_x = ((uint32_t)nx + (1u << m.tile_bits) - 1) >> m.tile_bits;
    m.tiles = m.tiles_x * (((uint32_t)ny + tile_h - 1) / tile_h);
    m.tiles_per_block = (uint32_t)((m.tiles + g - 1) / g);
    hipStream_t st = (hipStream_t)stream;
    const size_t lds = (size_t)4 * n_r * sizeof(unsigned long long);
    MC_HIP_CHECK(hipFuncSetAttribute((const void *)metrics_sums, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(metrics_max, dim3((unsigned)g), dim3(kThreads), 0, st, m);
    hipLaunchKernelGGL(metrics_sums, dim3((unsigned)g), dim3(kThreads), lds, st, m);
    MC_HIP_CHECK(hipGetLastError());
    MC_HIP_CHECK(wait_result(out, MC_METRICS_N, m.result, host, st));
    return MC_OK;
}
