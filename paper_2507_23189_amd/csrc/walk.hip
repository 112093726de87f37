// The photon walk of Sec. 3.1.3 on gfx950.
//
// Each lane carries one photon at a time in registers (position, direction,
// weight, path length, scatter count, step) and runs the walk one step per
// loop trip.  When a lane's photon ends it takes, at the wave's next round, the
// next photon id from its wave's current id range.  A wave takes ranges of
// `chunk` ids from its block's pool in LDS, and the block refills the pool from
// a global counter, so lanes stay busy until the budget is spent and the
// counter, one device-scope atomic per claim, sees a few per block.
//
// One step: a Philox4x32-10 block (counter = step, instance, id_lo, id_hi;
// key = seed) gives four uniforms u0..u3 and the free path s = -ln(u0)/mu_ext
// (Eq. 15).  If the free path ends inside the cuboid, clear of the walls by a
// margin that covers all rounding, the photon interacts: the weight update of
// Eq. 16 (implicit capture), Russian roulette (u3), and a new direction at the
// polar angle read from the LDS-resident inverse CDF (u1, direct index and
// linear interpolation of v = 1 - cos(theta)) or from Henyey-Greenstein
// (Eq. 11), with azimuth 2 pi u2, built in the orthonormal basis of Duff et
// al. 2017 around the old direction.  Otherwise the lane waits for a round,
// which finds the distance to the nearest wall, compares s with it, and moves
// the photon there to be reflected with the unpolarised Fresnel reflectance
// (u3) or to leave and be tallied.
//
// The kernel is bound by VALU issue: at tau = 16 it issues 2.8 cycles of VALU
// work per instruction all the time, which is its instructions' own price.
// On gfx950 a wave64 FP32 add, multiply or fma whose operands are all vector
// registers issues in 2 cycles, while compares, selects, min/max, conversions,
// shifts, 32-bit products and any FP32 operation with a scalar-register operand
// take 4 and transcendentals 8.  So the step holds only what every lane needs
// (about 310 cycles, 134 of them the random block): its FP32 constants sit in
// vector registers, the test against the walls has no division (three fma a
// coordinate pair and one three-way maximum), roulette and the step cap are
// looked at only where a photon of the wave could meet them, the parts of the
// random block that do not depend on the step are kept per photon, and walls
// (which 22 % of the lanes meet in a step at tau = 4, 6 % at tau = 16) are left
// to the rounds, about 400 cycles each, that run when refill_min lanes wait.
// Resolving walls in every step, with the distances for all lanes, took 2.69
// ms at tau = 4 and 8.6 at tau = 16 for 1e8 photons (mc_simulate, 512 x 512,
// exit log); this takes 2.30 and 6.5.
//
// Transport runs in FP32.  Weights are tallied in 64-bit fixed point
// (weight * 2^32, rounded to nearest): integer sums do not depend on the order
// in which photons finish, so results are bit-identical for any launch shape
// and for either tally path.  Exits through the imaged faces are first queued
// per wave in LDS and handled 64 at a time by the whole wave, so the pixel
// arithmetic runs with full lanes instead of on the few lanes that exit in
// any one step.  A flush then either
//   * appends them to the exit log (MC_EXIT_LOG, or room for it among the image
//     copies): each block owns a region of every key range and appends at the
//     position an LDS counter of the block hands out (one LDS add and one store
//     per exit); a second kernel
//     (log_bin) sums each range in an LDS histogram and writes the sums into
//     image copies with plain loads and stores.  Exits that find their region
//     full are added as in the other path; or
//   * adds them into a per-block LDS tally cache (direct-mapped pixel ids
//     claimed with an LDS compare-and-swap) whose sums go to the images once
//     per block, with a global atomic into one of at most eight per-XCD copies
//     of the images for the pixels that miss the cache.
// The card performs 24 thousand million global atomics a second at best,
// whatever the number of copies, so the log, which needs none, is the faster
// path from a few million photons up; below, the second pass costs more than
// the atomics, and both paths add directly.  Unscattered photons all leave
// through one pixel with one weight and are only counted.  A finalize pass
// sums the copies in integer arithmetic and converts to the caller's images.
// Scalar tallies use LDS atomics and lane accumulators, flushed once per
// block; reflections are not counted but derived from the step, event and
// exit counts when finalizing.  The kernel is specialised at compile time on
// the phase function, the squared-weight tally, per-photon records, path
// moments, batching and the exit log.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cmath>
#include <cstdint>
#include <algorithm>
#include <mutex>
#include <vector>

#include "common.hpp"
#include "philox.hpp"
#include "plan.hpp"

// Device scratch of mc_simulate_noalloc: the scalar words and the fixed-point
// copies of the images (and squared-weight images), at least one, for callers
// that cannot allocate a workspace.  Every GPU the library runs on holds its own copy
// until the process ends.  (Aligned to 64 KB: at multiples of 256 bytes, which follow
// the size of the code, 1e6 photons took 63.5 or 68.8 us.)
constexpr unsigned long long kNoAllocWords = 32 + (1ull << 21);
static __device__ __align__(65536) unsigned long long scratch[kNoAllocWords];

namespace mcmie {
namespace {

// One medium of a batched launch, in the order its work units are handed out.
struct BatchInst {
    float neg_ln2_over_mu, albedo, absorb, pad;   // as WalkArgs, for this medium
    const float *inv_cdf;     // device inverse table of this medium (n_cdf entries)
    uint64_t n_photons;
    uint64_t unit_begin;      // first work unit of this medium
    uint32_t counter;         // Philox counter word 1 of its photons
    uint32_t slot;            // index of its images and scalars in the caller's arrays
};

static_assert(sizeof(BatchInst) == kBatchInstBytes, "the workspace has room for the schedule");

struct WalkArgs {
    float size[3];
    float neg_ln2_over_mu;    // s = log2(u0) * neg_ln2_over_mu  (= -ln(u0) / mu_ext)
    float albedo, absorb;     // albedo and 1 - albedo
    float n21, n12sq;         // n_out / n_med and (n_med / n_out)^2
    float n12;                // n_med / n_out (exit refraction, records only)
    int matched;              // n_out == n_med: no Fresnel term
    float fresnel;            // 1 where the walls have a Fresnel term, 0 where they are index-matched
    float pos0[3], dir0[3], w0;
    float beam_radius;        // > 0: entry points uniform on the disk of this radius around pos0
    float roulette_w, roulette_p, inv_roulette_p;
    int n_cdf;
    const float *inv_cdf;
    float hg_a, hg_b, hg_c, hg_d;   // 1 + g, 2g, 1 - g^2, 1 - g
    uint32_t key0, key1, instance, max_steps;
    uint64_t photon_offset;
    uint32_t chunk;           // ids a wave takes from its block's pool (batched: photons of a work unit)
    // Ids (work units) of the launch, those each block starts with, and the
    // least and the share (1 / 2^shift) of the rest a block claims at once.
    uint32_t n_ids, claim0, claim_min, claim_shift;
    uint32_t quiet_steps;     // a photon of fewer steps meets neither roulette nor the step cap in kQuietSteps more
    uint32_t refill_min;      // lanes not walking that trigger a round (1..64)
    int cache_bits;           // log2 of the tally-cache slots (0: no cache)
    uint32_t n_side;          // pixels of the side image (cache key offset of the transmitted image)
    int side_nx, side_ny, trans_nx, trans_ny;
    // Pixels per mm: side rows (y), side columns (z), transmitted rows (y),
    // transmitted columns (x).
    float pix_scale[4];
    unsigned long long *ws_scal;   // workspace: 16 fixed-point scalar sums, work counter at MC_S_RESERVED
    unsigned long long *ws_img;    // workspace: kCopies x n_pix fixed-point weight sums
    unsigned long long *ws_img2;   // workspace (MC_SIGMA): kCopies x n_pix squared-weight sums
    uint64_t n_pix;
    uint32_t spread;          // the image copies are permuted (spread_pixel); without the exit log
    uint32_t copy_mask;       // image copy of a wave: XCC_ID & copy_mask (kCopies - 1, or 0 for one copy)
    int32_t *rec_i;
    float *rec_f;
    double *side_wk, *side_wl;     // MC_MOMENTS: per side pixel, sum w k and sum w L
    double *side_w2k, *side_w2l;   // MC_MOMENTS_PIXEL2: per side pixel, sum w^2 k and sum w^2 L
    uint64_t rec_rows, record_stride;
    // Exit log (kOptLog): block b's entries of key range r occupy
    // log[(r * gridDim.x + b) * log_cap ...], their number (at most log_cap)
    // is log_count[r * gridDim.x + b], written when the block ends.
    unsigned long long *log;
    uint32_t *log_count;
    uint32_t log_cap, log_bits;      // log_bits: scrambled group index width, >= log_rbits
    uint32_t log_rbits;              // key ranges: 2^log_rbits
    // Batched launch: media in schedule order, work units over all of them.
    const BatchInst *insts;
    uint32_t n_inst;          // media (slots) in the launch
    uint32_t n_pix_inst;      // side + transmitted pixels of one medium (key stride)
};

constexpr double kFix = 4294967296.0;      // fixed-point scale 2^32 per unit weight

// w * 2^32 rounded to nearest, ties to even, for 0 <= w < 2^32.  The integer
// part of w and its fraction are exact in FP32, and the fraction times 2^32
// is an exact FP32 value below 2^32, so two FP32 conversions give the same
// integer as llrint((double)w * 2^32) with no FP64 arithmetic (an even
// multiple of 2^32 does not change the tie-breaking parity).  No fused
// multiply-add may absorb w's own rounding: a squared weight passed as w * w
// is the rounded FP32 product.
__device__ __forceinline__ unsigned long long fix(float w)
{
#pragma clang fp contract(off)
    const float hi = truncf(w);
    const float lo = rintf((w - hi) * 4294967296.f);
    return ((unsigned long long)(uint32_t)hi << 32) + (unsigned long long)(uint32_t)lo;
}

// The same for 0 <= w < 1 (every weight of the walk unless roulette is set
// to raise weights above 1): the integer part is 0 and w * 2^32 < 2^32.
__device__ __forceinline__ unsigned long long fix_below_one(float w)
{
    return (unsigned long long)(uint32_t)rintf(w * 4294967296.f);
}

// Pixel = floor(coord / size * n), clamped to the image (IEEE division, so a
// coordinate on a pixel edge lands where the FP64 definition puts it).  Used
// for the beam's unscattered exit pixel, where every such photon lands on
// the same point.
__device__ __forceinline__ int pixel(float coord, float size, int n)
{
    const int i = (int)floorf(coord / size * (float)n);
    return min(max(i, 0), n - 1);
}

// The same with one product by pixels per mm in place of the division, for
// the exits of scattered photons: only at a coordinate exactly on a pixel
// edge may the product round to the other side of it.
__device__ __forceinline__ int pixel_scaled(float coord, float per_mm, int n)
{
    const int i = (int)floorf(coord * per_mm);
    return min(max(i, 0), n - 1);
}

// Distances to the walls ahead along d, per axis.  With r = 1/d, the walls
// at L and at 0 lie (L - p) r and -p r ahead; for p inside the box one of the
// two is negative, so the larger is the wall the photon moves towards.  It is
// clamped at 0, so a position that rounding left a hair outside the box is
// taken back at once.  An axis with d = 0 gives r = inf and so t = inf: it is
// never hit (short of a position exactly on one of its walls, where 0 x inf
// makes the far term NaN, the maximum drops it and t is 0; the host keeps the
// source off that case).  No compare or select: three full-rate operations
// and one three-way maximum per axis.
__device__ __forceinline__ void wall_distances(float px, float py, float pz, float dx, float dy, float dz,
                                               float Lx, float Ly, float Lz, float &tx, float &ty, float &tz)
{
    const float rx = __builtin_amdgcn_rcpf(dx), ry = __builtin_amdgcn_rcpf(dy), rz = __builtin_amdgcn_rcpf(dz);
    tx = fmaxf(fmaxf((Lx - px) * rx, -px * rx), 0.f);
    ty = fmaxf(fmaxf((Ly - py) * ry, -py * ry), 0.f);
    tz = fmaxf(fmaxf((Lz - pz) * rz, -pz * rz), 0.f);
}

// The axis of the nearest wall, db = min(tx, ty, tz) (ties go to the lower
// axis).  The walk takes it only for the steps that reach a wall.
__device__ __forceinline__ int wall_axis(float db, float tx, float ty)
{
    return db == tx ? 0 : (db == ty ? 1 : 2);
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}


// Where the copies of an image of n pixels hold pixel p: every whole block of
// 4096 is permuted, so that neighbours lie 265 words apart.  Exits crowd around
// the beam, and atomics on one 64-byte line, or on lines of few L2 channels,
// wait for each other (83 million a second on one word; 24 thousand million on
// the whole card, at best and for any number of copies).  1e9 atomics around
// the centre, spread as a normal distribution of 2, 5, 10 and 40 pixels, mean
// over images of 64 x 64 to 1024 x 1024, ms: in order 146 / 79 / 69 / 55, so
// 106 / 58 / 49 / 48, blocks of 1024 116 / 60 / 49 / 48.
constexpr uint32_t kSpreadBits = 12, kSpreadMul = 265, kSpreadShift = 37;
__device__ __forceinline__ uint32_t spread_pixel(uint32_t p, uint32_t n)
{
    const uint32_t block = p >> kSpreadBits;
    const uint32_t at = (p * kSpreadMul + block * kSpreadShift) & ((1u << kSpreadBits) - 1u);
    return block < n >> kSpreadBits ? (block << kSpreadBits) | at : p;
}

constexpr uint32_t kEmpty = 0xFFFFFFFFu;   // free tally-cache slot
// Steps a wave takes at most before it looks again whether any of its photons
// could meet roulette or the step cap in as many (WalkArgs::quiet_steps).
constexpr int kQuietSteps = 32;
// A block's pool of photon ids (or work units): the next id in the low word and
// the end of its range in the high one.  A wave takes ids with one LDS add; the
// wave that finds the range used up marks the pool as being filled, claims
// ids from the global counter and publishes them, while the block's other
// waves go on with the photons they hold.  Without a range the high word is 0
// and the low one says whether the pool is being filled or closed for good.
constexpr uint32_t kPoolFilling = 0x40000000u, kPoolClosed = 0x80000000u;
__device__ __forceinline__ unsigned long long pool_range(uint32_t lo, uint32_t hi)
{
    return ((unsigned long long)hi << 32) | lo;
}
// Free path of a photon that did not end at a wall (a drawn one is positive).
constexpr float kKilled = -1.f, kCapped = -2.f;
// A free path ends inside the cuboid by a margin when each coordinate, scaled
// to [-1, 1], stays below this.  The wall distances then all exceed it, however
// they round: a coordinate p <= L (1 - 1e-5) after s d leaves (L - p0) at
// least 1e-5 L above s d, and the distance (L - p0) / d is formed to a few
// units in 2^-24.  A position closer to a wall is compared with the distance
// itself.
constexpr float kInside = 1.f - 2e-5f, kOutside = 2.f;

constexpr int kOptSigma = 1, kOptRecord = 2, kOptMoments = 4, kOptBatch = 8, kOptLog = 16;
// Exit log: image exits appended as (key << 32 | weight bits).  Keys fall
// into 2^rbits ranges; every block of the launch owns a region of log_cap
// entries in each range's part of the log and appends to it at the position a
// counter in its LDS hands out (no global atomic).  The waves of a block thus
// fill the same few lines of each range together, which stay in the L2 until
// they are whole.  Keys go to ranges by groups of eight (one 64-byte line of a
// tally copy): the group g is scrambled by p = g * kLogHashMul mod 2^bits (an
// odd multiplier, so a bijection), its top rbits bits pick the range and the
// rest, with the key's place in its group, index the key within the range.
// Bright spots of an image thus spread evenly over the ranges.  rbits grows
// with the images so that a range holds at most 2^kLogHistBits keys where the
// LDS allows (one binning block per range and copy).
constexpr uint32_t inverse_mod_2_32(uint32_t m)   // of an odd m (Newton: x <- x (2 - m x))
{
    uint32_t x = m;
    for (int i = 0; i < 5; ++i) x *= 2u - m * x;
    return x;
}
constexpr uint32_t kLogHashMul = 0x9E3779B1u;
__device__ __forceinline__ uint32_t log_scramble(uint32_t key, uint32_t bits)
{
    return ((key >> 3) * kLogHashMul) & ((1u << bits) - 1u);
}
__device__ __forceinline__ uint32_t log_bucket(uint32_t key, uint32_t bits, uint32_t rbits)
{
    return log_scramble(key, bits) >> (bits - rbits);
}
__device__ __forceinline__ uint32_t log_index(uint32_t key, uint32_t bits, uint32_t rbits)
{
    return ((log_scramble(key, bits) & ((1u << (bits - rbits)) - 1u)) << 3) | (key & 7u);
}
static_assert(kNoAllocWords == kWsScalarWords + (1ull << 21) && kNoAllocWords * 8 == MC_NOALLOC_SCRATCH_BYTES,
              "scratch holds the scalar words and 2^21 image words");
constexpr int kLdsBallistic = 15;          // LDS scalar word (per medium) counting first-step exits
constexpr int kWsBallistic = 19;           // workspace word (per medium) of that count
constexpr int kWsBeamKey = 20;             // workspace word (first medium): beam exit key + 1, or 0
constexpr int kWsLogFallback = 21;         // workspace word: exits added directly because the log was full

// Waves per SIMD a walk kernel is built for: eight (64 vector registers
// each), or six (80 each) with path moments, whose tallies would otherwise
// leave no registers for the step's constants (measured: six waves with the
// constants beat eight without by 7 %, while the plain walk loses 3 % at six).
template <int OPT>
constexpr int walk_waves_per_simd() { return (OPT & 4) ? 6 : 8; }

// The kernel's arguments, read anew from the kernel argument segment.  What
// only the rounds need is loaded there (a few scalar loads, hidden by the
// other waves) rather than held in registers across the loop: the walk is at
// its register limits, and each value kept longer spilled another.
using ArgsPtr = const __attribute__((address_space(4))) WalkArgs *;
__device__ __forceinline__ ArgsPtr reload_args()
{
    ArgsPtr p = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

template <int PHASE, int OPT>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(walk_waves_per_simd<OPT>())))
void walk_kernel(WalkArgs a)
{
    constexpr bool SIGMA = OPT & kOptSigma, RECORD = OPT & kOptRecord, MOMENTS = OPT & kOptMoments;
    constexpr bool BATCH = OPT & kOptBatch, LOG = OPT & kOptLog;
    constexpr bool PATH = RECORD || MOMENTS;   // kernels that keep each photon's path length and scatter count
    constexpr bool GLOBAL_TABLE = BATCH;   // batched: each medium's inverse table stays in global memory
    // LDS layout: inverse table (n_cdf floats, padded to 4; batched launches
    // read each medium's table from global memory instead), scalar words
    // (MC_N_SCALARS, or kBatchScal per medium; two of them hold the id pool and the
    // count of exits past the log), tally cache (slots words of
    // weight, [SIGMA] slots words of squared weight, slots uint32 keys),
    // per-wave exit queues (3 x kQueue floats, a fourth for the medium's slot),
    // with the exit log then the block's 2^log_rbits append counters.
    // (The kernel declares no static LDS: the dynamic array starts at offset 0,
    // and its 16-byte alignment keeps the 64-bit words below aligned.)
    extern __shared__ __attribute__((aligned(16))) float s_table[];
    constexpr int kQueueArrays = BATCH ? 4 : 3;
    unsigned long long *s_scal = (unsigned long long *)(s_table + (GLOBAL_TABLE ? 0 : ((a.n_cdf + 3) & ~3)));
    const int n_scal = BATCH ? (int)a.n_inst * kBatchScal : MC_N_SCALARS;
    const int slots = a.cache_bits ? 1 << a.cache_bits : 0;
    // The block's pool of photon ids (work units), see kPoolFilling.
    unsigned long long *s_pool = s_scal + kLdsPool;
    unsigned long long *s_full = s_scal + kLdsFull;   // exit log: exits that found their region full
    unsigned long long *s_cw = s_scal + n_scal;
    unsigned long long *s_cw2 = s_cw + (SIGMA ? slots : 0);
    uint32_t *s_key = (uint32_t *)(s_cw2 + slots);
    float *s_queue = (float *)(s_key + slots);
    // Exit log: entries the block has appended to each key range.
    uint32_t *s_lcnt = (uint32_t *)(s_queue + (blockDim.x >> 6) * (kQueueArrays * kQueue));
    if (LOG)
        for (int i = threadIdx.x; i < (1 << a.log_rbits); i += blockDim.x) s_lcnt[i] = 0u;

    if (PHASE == MC_PHASE_MIE && !GLOBAL_TABLE)
        for (int i = threadIdx.x; i < a.n_cdf; i += blockDim.x) s_table[i] = a.inv_cdf[i];
    for (int i = threadIdx.x; i < n_scal; i += blockDim.x)
        if (i != kLdsPool) s_scal[i] = 0ull;
    if (threadIdx.x == 0) {
        const uint64_t lo = min((uint64_t)blockIdx.x * a.claim0, (uint64_t)a.n_ids);
        const uint64_t hi = min(lo + a.claim0, (uint64_t)a.n_ids);
        *s_pool = lo < hi ? pool_range((uint32_t)lo, (uint32_t)hi) : 0ull;
    }
    for (int i = threadIdx.x; i < slots; i += blockDim.x) {
        s_cw[i] = 0ull;
        if (SIGMA) s_cw2[i] = 0ull;
        s_key[i] = kEmpty;
    }
    // Unscattered photons that leave on their first step all take the same
    // path from the source to the same pixel with the same weight w0, so the
    // walk only counts them (per medium) and the finalize pass adds count x w0
    // to that pixel.  The pixel (its key within a medium's key range) and face
    // are found here, by every thread, with the walk's own arithmetic; face -1
    // when the beam leaves through a face without an image (or through the
    // side image while its path moments are tallied).
    int beam_face = -2;   // -2: no face (it matches no photon's face, which is -1 or up)
    {
        float tx, ty, tz;
        wall_distances(a.pos0[0], a.pos0[1], a.pos0[2], a.dir0[0], a.dir0[1], a.dir0[2], a.size[0], a.size[1],
                       a.size[2], tx, ty, tz);
        const float db = fminf(fminf(tx, ty), tz);
        const int ax = wall_axis(db, tx, ty);
        const float bx = fmaf(db, a.dir0[0], a.pos0[0]), by = fmaf(db, a.dir0[1], a.pos0[1]);
        const float bz = fmaf(db, a.dir0[2], a.pos0[2]);
        const float da = ax == 0 ? a.dir0[0] : (ax == 1 ? a.dir0[1] : a.dir0[2]);
        int face = -2;
        uint32_t key = 0;
        if (da > 0.f && (ax == 0 || ax == 2) && !(MOMENTS && ax == 0) && !(a.beam_radius > 0.f)) {
            face = 2 * ax + 1;
            key = ax == 0 ? (uint32_t)(pixel(by, a.size[1], a.side_ny) * a.side_nx + pixel(bz, a.size[2], a.side_nx))
                          : a.n_side + (uint32_t)(pixel(by, a.size[1], a.trans_ny) * a.trans_nx +
                                                  pixel(bx, a.size[0], a.trans_nx));
            if (blockIdx.x == 0 && threadIdx.x == 0) a.ws_scal[kWsBeamKey] = (unsigned long long)key + 1ull;
        }
        beam_face = face;
    }
    // Every wave reads the whole table and adds into the scalars, cache and
    // log cursors set up above by the block's threads together.
    __syncthreads();

    const int lane = __lane_id();
    const uint32_t xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & a.copy_mask;   // hwreg(HW_REG_XCC_ID, 0, 4)
    auto my_img = [&]() { const ArgsPtr ra = reload_args(); return ra->ws_img + (uint64_t)xcc * ra->n_pix; };
    auto my_img2 = [&]() { const ArgsPtr ra = reload_args(); return ra->ws_img2 + (uint64_t)xcc * ra->n_pix; };
    float *q_y = s_queue + (threadIdx.x >> 6) * (kQueueArrays * kQueue);
    float *q_b = q_y + kQueue;
    float *q_w = q_b + kQueue;                 // weight bits, bit 31 set for the side image
    float *q_s = q_w + kQueue;                 // batched: the medium's slot (uint32 bits)
    uint32_t q_n = 0;                          // wave-uniform queue fill

    // Tally the first n queued exits, one per lane: pixel key, then the LDS
    // cache (claim or hit, up to four linear probes) or, when every probed
    // slot holds another pixel, a global atomic.  With the exit log the exits
    // are appended to the log instead, until their range's region is full.
    // What comes after that is mostly the few pixels that filled the region, so
    // the cache takes nearly all of it (with global atomics alone, on pixels and
    // a counter that all blocks share, 1e8 photons at optical depth 1 took
    // 22.4 ms at 64 x 64 and 3.46 ms at 1024 x 1024; now 1.34 and 1.25).
    auto flush = [&](uint32_t n) {
        const ArgsPtr ra = reload_args();
        __builtin_amdgcn_wave_barrier();
        const bool act = (uint32_t)lane < n;
        uint32_t key = 0;
        float wf = 0.f;
        unsigned long long wq = 0ull, wq2 = 0ull;
        if (act) {
            const float y = q_y[lane], b = q_b[lane];
            const uint32_t wb = __float_as_uint(q_w[lane]);
            const bool side = wb >> 31;
            wf = __uint_as_float(wb & 0x7FFFFFFFu);
            const uint32_t key_base = BATCH ? __float_as_uint(q_s[lane]) * ra->n_pix_inst : 0u;
            // (Held in scalar registers: a select between two arguments would
            // become a vector load from the selected address.)
            float scale[4] = {ra->pix_scale[0], ra->pix_scale[1], ra->pix_scale[2], ra->pix_scale[3]};
            int dim[4] = {ra->side_ny, ra->side_nx, ra->trans_ny, ra->trans_nx};
            asm volatile("" : "+s"(scale[0]), "+s"(scale[1]), "+s"(scale[2]), "+s"(scale[3]));
            asm volatile("" : "+s"(dim[0]), "+s"(dim[1]), "+s"(dim[2]), "+s"(dim[3]));
            const float per_row = side ? scale[0] : scale[2], per_col = side ? scale[1] : scale[3];
            const int n_row = side ? dim[0] : dim[2], n_col = side ? dim[1] : dim[3];
            const uint32_t pix = (uint32_t)(pixel_scaled(y, per_row, n_row) * n_col + pixel_scaled(b, per_col, n_col));
            key = key_base + (side ? 0u : ra->n_side);
            if (LOG) key += pix;
            else key += spread_pixel(pix, ra->spread ? (side ? ra->n_side : ra->n_pix_inst - ra->n_side) : 0u);
        }
        bool to_image = act;
        if (LOG) {
            // Append to the block's region of the key's range at the position
            // the block's LDS counter hands out.
            const uint32_t bucket = log_bucket(key, ra->log_bits, ra->log_rbits);
            if (act) {
                const uint32_t e = atomicAdd(&s_lcnt[bucket], 1u);
                if (e < ra->log_cap) {
                    ra->log[(uint64_t)(bucket * gridDim.x + blockIdx.x) * ra->log_cap + e] =
                        ((unsigned long long)key << 32) | __float_as_uint(wf);
                    to_image = false;
                }
            }
        }
        if (to_image) {
            wq = fix(wf);
            wq2 = SIGMA ? fix(wf * wf) : 0ull;
            if (LOG) atomicAdd(s_full, 1ull);
            bool cached = false;
            if (slots) {
                uint32_t slot = (key * 2654435761u) >> (32 - ra->cache_bits);
                for (int probe = 0; probe < 4 && !cached; ++probe) {
                    const uint32_t old = atomicCAS(&s_key[slot], kEmpty, key);
                    if (old == kEmpty || old == key) {
                        atomicAdd(&s_cw[slot], wq);
                        if (SIGMA) atomicAdd(&s_cw2[slot], wq2);
                        cached = true;
                    }
                    slot = (slot + 1) & (uint32_t)(slots - 1);
                }
            }
            if (!cached) {
                atomicAdd(my_img() + key, wq);
                if (SIGMA) atomicAdd(my_img2() + key, wq2);
            }
        }
        __builtin_amdgcn_wave_barrier();
    };

    const float tab_scale = (float)(a.n_cdf - 1);

    // Wave-uniform id range: next id and ids left in the claimed chunk.
    uint64_t q_next = 0;
    uint32_t q_rem = 0;
    bool exhausted = false;
    // Take up to `want` ids from the block's pool, filling it from the global
    // counter when it is empty (one lane calls this).  Returns the ids taken,
    // first in *base, or 0: *done says whether any may still come.
    auto take_ids = [&](ArgsPtr ra, uint32_t want, uint32_t *base, bool *done) -> uint32_t {
        *done = false;
        unsigned long long v = __hip_atomic_load(s_pool, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((uint32_t)v < (uint32_t)(v >> 32)) {
            v = atomicAdd(s_pool, (unsigned long long)want);
            const uint32_t next = (uint32_t)v, end = (uint32_t)(v >> 32);
            if (next < end) {
                *base = next;
                return min(want, end - next);
            }
            v += want;
        }
        const uint32_t end = (uint32_t)(v >> 32);
        if (end == 0u && (uint32_t)v >= kPoolFilling) {
            *done = (uint32_t)v >= kPoolClosed;
            return 0u;
        }
        if (atomicCAS(s_pool, v, (unsigned long long)kPoolFilling) != v) return 0u;
        const uint32_t n = ra->n_ids;
        const uint64_t first = (uint64_t)gridDim.x * ra->claim0;   // ids the blocks started with
        uint64_t g = n;
        uint32_t size = 0;
        if (first < n) {
            size = max((n - max(end, (uint32_t)first)) >> ra->claim_shift, ra->claim_min);
            g = first + atomicAdd(ra->ws_scal + MC_S_RESERVED, (unsigned long long)size);
        }
        if (g >= n) {
            __hip_atomic_store(s_pool, (unsigned long long)kPoolClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            *done = true;
            return 0u;
        }
        const uint32_t lo = (uint32_t)g, hi = (uint32_t)min(g + size, (uint64_t)n), got = min(want, hi - lo);
        __hip_atomic_store(s_pool, pool_range(lo + got, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        *base = lo;
        return got;
    };

    // Lane state.  A lane walks while its photon's last step ended inside the
    // cuboid (out < kInside, see there; the wave-uniform mask of these lanes
    // is `alive`), holds no photon (`empty`), or waits for a round with a
    // photon whose step met a wall, or that roulette killed (s = kKilled) or
    // the step cap stopped (s = kCapped).
    uint64_t alive = 0ull, empty = ~0ull;
    float out = kOutside;
    // Steps the wave may still take before it has to look again whether one of
    // its photons could meet roulette or the step cap (0 or less: some could now).
    // It counts down in every step and starts anew at the rounds (calm_at_round).
    int calm = 0;
    uint64_t id = 0;
    PhotonKey pk{};
    float px = 0.f, py = 0.f, pz = 0.f, dx = 0.f, dy = 0.f, dz = 1.f;
    float w = 0.f, L = 0.f, A = 0.f, s = 0.f;
    uint32_t k = 0, step = 0, r3 = 0;
    // Lane accumulators (interactions are steps less wall hits).
    unsigned long long acc_abs = 0ull;
    uint32_t acc_hits = 0, acc_steps = 0, acc_photons = 0, acc_ball = 0;
    double acc_w2 = 0.0, acc_w2k = 0.0, acc_w2l = 0.0;   // MOMENTS: image-wide second moments
    // The medium of the lane's photon (batched launches change it per photon;
    // otherwise these stay the launch's values).
    uint32_t l_slot = kEmpty, q_p = 0;
    float l_mu = a.neg_ln2_over_mu, l_alb = a.albedo, l_abs = a.absorb;
    // FP32 operations with a scalar-register operand issue at half the rate
    // of those whose operands are all vector registers; the constants of the
    // step therefore live in vector registers (the empty asm hides that they
    // are wave-uniform; batched media keep theirs per lane anyway).
    float v_sx = 2.f / a.size[0], v_sy = 2.f / a.size[1], v_sz = 2.f / a.size[2], v_tab = tab_scale;
    asm volatile("" : "+v"(l_mu), "+v"(l_alb), "+v"(l_abs));
    asm volatile("" : "+v"(v_sx), "+v"(v_sy), "+v"(v_sz), "+v"(v_tab));
    float v_ha = a.hg_a, v_hb = a.hg_b, v_hc = a.hg_c, v_hd = a.hg_d;
    if (PHASE == MC_PHASE_HG) asm volatile("" : "+v"(v_ha), "+v"(v_hb), "+v"(v_hc), "+v"(v_hd));
    const float *l_tab = a.inv_cdf;
    // Batched: move the lane accumulators into the LDS scalars of its medium.
    auto flush_lane = [&]() {
        unsigned long long *sc = s_scal + l_slot * kBatchScal;
        atomicAdd(&sc[MC_S_ABSORBED], acc_abs);
        atomicAdd(&sc[MC_S_EVENTS], (unsigned long long)acc_steps - (unsigned long long)acc_hits);
        atomicAdd(&sc[MC_S_STEPS], (unsigned long long)acc_steps);
        atomicAdd(&sc[MC_S_PHOTONS], (unsigned long long)acc_photons);
        if (acc_ball) atomicAdd(&sc[kLdsBallistic], (unsigned long long)acc_ball);
        acc_abs = 0ull;
        acc_hits = acc_steps = acc_photons = acc_ball = 0;
    };
    // The round keys derive from the seed at each block (scalar adds) rather
    // than living in 20 scalar registers across the loop.
    auto draw = [&](uint32_t at) {
        uint32_t k0 = a.key0, k1 = a.key1;
        asm volatile("" : "+s"(k0), "+s"(k1));
        return philox_step(pk, at, k0, k1);
    };
    // An interaction after the free path s, from random words w1, w2 and r3:
    // move, absorb (Eq. 16), scatter; where the wave is not calm, roulette and
    // the step cap too.  (The empty asm keeps that block behind its scalar
    // branch.  A photon that ended there scatters all the same, unless its
    // direction is recorded.)
    auto interact = [&](uint32_t w1, uint32_t w2) {
        px = fmaf(s, dx, px); py = fmaf(s, dy, py); pz = fmaf(s, dz, pz);
        if (PATH) {
            L += s;
            ++k;
        }
        A = fmaf(w, l_abs, A);
        asm volatile("" : "+v"(A), "+v"(w));   // A first: w is then updated in place
        w *= l_alb;
        if (calm <= 0) {
            asm volatile("");
            const uint32_t scal_at = BATCH ? l_slot * kBatchScal : 0u;   // the medium's LDS scalars
            if (w < a.roulette_w) {
                if (uniform01(r3) < a.roulette_p) {
                    const float wn = w * a.inv_roulette_p;
                    atomicAdd(&s_scal[scal_at + MC_S_ROULETTE_NET], fix(wn) - fix(w));
                    w = wn;
                } else {
                    atomicAdd(&s_scal[scal_at + MC_S_ROULETTE_NET], 0ull - fix(w));
                    atomicAdd(&s_scal[scal_at + MC_S_ROULETTE_KILLS], 1ull);
                    w = 0.f;
                    s = kKilled;
                    out = kOutside;
                }
            }
            if (s >= 0.f && step >= a.max_steps) {
                s = kCapped;
                out = kOutside;
            }
        }
        if (RECORD && s == kKilled) return;
        const float u1 = uniform01(w1), u2 = uniform01(w2);
        float v;
        if (PHASE == MC_PHASE_MIE) {
            // u1 <= 1 - 2^-24, so u1 (n - 1) rounds below n - 1 (exact when
            // n - 1 is a power of two, else more than half an ulp short of
            // it): i <= n - 2 and entry i + 1 exists.
            const float tt = u1 * v_tab;
            const int i = (int)tt;
            // The fraction from the unrounded product u1 (n - 1).
            const float f = fmaf(u1, v_tab, -(float)i);
            const float t0 = GLOBAL_TABLE ? l_tab[i] : s_table[i];
            const float t1 = GLOBAL_TABLE ? l_tab[i + 1] : s_table[i + 1];
            v = fmaf(f, t1 - t0, t0);
        } else {
            const float D = fmaf(-v_hb, u1, v_ha);
            const float rD = __builtin_amdgcn_rcpf(D);
            v = v_hd * u1 * fmaf(v_hc, rD, v_hd) * rD;
        }
        const float ct = 1.f - v;
        // A table value lies in [0, 2], and so does a rounded point between
        // two of them: v (2 - v) >= 0.  The HG formula can overshoot 2.
        const float st = __builtin_amdgcn_sqrtf(PHASE == MC_PHASE_MIE ? v * (2.f - v)
                                                                      : fmaxf(v * (2.f - v), 0.f));
        const float cp = __builtin_amdgcn_cosf(u2);        // cos(2 pi u2)
        const float sp = __builtin_amdgcn_sinf(u2);        // sin(2 pi u2)
        // Orthonormal basis around d (Duff et al. 2017), with its factors
        // sign(dz) = +-1 drawn together: sin phi takes it here and the new dz
        // below (products with +-1 are exact, so the bits are those of the
        // basis written out).
        uint32_t sz = __float_as_uint(dz) & 0x80000000u;
        asm volatile("" : "+v"(sz));   // one AND and two XORs at full rate, not two three-input operations at half
        const float ia = __builtin_amdgcn_rcpf(1.f + fabsf(dz));
        const float b = dx * dy * ia;
        const float e1 = fmaf(dx * dx, -ia, 1.f), e2 = fmaf(dy * dy, -ia, 1.f);
        const float sq = __uint_as_float(__float_as_uint(sp) ^ sz);
        const float qx = fmaf(cp, e1, -(sq * b)), qy = fmaf(-cp, b, sq * e2), qz = fmaf(cp, dx, sq * dy);
        const float nx = fmaf(ct, dx, st * qx), ny = fmaf(ct, dy, st * qy), nz = fmaf(ct, fabsf(dz), -(st * qz));
        // |n|^2 is 1 up to rounding, so one Newton step of 1/sqrt from 1
        // (1.5 - |n|^2 / 2) renormalises to within 1e-13.
        const float inv = fmaf(-0.5f, fmaf(nx, nx, fmaf(ny, ny, nz * nz)), 1.5f);
        dx = nx * inv; dy = ny * inv; dz = __uint_as_float(__float_as_uint(nz * inv) ^ sz);
    };

    // A lane whose photon meets a wall or ends keeps its state until a round
    // handles several such lanes at once: when at least refill_min lanes do
    // not walk (refill_min <= 64, so also when none does).  Only some lanes
    // leave the interior in any one step, so resolving walls, tallying and
    // refilling every step would run all that with most lanes masked off.
    // Once the photon ids are used up no lane can be refilled, and a round
    // runs when refill_min lanes wait or at least as many wait as walk.
    // Either way it runs when at most round_at lanes walk.
    uint32_t round_at = 64u;

    // The loop begins 12 (with the log) or 20 bytes past a multiple of 32, whatever
    // comes before it: instructions are fetched in aligned lines, and where the loop
    // lies in them moves times by 2 % and the end of some launches by 5 % (0 / 8 / 12 /
    // 16 / 20 / 24 bytes past: 1e5 photons, without the log, 42.9 / 42.0 / 41.9 / 41.8 / 41.6 /
    // 41.7 us; tau = 16 with it, nine counts from 3e6 to 3.3e7, geometric mean relative to
    // the first 1 / 1.003 / 1.004 / 1.017 / 1.020 / 1.008; 1e8 at tau = 1 1 / 0.992 / 0.990 / 0.993 /
    // 0.992 / 0.992).
    if (LOG) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    else asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    for (;;) {
        if ((uint32_t)__popcll(alive) <= round_at) {
            const ArgsPtr ra = reload_args();
            const bool waits = __builtin_amdgcn_inverse_ballot_w64(~(alive | empty));
            const float v_lx = ra->size[0], v_ly = ra->size[1], v_lz = ra->size[2];
            const float v_n21 = ra->n21, v_n12sq = ra->n12sq, v_fresnel = ra->fresnel;
            // ---- walls: the photons that left the interior ----------------------
            int face = -1, axis = 0;
            bool again = false, early = false;
            if (waits && s >= 0.f) {
                // Nearest wall along the direction.
                float tx, ty, tz;
                wall_distances(px, py, pz, dx, dy, dz, v_lx, v_ly, v_lz, tx, ty, tz);
                const float db = fminf(fminf(tx, ty), tz);
                early = !(s >= db);   // within the margin of a wall, but short of it
                if (!early) {
                    // Boundary: clamp into the box (a move that overshot the wall
                    // by rounding lands on it), then reflect (u3 < R) or leave.
                    // Written as selects so the wave runs it without branches.
                    px = fmaf(db, dx, px); py = fmaf(db, dy, py); pz = fmaf(db, dz, pz);
                    if (PATH) L += db;
                    ++acc_hits;
                    axis = wall_axis(db, tx, ty);
                    const bool on_x = axis == 0, on_y = axis == 1, on_z = axis == 2;
                    const float da = on_x ? dx : (on_y ? dy : dz);
                    const bool pos_side = da > 0.f;
                    px = __builtin_amdgcn_fmed3f(px, 0.f, v_lx);
                    py = __builtin_amdgcn_fmed3f(py, 0.f, v_ly);
                    pz = __builtin_amdgcn_fmed3f(pz, 0.f, v_lz);
                    // Index-matched walls reflect nothing: R is scaled by 0 there.
                    const float ci = fabsf(da);
                    const float st2 = v_n12sq * fmaf(-ci, ci, 1.f);
                    // 1 - st2 > 0 wherever R uses ct; under TIR the select drops it.
                    const float ct = __builtin_amdgcn_sqrtf(1.f - st2);
                    const float ds = fmaf(v_n21, ct, ci), dp = fmaf(v_n21, ci, ct);   // both > 0 (ci > 0)
                    const float r = __builtin_amdgcn_rcpf(ds * dp);
                    const float rs = fmaf(-v_n21, ct, ci) * dp * r;
                    const float rp = fmaf(v_n21, ci, -ct) * ds * r;
                    const float R = v_fresnel * (st2 >= 1.f ? 1.f : 0.5f * fmaf(rs, rs, rp * rp));
                    const bool refl = uniform01(r3) < R;
                    dx = refl && on_x ? -dx : dx;
                    dy = refl && on_y ? -dy : dy;
                    dz = refl && on_z ? -dz : dz;
                    again = refl && step < ra->max_steps;
                    if (refl && !again) s = kCapped;
                    face = refl ? -1 : 2 * axis + (pos_side ? 1 : 0);
                }
            }
            // Rare: the step stayed inside after all and interacts.
            calm = calm_at_round(calm, __builtin_amdgcn_ballot_w64(early) != 0ull);
            if (early) {
                const Block4 r = draw(step - 1u);
                interact(r.r1, r.r2);
                again = s >= 0.f;
            }
            if (again) out = 0.f;
            // ---- end-of-photon work --------------------------------------------
            const uint64_t go_on = __builtin_amdgcn_ballot_w64(again);
            const bool pending = waits && !again;
            if (pending) {
                const uint32_t scal_at = BATCH ? l_slot * kBatchScal : 0u;
                if (s == kCapped) {
                    atomicAdd(&s_scal[scal_at + MC_S_CAPPED_W], fix(w));
                    atomicAdd(&s_scal[scal_at + MC_S_CAPPED], 1ull);
                }
                // Faces +x and +z are totalled from their images when finalizing.
                const bool below_one = __builtin_amdgcn_ballot_w64(max(__float_as_uint(w), __float_as_uint(A)) >= 0x3F800000u) == 0;   // wave-uniform
                if (face >= 0 && (face | 4) != 5)
                    atomicAdd(&s_scal[scal_at + MC_S_FACE + face], below_one ? fix_below_one(w) : fix(w));
                if (MOMENTS && face == 1) {
                    // Path moments of the side image (perturbation Monte Carlo):
                    // first order per pixel, second order summed over the image
                    // in lane registers (per pixel as well when asked for).
                    const uint32_t key = (uint32_t)(pixel_scaled(py, ra->pix_scale[0], ra->side_ny) * ra->side_nx +
                                                    pixel_scaled(pz, ra->pix_scale[1], ra->side_nx));
                    const double wd = (double)w, wk = wd * (double)k, wl = wd * (double)L;
                    atomicAdd(ra->side_wk + key, wk);
                    atomicAdd(ra->side_wl + key, wl);
                    acc_w2 += wd * wd;
                    acc_w2k += wd * wk;
                    acc_w2l += wd * wl;
                    if (ra->side_w2k) {
                        atomicAdd(ra->side_w2k + key, wd * wk);
                        atomicAdd(ra->side_w2l + key, wd * wl);
                    }
                }
                acc_abs += below_one ? fix_below_one(A) : fix(A);
                acc_steps += step;
                ++acc_photons;
                if (RECORD) {
                    const uint64_t rel = id - ra->photon_offset;
                    if (rel % ra->record_stride == 0 && rel / ra->record_stride < ra->rec_rows) {
                        const uint64_t row = rel / ra->record_stride, n = ra->rec_rows;
                        float ox = dx, oy = dy, oz = dz;
                        if (s >= 0.f && !ra->matched) {
                            // Refracted direction outside the wall (Snell).
                            ox *= ra->n12; oy *= ra->n12; oz *= ra->n12;
                            const float t2 = (axis == 0 ? oy * oy + oz * oz
                                                        : (axis == 1 ? ox * ox + oz * oz : ox * ox + oy * oy));
                            const float on = copysignf(sqrtf(fmaxf(1.f - t2, 0.f)),
                                                       axis == 0 ? dx : (axis == 1 ? dy : dz));
                            if (axis == 0) ox = on; else if (axis == 1) oy = on; else oz = on;
                        }
                        ra->rec_i[MC_REC_I_FACE * n + row] = face;
                        ra->rec_i[MC_REC_I_CAUSE * n + row] = s >= 0.f ? 0 : (s == kKilled ? 1 : 2);
                        ra->rec_i[MC_REC_I_K * n + row] = (int32_t)k;
                        ra->rec_i[MC_REC_I_STEPS * n + row] = (int32_t)step;
                        ra->rec_f[(MC_REC_F_POS + 0) * n + row] = px;
                        ra->rec_f[(MC_REC_F_POS + 1) * n + row] = py;
                        ra->rec_f[(MC_REC_F_POS + 2) * n + row] = pz;
                        ra->rec_f[(MC_REC_F_DIR + 0) * n + row] = ox;
                        ra->rec_f[(MC_REC_F_DIR + 1) * n + row] = oy;
                        ra->rec_f[(MC_REC_F_DIR + 2) * n + row] = oz;
                        ra->rec_f[MC_REC_F_W * n + row] = w;
                        ra->rec_f[MC_REC_F_L * n + row] = L;
                        ra->rec_f[MC_REC_F_A * n + row] = A;
                    }
                }
            }
            // ---- queue exits through the imaged faces (+x side, +z transmitted) ----
            // An exit face (0..5) belongs to a photon that left through it.  A
            // photon that leaves on its first step met a wall before any
            // interaction, so leaving through the beam's own exit face at step
            // 1 makes it an unscattered first-step exit.
            const bool ballistic = pending && step == 1 && face == beam_face;
            acc_ball += ballistic ? 1u : 0u;
            const bool to_img = (face | 4) == 5 && !ballistic;
            const uint64_t m = __builtin_amdgcn_ballot_w64(to_img);
            if (m) {
                const uint32_t n_push = __popcll(m);
                if (q_n + n_push > (uint32_t)kQueue) {
                    flush(q_n);
                    q_n = 0;
                }
                if (to_img) {
                    const uint32_t at = q_n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    q_y[at] = py;
                    q_b[at] = face == 1 ? pz : px;
                    q_w[at] = __uint_as_float(__float_as_uint(w) | (face == 1 ? 0x80000000u : 0u));
                    if (BATCH) q_s[at] = __uint_as_float(l_slot);
                }
                q_n += n_push;
            }

            // Lane counters stay below 2^31: steps bound the others, and a
            // photon adds at most max_steps <= 2^24.  Past 2^31 they move into
            // the 64-bit LDS words (batched: of the lane's medium).  (Hits of
            // a photon still walking are counted before its steps; the sums
            // are modulo 2^64, so the difference comes out right at the end.)
            if (__builtin_amdgcn_ballot_w64(acc_steps >= 0x80000000u)) {
                if (BATCH) {
                    if (acc_steps >= 0x80000000u) flush_lane();
                } else {
                    atomicAdd(&s_scal[MC_S_EVENTS], (unsigned long long)acc_steps - (unsigned long long)acc_hits);
                    atomicAdd(&s_scal[MC_S_STEPS], (unsigned long long)acc_steps);
                    atomicAdd(&s_scal[MC_S_PHOTONS], (unsigned long long)acc_photons);
                    atomicAdd(&s_scal[kLdsBallistic], (unsigned long long)acc_ball);
                    acc_hits = acc_steps = acc_photons = acc_ball = 0;
                }
            }

            // ---- refill free lanes ---------------------------------------------
            alive |= go_on;
            const uint64_t need = ~alive;
            if (q_rem == 0 && !exhausted && need) {
                // Single medium: take the next `chunk` photon ids.  Batched:
                // the next work unit, `chunk` photons of one medium.
                uint32_t base = 0, got = 0;
                bool done = false;
                if (lane == 0) got = take_ids(ra, BATCH ? 1u : ra->chunk, &base, &done);
                base = __builtin_amdgcn_readfirstlane(base);
                got = __builtin_amdgcn_readfirstlane(got);
                exhausted = __builtin_amdgcn_readfirstlane((uint32_t)done) != 0u;
                if (!BATCH) {
                    q_next = base;
                    q_rem = got;
                } else if (got) {
                    // The unit's medium: the last one whose first unit is <= base
                    // (media without photons own no units and are never found).
                    uint32_t l = 0, h = ra->n_inst;
                    while (h - l > 1) {
                        const uint32_t mid = (l + h) >> 1;
                        if (ra->insts[mid].unit_begin <= base) l = mid; else h = mid;
                    }
                    q_p = l;
                    q_next = (base - ra->insts[l].unit_begin) * ra->chunk;
                    q_rem = (uint32_t)min((uint64_t)ra->chunk, ra->insts[l].n_photons - q_next);
                }
            }
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
            const bool starts = __builtin_amdgcn_inverse_ballot_w64(need) && rank < q_rem;
            if (starts) {
                const uint64_t new_id = (BATCH ? 0ull : ra->photon_offset) + q_next + rank;
                if (RECORD) id = new_id;
                uint32_t ctr = ra->instance;
                if (BATCH) {
                    const BatchInst &bi = ra->insts[q_p];
                    ctr = bi.counter;
                    if (bi.slot != l_slot) {
                        if (l_slot != kEmpty) flush_lane();
                        l_slot = bi.slot;
                        l_mu = bi.neg_ln2_over_mu;
                        l_alb = bi.albedo;
                        l_abs = bi.absorb;
                        l_tab = bi.inv_cdf;
                    }
                }
                pk = photon_key(ctr, new_id, ra->key0, ra->key1);
                px = ra->pos0[0];
                py = ra->pos0[1];
                pz = ra->pos0[2];
                if (ra->beam_radius > 0.f) {
                    // Finite beam: entry point uniform on the disk, from the
                    // photon's Philox block at the reserved step counter.
                    const Block4 rb = draw(0xFFFFFFFFu);
                    const float rho = ra->beam_radius * __builtin_amdgcn_sqrtf(uniform01(rb.r0));
                    const float u1 = uniform01(rb.r1);
                    px = fmaf(rho, __builtin_amdgcn_cosf(u1), px);    // cos(2 pi u1)
                    py = fmaf(rho, __builtin_amdgcn_sinf(u1), py);    // sin(2 pi u1)
                }
                dx = ra->dir0[0];
                dy = ra->dir0[1];
                dz = ra->dir0[2];
                w = ra->w0;
                A = 0.f; out = 0.f; step = 0;
                if (PATH) { L = 0.f; k = 0; }
            }
            const uint32_t took = min((uint32_t)__popcll(need), q_rem);
            q_next += took;
            q_rem -= took;
            alive |= __builtin_amdgcn_ballot_w64(starts);
            empty = ~alive;
            const uint32_t n_alive = (uint32_t)__popcll(alive), n_idle = ra->refill_min;
            // (Without a walking lane but not exhausted: another wave of the block
            // is filling the pool, and the next round looks again.)
            if (n_alive == 0u && exhausted) break;
            round_at = exhausted ? max(n_alive / 2u, n_alive - min(n_alive, n_idle)) : 64u - n_idle;
            if (!starts && !again) out = kOutside;
        }

        // ---- one step of the walking lanes ----------------------------------
        if (calm <= 0 && __builtin_amdgcn_ballot_w64(step >= a.quiet_steps) == 0ull) calm = kQuietSteps;
        if (__builtin_amdgcn_inverse_ballot_w64(alive)) {
            const Block4 r = draw(step);
            r3 = r.r3;
            s = __builtin_amdgcn_logf(uniform01(r.r0)) * l_mu;     // Eq. 15
            ++step;
            // Still inside the cuboid, by a margin, at the end of the free
            // path?  Then no wall is nearer (kInside).
            const float ex = fmaf(fmaf(s, dx, px), v_sx, -1.f), ey = fmaf(fmaf(s, dy, py), v_sy, -1.f);
            const float ez = fmaf(fmaf(s, dz, pz), v_sz, -1.f);
            out = fmaxf(fmaxf(fabsf(ex), fabsf(ey)), fabsf(ez));
            if (out < kInside) interact(r.r1, r.r2);
        }
        alive = __builtin_amdgcn_ballot_w64(out < kInside);
        --calm;
    }
    flush(q_n);

    // ---- block-level flush of the scalar tallies and the cache ---------------
    if (BATCH) {
        if (l_slot != kEmpty) flush_lane();
        __syncthreads();
        for (int i = threadIdx.x; i < n_scal; i += blockDim.x) {
            const int j = i % kBatchScal;
            const unsigned long long v = s_scal[i];
            if (v != 0ull && i != kLdsPool && i != kLdsFull && (j < MC_S_RESERVED || j == kLdsBallistic))
                atomicAdd(&a.ws_scal[(uint64_t)(i / kBatchScal) * kWsScalarWords +
                                     (j == kLdsBallistic ? kWsBallistic : j)], v);
        }
    } else {
        const unsigned long long wabs = wave_sum(acc_abs);
        // Lane counters are below 2^32; their wave sums are taken in 64 bits.
        const unsigned long long wev = wave_sum((unsigned long long)acc_steps - (unsigned long long)acc_hits);
        const unsigned long long wst = wave_sum((unsigned long long)acc_steps);
        const unsigned long long wph = wave_sum((unsigned long long)acc_photons);
        const unsigned long long wbl = wave_sum((unsigned long long)acc_ball);
        if (lane == 0) {
            if (wbl) atomicAdd(&s_scal[kLdsBallistic], wbl);
            atomicAdd(&s_scal[MC_S_ABSORBED], wabs);
            atomicAdd(&s_scal[MC_S_EVENTS], wev);
            atomicAdd(&s_scal[MC_S_STEPS], wst);
            atomicAdd(&s_scal[MC_S_PHOTONS], wph);
        }
        if (MOMENTS) {
            const double m0 = wave_sum(acc_w2), m1 = wave_sum(acc_w2k), m2 = wave_sum(acc_w2l);
            if (lane == 0) {
                double *s_m2 = (double *)(s_scal + MC_S_SIDE_W2);
                atomicAdd(s_m2 + 0, m0);
                atomicAdd(s_m2 + 1, m1);
                atomicAdd(s_m2 + 2, m2);
            }
        }
        __syncthreads();
        if (threadIdx.x < MC_S_RESERVED) {
            const unsigned long long v = s_scal[threadIdx.x];
            if (v != 0ull && threadIdx.x != kLdsPool && threadIdx.x != kLdsFull) atomicAdd(&a.ws_scal[threadIdx.x], v);
        } else if (threadIdx.x == kLdsBallistic) {
            const unsigned long long v = s_scal[kLdsBallistic];
            if (v != 0ull) atomicAdd(&a.ws_scal[kWsBallistic], v);
        } else if (MOMENTS && threadIdx.x >= MC_S_SIDE_W2 && threadIdx.x <= MC_S_SIDE_W2L) {
            const double v = __longlong_as_double((long long)s_scal[threadIdx.x]);
            if (v != 0.0) atomicAdd((double *)&a.ws_scal[threadIdx.x], v);
        }
    }
    if (LOG && threadIdx.x == 0 && *s_full != 0ull) atomicAdd(a.ws_scal + kWsLogFallback, *s_full);
    for (int i = threadIdx.x; i < slots; i += blockDim.x) {
        const uint32_t key = s_key[i];
        if (key == kEmpty) continue;
        atomicAdd(my_img() + key, s_cw[i]);
        if (SIGMA) atomicAdd(my_img2() + key, s_cw2[i]);
    }
    // The block's entries in each range of the exit log (all its waves have
    // appended: the barrier above).
    if (LOG)
        for (int i = threadIdx.x; i < (1 << a.log_rbits); i += blockDim.x)
            a.log_count[i * gridDim.x + blockIdx.x] = min(s_lcnt[i], a.log_cap);
}

// Zero the workspace words [0, n_ws) and [ws2, ws2 + n_ws2) and, unless
// accumulating, the outputs that the walk itself writes (path moments, records);
// the finalize writes the others whole.  (A fill kernel, not memset, so the
// sequence stays valid under stream capture.)
__global__ void init_kernel(unsigned long long *ws, size_t n_ws, unsigned long long *ws2, size_t n_ws2, size_t n_side,
                            int32_t *rec_i, float *rec_f, size_t n_rec, double *side_wk, double *side_wl,
                            double *side_w2k, double *side_w2l, int zero_all)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = t0; i < n_ws; i += stride) ws[i] = 0ull;
    for (size_t i = t0; i < n_ws2; i += stride) ws2[i] = 0ull;
    if (!zero_all) return;
    if (side_wk)
        for (size_t i = t0; i < n_side; i += stride) {
            side_wk[i] = 0.0;
            side_wl[i] = 0.0;
            if (side_w2k) {
                side_w2k[i] = 0.0;
                side_w2l[i] = 0.0;
            }
        }
    for (size_t i = t0; i < (size_t)MC_REC_I_N * n_rec; i += stride) rec_i[i] = (i / n_rec == MC_REC_I_FACE) ? -1 : 0;
    for (size_t i = t0; i < (size_t)MC_REC_F_N * n_rec; i += stride) rec_f[i] = 0.f;
}

// Sum the exit log into the image copies.  Block (range b, part p, copy s)
// takes the regions of range b that every n_copies-th of the walk's blocks,
// from block s, wrote (log_count entries each), adds the fixed-point weights (and
// squared weights) of the entries whose index within the range lies in part
// p into an LDS histogram of 2^kLogHistBits sums, then writes the sums into
// copy s.  The first n_cleared copies (copy 0, or all) also hold the walk's
// fallback atomics (exits that found their region full), so they were cleared
// and take the non-zero sums as adds; the other copies were not cleared and
// take every key's sum as a store (the blocks of copy s cover each of its keys
// exactly once).  No
// other writer touches those keys now, so plain loads and stores do.  The
// sums are of the same fix() values the walk would have added, so the
// images equal those of the atomic path bit for bit.
template <bool SIGMA>
__global__ __launch_bounds__(1024) void log_bin(const unsigned long long *log, const uint32_t *count, uint32_t cap,
                                                uint32_t walk_blocks, unsigned long long *copies,
                                                unsigned long long *copies2, uint32_t n_copies, uint32_t n_cleared,
                                                uint64_t n_total, uint32_t parts, uint32_t bits, uint32_t rbits, uint32_t inv_mul)
{
    extern __shared__ __attribute__((aligned(16))) unsigned long long s_hist[];
    constexpr uint32_t H = 1u << kLogHistBits;
    unsigned long long *s_hist2 = s_hist + H;
    const uint32_t s = blockIdx.x % n_copies, rest = blockIdx.x / n_copies;
    const uint32_t part = rest % parts, b = rest / parts;
    for (uint32_t i = threadIdx.x; i < H; i += blockDim.x) {
        s_hist[i] = 0ull;
        if (SIGMA) s_hist2[i] = 0ull;
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, waves = blockDim.x >> 6;
    constexpr uint32_t U = 4;   // entries in flight per lane
    // Copy s takes the walk's blocks s, s + n_copies, s + 2 n_copies, ...:
    // the walk's blocks log very unequal numbers of exits (each claims as it goes,
    // and the older workgroup on a compute unit wins most issue cycles: at tau = 4
    // and 1e8 photons the first 256 of 512 blocks log 3.6 times as many as the
    // rest), so contiguous shares would load some copies 1.56 times the mean.  Each
    // wave takes every waves-th of them and reads its entries U x 64 at a time.
    for (uint32_t g = s + n_copies * (threadIdx.x >> 6); g < walk_blocks; g += n_copies * waves) {
        const uint64_t region = (uint64_t)b * walk_blocks + g;
        const uint32_t n = count[region];
        const unsigned long long *ent = log + region * cap;
        for (uint32_t base = 0; base < n; base += U * 64) {
            unsigned long long e[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = base + u * 64 + lane;
                e[u] = i < n ? ent[i] : 0ull;
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                if (base + u * 64 + lane >= n) continue;
                const uint32_t h = log_index((uint32_t)(e[u] >> 32), bits, rbits);
                if ((h >> kLogHistBits) != part) continue;
                const float wf = __uint_as_float((uint32_t)e[u]);
                atomicAdd(&s_hist[h & (H - 1)], fix(wf));
                if (SIGMA) atomicAdd(&s_hist2[h & (H - 1)], fix(wf * wf));
            }
        }
    }
    __syncthreads();
    unsigned long long *dst = copies + (uint64_t)s * n_total;
    unsigned long long *dst2 = SIGMA ? copies2 + (uint64_t)s * n_total : nullptr;
    const uint32_t per_range = 1u << (bits - rbits + 3);
    for (uint32_t i = threadIdx.x; i < H; i += blockDim.x) {
        const uint32_t h = part * H + i;
        if (h >= per_range) break;
        // Undo the scramble: p = range bits | group bits, g = p / kLogHashMul mod 2^bits.
        const uint32_t p = (b << (bits - rbits)) | (h >> 3);
        const uint64_t key = ((uint64_t)((p * inv_mul) & ((1u << bits) - 1u)) << 3) | (h & 7u);
        if (key >= n_total) continue;
        const unsigned long long v = s_hist[i];
        const unsigned long long v2 = SIGMA ? s_hist2[i] : 0ull;
        if (s >= n_cleared) {
            dst[key] = v;
            if (SIGMA) dst2[key] = v2;
        } else {
            if (v) dst[key] += v;
            if (SIGMA && v2) dst2[key] += v2;
        }
    }
}

// Sum the n_copies fixed-point copies of every pixel (integer adds, so the
// order is immaterial) and write them to the caller's images, or add them
// (ADD), as int64 (FIX) or converted to double.
// One medium per blockIdx.y: its pixels are keys [y * n_pix, (y + 1) * n_pix)
// of copies that hold n_total keys each; its images start at y * n_side and
// y * (n_pix - n_side) in the outputs.  blockIdx.z = 1 takes the squared
// weights.
//
// Unscattered first-step exits were only counted (workspace word kWsBallistic
// of each medium); the beam pixel (word kWsBeamKey) gets count x ball_w.
//
// A block takes kFinPix pixels per thread of one image; with SPREAD they are a
// block of spread_pixel, which it undoes through LDS.  Their weights' sum, its
// share of the +x or +z face's total, replaces its first word in copy 0 (which
// no other block reads) for finalize_scalars to add up: an atomic per block on
// one word took 12 ns each, one after the other, 12 of the 21 us at 512 x 512.
constexpr int kFinPix = 4;
template <bool SPREAD>
constexpr int fin_threads() { return SPREAD ? 1024 : 256; }
template <bool SPREAD>
constexpr int fin_block() { return fin_threads<SPREAD>() * kFinPix; }
static_assert(fin_block<true>() == 1 << kSpreadBits, "a block undoes one permutation");
struct FinArgs {
    unsigned long long *copies[2];     // of the weights and of their squares
    void *side[2], *trans[2];
    unsigned long long ball_w[2];
    int n_copies;
    uint64_t n_total;
    uint32_t n_pix, n_side;
    const unsigned long long *ws_scal;
    double *scalars;
    int fix, add;                      // int64 images; add to the outputs
    uint32_t block;                    // pixels per block of finalize_images
};

template <bool SPREAD>
__global__ __launch_bounds__(fin_threads<SPREAD>()) void finalize_images(FinArgs a)
{
    constexpr int kThreads = fin_threads<SPREAD>(), kBlock = fin_block<SPREAD>();
    const uint64_t inst = blockIdx.y;
    const int z = blockIdx.z;
    const uint32_t side_blocks = (a.n_side + kBlock - 1) / kBlock;
    const bool is_side = blockIdx.x < side_blocks;
    const uint32_t nth = is_side ? blockIdx.x : blockIdx.x - side_blocks;
    const uint32_t first = (is_side ? 0u : a.n_side) + nth * kBlock;
    // (differences, which stay below 2^32 where an index past the end may not)
    const uint32_t n_here = min((is_side ? a.n_side : a.n_pix) - first, (uint32_t)kBlock);
    unsigned long long *copies = a.copies[z] + inst * a.n_pix;
    long long *out = (long long *)(is_side ? a.side[z] : a.trans[z]) +
                     (is_side ? inst * a.n_side : inst * (a.n_pix - a.n_side) - a.n_side);
    const unsigned long long beam_key = a.ws_scal[kWsBeamKey];
    const unsigned long long beam_v = a.ws_scal[inst * kWsScalarWords + kWsBallistic] * a.ball_w[z];
    // The loads of all copies and outputs are issued before any is used.
    unsigned long long part[kFinPix][kCopies];
    long long prev[kFinPix];
#pragma unroll
    for (int u = 0; u < kFinPix; ++u) {
        const uint32_t k = u * kThreads + threadIdx.x, i = first + k;
        const bool in = k < n_here;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) part[u][c] = in && c < a.n_copies ? copies[(uint64_t)c * a.n_total + i] : 0ull;
        prev[u] = a.add && in ? out[i] : 0ll;   // the output's bits (int64, or a double's)
    }
    unsigned long long v[kFinPix];
#pragma unroll
    for (int u = 0; u < kFinPix; ++u) {
        v[u] = 0ull;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) v[u] += part[u][c];
    }
    if (SPREAD) {
        // The word at k is that of pixel (k - shift) / kSpreadMul in a whole block.
        constexpr uint32_t inv = inverse_mod_2_32(kSpreadMul);
        __shared__ unsigned long long s_pix[kBlock];
#pragma unroll
        for (int u = 0; u < kFinPix; ++u) {
            const uint32_t k = u * kThreads + threadIdx.x;
            s_pix[n_here == (uint32_t)kBlock ? ((k - nth * kSpreadShift) * inv) & (kBlock - 1) : k] = v[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kFinPix; ++u) v[u] = s_pix[u * kThreads + threadIdx.x];
    }
    unsigned long long sum = 0ull;
#pragma unroll
    for (int u = 0; u < kFinPix; ++u) {
        const uint32_t k = u * kThreads + threadIdx.x, i = first + k;
        if (k >= n_here) break;
        if (beam_key == (uint64_t)i + 1) v[u] += beam_v;
        if (a.fix) out[i] = prev[u] + (long long)v[u];
        else ((double *)out)[i] = __longlong_as_double(prev[u]) + (double)(long long)v[u] * (1.0 / kFix);
        sum += v[u];
    }
    if (z != 0) return;
    __shared__ unsigned long long s_part[kThreads / 64];
    sum = wave_sum(sum);
    if (__lane_id() == 0) s_part[threadIdx.x >> 6] = sum;
    __syncthreads();   // (every word of the block has been read)
    if (threadIdx.x < 64) {
        sum = wave_sum(threadIdx.x < kThreads / 64 ? s_part[threadIdx.x] : 0ull);
        if (threadIdx.x == 0) copies[first] = sum;
    }
}

// Fixed-point scalar sums to the caller's doubles (weights scaled back by
// 2^-32, counts as they are); the second-order side moments are FP64 sums.
// The +x and +z faces' totals are those of their images, added up from the
// blocks of finalize_images.  One medium per block.
constexpr int kScalThreads = 256;
__global__ __launch_bounds__(kScalThreads) void finalize_scalars(FinArgs a)
{
    const uint64_t inst = blockIdx.x;
    const unsigned long long *ws_scal = a.ws_scal + inst * kWsScalarWords;
    const unsigned long long *copies = a.copies[0] + inst * a.n_pix;
    double *scalars = a.scalars + inst * MC_N_SCALARS;
    const int t = threadIdx.x;
    unsigned long long face[2] = {0ull, 0ull};
    for (uint64_t i = t * a.block; i < a.n_side; i += kScalThreads * a.block) face[0] += copies[i];
    for (uint64_t i = (uint64_t)a.n_side + t * a.block; i < a.n_pix; i += kScalThreads * a.block) face[1] += copies[i];
    __shared__ unsigned long long s_face[2][kScalThreads / 64];
    for (int f = 0; f < 2; ++f) {
        const unsigned long long v = wave_sum(face[f]);
        if (__lane_id() == 0) s_face[f][t >> 6] = v;
    }
    __syncthreads();
    if (t >= MC_N_SCALARS) return;
    double v = 0.0;
    if (t < MC_S_RESERVED) {
        const bool weight = t <= MC_S_CAPPED_W;
        long long n = (long long)ws_scal[t];
        if (t == MC_S_FACE + 1 || t == MC_S_FACE + 5) {
            const unsigned long long *f = s_face[t == MC_S_FACE + 1 ? 0 : 1];
            n = (long long)(f[0] + f[1] + f[2] + f[3]);
        }
        // Reflections are not counted by the walk: every step interacts or
        // reaches a wall, and a wall step reflects unless the photon leaves,
        // which every photon not killed by roulette or capped does once.
        if (t == MC_S_REFLECTIONS)
            n = (long long)(ws_scal[MC_S_STEPS] - ws_scal[MC_S_EVENTS] -
                            (ws_scal[MC_S_PHOTONS] - ws_scal[MC_S_ROULETTE_KILLS] - ws_scal[MC_S_CAPPED]));
        v = weight ? (double)n * (1.0 / kFix) : (double)n;
    } else if (t >= MC_S_SIDE_W2 && t <= MC_S_SIDE_W2L) {
        v = __longlong_as_double((long long)ws_scal[t]);
    }
    scalars[t] = a.add ? scalars[t] + v : v;
}

__global__ void philox_blocks_kernel(uint32_t k0, uint32_t k1, uint32_t instance, const uint64_t *ids,
                                     uint64_t n_ids, uint32_t step0, uint32_t n_steps, uint32_t *out)
{
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_ids * (uint64_t)n_steps) return;
    const uint64_t i = t / n_steps;
    const uint32_t st = step0 + (uint32_t)(t % n_steps);
    const uint64_t id = ids[i];
    const Block4 r = philox4x32_10(st, instance, (uint32_t)id, (uint32_t)(id >> 32), k0, k1);
    out[4 * t + 0] = r.r0;
    out[4 * t + 1] = r.r1;
    out[4 * t + 2] = r.r2;
    out[4 * t + 3] = r.r3;
}

// Sums over an image in two kernels and a fixed order (deterministic): block b
// of the first takes pixels b x 1024 + t + j x (gridDim x 1024) in lane t, adds
// over its waves by a fixed tree and over the waves in order, and leaves N
// partials in part[N b ...]; sum_parts adds those of up to kSumBlocks blocks,
// one per lane of a block of that size, in the same way.  They are bound by
// launch and latency, not by the bytes (512 x 512: 6 MB, 1.3 us at the card's
// copy rate): 2048 pixels per block and the partials added side by side take
// 8.9 us for mc_grad's two kernels where 8192 per block and one chain took 11.9.
constexpr uint32_t kSumThreads = 1024, kSumBlocks = 256;
template <int N>
__device__ __forceinline__ void block_sum(double (&acc)[N], double (&s_part)[N][kSumThreads / 64])
{
    const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
#pragma unroll
    for (int c = 0; c < N; ++c) {
        acc[c] = wave_sum(acc[c]);
        if (__lane_id() == 0) s_part[c][wave] = acc[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < N; ++c) {
        acc[c] = 0.0;
        for (uint32_t w = 0; w < waves; ++w) acc[c] += s_part[c][w];
    }
}

template <int N>
__device__ __forceinline__ void sum_parts(const double *part, uint32_t n_blocks, double (&acc)[N])
{
    __shared__ double s_part[N][kSumThreads / 64];
#pragma unroll
    for (int c = 0; c < N; ++c) acc[c] = threadIdx.x < n_blocks ? part[N * threadIdx.x + c] : 0.0;
    block_sum(acc, s_part);
}

// The blocks such a sum over n pixels takes, N partials each, with room for
// `room` doubles.
template <int N>
uint32_t sum_blocks(uint64_t n, uint64_t room)
{
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({kSumBlocks, (n + 2047) / 2048, room / N}));
}

// sum_p g_p M_k[p], sum_p g_p M_L[p] and, with per-pixel h (H), sum_p h_p
// M2_k[p] and sum_p h_p M2_L[p].
template <bool H>
__global__ __launch_bounds__(kSumThreads) void grad_partial(const double *g, const double *h, const double *wk,
                                                            const double *wl, const double *w2k, const double *w2l,
                                                            uint64_t n, double *part)
{
    constexpr int N = H ? 4 : 2;
    __shared__ double s_part[N][kSumThreads / 64];
    double acc[N] = {};
    const uint64_t stride = (uint64_t)gridDim.x * kSumThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kSumThreads + threadIdx.x; i < n; i += stride) {
        acc[0] = fma(g[i], wk[i], acc[0]);
        acc[1] = fma(g[i], wl[i], acc[1]);
        if constexpr (H) {
            acc[2] = fma(h[i], w2k[i], acc[2]);
            acc[3] = fma(h[i], w2l[i], acc[3]);
        }
    }
    block_sum(acc, s_part);
    if (threadIdx.x == 0)
        for (int c = 0; c < N; ++c) part[N * blockIdx.x + c] = acc[c];
}

// With a uniform h instead, h times the image-wide second moments.
template <bool H>
__global__ __launch_bounds__(kSumBlocks) void grad_final(const double *part, uint32_t n_blocks, double h_uniform,
                                                         const double *scalars, double *out)
{
    double acc[H ? 4 : 2];
    sum_parts(part, n_blocks, acc);
    if (threadIdx.x != 0) return;
    out[0] = acc[0];
    out[1] = acc[1];
    if constexpr (H) {
        out[2] = acc[2];
        out[3] = acc[3];
    } else {
        out[2] = h_uniform != 0.0 ? h_uniform * scalars[MC_S_SIDE_W2K] : 0.0;
        out[3] = h_uniform != 0.0 ? h_uniform * scalars[MC_S_SIDE_W2L] : 0.0;
    }
}

// The side image's squared distance from a target less sum w^2, and its
// derivative 2 (I - T), in one pass over the images where tensor operations
// take five.
__global__ __launch_bounds__(kSumThreads) void l2_partial(const double *side, const double *target, uint64_t n,
                                                          double *g, double *part)
{
    __shared__ double s_part[1][kSumThreads / 64];
    double acc[1] = {0.0};
    const uint64_t stride = (uint64_t)gridDim.x * kSumThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kSumThreads + threadIdx.x; i < n; i += stride) {
        const double d = side[i] - target[i];
        g[i] = 2.0 * d;
        acc[0] = fma(d, d, acc[0]);
    }
    block_sum(acc, s_part);
    if (threadIdx.x == 0) part[blockIdx.x] = acc[0];
}

__global__ __launch_bounds__(kSumBlocks) void l2_final(const double *part, uint32_t n_blocks, const double *scalars,
                                                       double *loss)
{
    double acc[1];
    sum_parts(part, n_blocks, acc);
    if (threadIdx.x == 0) *loss = acc[0] - scalars[MC_S_SIDE_W2];
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

bool dims_ok(const mc_detector_t &d) { return d.side_nx >= 1 && d.side_ny >= 1 && d.trans_nx >= 1 && d.trans_ny >= 1; }

// Checks of the cuboid and its walls (Sec. 3.1.1: parameter validity).
int check_geometry(const char *fn, const mc_geometry_t &geo)
{
    for (int i = 0; i < 3; ++i)
        if (!finite_pos(geo.size_mm[i])) return fail(MC_EINVAL, "%s: size_mm[%d] must be > 0", fn, i);
    if (!finite_pos(geo.n_medium) || !finite_pos(geo.n_outside))
        return fail(MC_EINVAL, "%s: refractive indices must be > 0", fn);
    return MC_OK;
}

// Component i of the beam direction inside the medium (refracted at the
// z = 0 face, Snell), as the walk gets it: FP32, a zero always +0.
float entry_dir(const mc_source_t &src, const mc_geometry_t &geo, int i)
{
    const double dl = std::sqrt(src.dir[0] * src.dir[0] + src.dir[1] * src.dir[1] + src.dir[2] * src.dir[2]);
    const double eta = geo.n_outside / geo.n_medium;
    double d[3] = {eta * (src.dir[0] / dl), eta * (src.dir[1] / dl), 0.0};
    d[2] = std::sqrt(std::max(0.0, 1.0 - d[0] * d[0] - d[1] * d[1]));
    const float f = (float)d[i];
    return f == 0.f ? 0.f : f;   // -0 (or an underflow to it) becomes +0
}

// Checks of the source, detector, tally buffers and run settings shared by
// single and batched walks.
int check_setup(const char *fn, const mc_source_t &src, const mc_geometry_t &geo, const mc_detector_t &det,
                const mc_run_t &rn, const mc_tally_t &t)
{
    if (!(src.pos_mm[2] == 0.0) || !(src.pos_mm[0] >= 0.0 && src.pos_mm[0] <= geo.size_mm[0]) ||
        !(src.pos_mm[1] >= 0.0 && src.pos_mm[1] <= geo.size_mm[1]))
        return fail(MC_EINVAL, "%s: the source must lie on the z = 0 face", fn);
    const double dl = std::sqrt(src.dir[0] * src.dir[0] + src.dir[1] * src.dir[1] + src.dir[2] * src.dir[2]);
    if (!(dl > 0.0) || !std::isfinite(dl) || !(src.dir[2] > 0.0))
        return fail(MC_EINVAL, "%s: the source direction must point into the cuboid (dir[2] > 0)", fn);
    const double R = src.beam_radius_mm;
    if (!(R >= 0.0) || !std::isfinite(R))
        return fail(MC_EINVAL, "%s: beam_radius_mm must be finite and >= 0", fn);
    if (R > 0.0 && (src.pos_mm[0] - R < 0.0 || src.pos_mm[0] + R > geo.size_mm[0] || src.pos_mm[1] - R < 0.0 ||
                    src.pos_mm[1] + R > geo.size_mm[1]))
        return fail(MC_EINVAL, "%s: the beam disk must lie inside the z = 0 face", fn);
    // A photon exactly on a side wall with no direction component across it
    // would meet that wall at distance 0 (the walk's wall distance has no
    // zero-component test): keep the entry points off the far side walls
    // when the refracted beam runs parallel to them.
    for (int i = 0; i < 2; ++i)
        if (entry_dir(src, geo, i) == 0.f && (float)src.pos_mm[i] + (float)R >= (float)geo.size_mm[i])
            return fail(MC_EINVAL, "%s: the beam must not run along the face %s = %g", fn, i ? "y" : "x",
                        geo.size_mm[i]);
    if (!dims_ok(det)) return fail(MC_EINVAL, "%s: image dimensions must be >= 1", fn);
    if (!t.side || !t.trans || !t.scalars) return fail(MC_EINVAL, "%s: side, trans and scalars are required", fn);
    if ((det.flags & MC_SIGMA) && (!t.side_w2 || !t.trans_w2))
        return fail(MC_EINVAL, "%s: MC_SIGMA needs side_w2 and trans_w2", fn);
    if (rn.max_steps < 1 || rn.max_steps > (1u << 24))
        return fail(MC_EINVAL, "%s: max_steps must be in 1..2^24", fn);
    if (!(rn.roulette_w >= 0.0) || !(rn.roulette_p > 0.0 && rn.roulette_p <= 1.0))
        return fail(MC_EINVAL, "%s: roulette_w >= 0 and roulette_p in (0, 1] required", fn);
    if (rn.block_size != 0 && (rn.block_size < 64 || rn.block_size > 1024 || rn.block_size % 64))
        return fail(MC_EINVAL, "%s: block_size must be a multiple of 64 in 64..1024", fn);
    if (rn.grid_blocks < 0) return fail(MC_EINVAL, "%s: grid_blocks must be >= 0", fn);
    if (rn.chunk > 65536) return fail(MC_EINVAL, "%s: chunk must be at most 65536", fn);
    return MC_OK;
}

// Fixed-point sums stay below 2^63: every weight is at most
// max(1, roulette_w / roulette_p), so n_photons times that (squared for
// MC_SIGMA) must stay below 2^31.
int check_overflow(const char *fn, uint64_t n_photons, const mc_detector_t &det, const mc_run_t &rn)
{
    const double wmax = std::max(1.0, rn.roulette_w / rn.roulette_p);
    const double bound = (double)n_photons * ((det.flags & MC_SIGMA) ? wmax * wmax : wmax);
    if (!(bound < 2147483648.0))
        return fail(MC_EINVAL, "%s: %llu photons with weights up to %g could overflow the fixed-point tallies; "
                    "split the run into photon ranges", fn, (unsigned long long)n_photons, wmax);
    return MC_OK;
}

// Launch-independent kernel arguments: the cuboid and its walls, the entry
// beam (refracted at the z = 0 face, keeping 1 - R of its weight), roulette,
// the Philox key and the detector.
void fill_common(WalkArgs &a, const mc_source_t &src, const mc_geometry_t &geo, const mc_detector_t &det,
                 const mc_run_t &rn)
{
    for (int i = 0; i < 3; ++i) a.size[i] = (float)geo.size_mm[i];
    a.matched = geo.n_outside == geo.n_medium;
    a.fresnel = a.matched ? 0.f : 1.f;
    a.n21 = (float)(geo.n_outside / geo.n_medium);
    a.n12 = (float)(geo.n_medium / geo.n_outside);
    a.n12sq = (float)((geo.n_medium / geo.n_outside) * (geo.n_medium / geo.n_outside));
    const double dl = std::sqrt(src.dir[0] * src.dir[0] + src.dir[1] * src.dir[1] + src.dir[2] * src.dir[2]);
    double din[3] = {src.dir[0] / dl, src.dir[1] / dl, src.dir[2] / dl};
    double R0 = 0.0;
    if (!a.matched) {
        const double n1 = geo.n_outside, n2 = geo.n_medium, ci = din[2];
        const double si = std::sqrt(std::max(0.0, 1.0 - ci * ci)), st = n1 / n2 * si;
        if (st >= 1.0) {
            R0 = 1.0;
        } else {
            const double ct = std::sqrt(1.0 - st * st);
            const double rs = (n1 * ci - n2 * ct) / (n1 * ci + n2 * ct);
            const double rp = (n2 * ci - n1 * ct) / (n2 * ci + n1 * ct);
            R0 = 0.5 * (rs * rs + rp * rp);
        }
    }
    for (int i = 0; i < 3; ++i) {
        a.pos0[i] = (float)src.pos_mm[i];
        a.dir0[i] = entry_dir(src, geo, i);
    }
    a.w0 = (float)(1.0 - R0);
    a.beam_radius = (float)src.beam_radius_mm;
    a.roulette_w = (float)rn.roulette_w;
    a.roulette_p = (float)rn.roulette_p;
    a.inv_roulette_p = (float)(1.0 / rn.roulette_p);
    a.key0 = (uint32_t)rn.seed;
    a.key1 = (uint32_t)(rn.seed >> 32);
    a.max_steps = rn.max_steps;
    a.side_nx = det.side_nx; a.side_ny = det.side_ny;
    a.trans_nx = det.trans_nx; a.trans_ny = det.trans_ny;
    a.pix_scale[0] = (float)(det.side_ny / geo.size_mm[1]);
    a.pix_scale[1] = (float)(det.side_nx / geo.size_mm[2]);
    a.pix_scale[2] = (float)(det.trans_ny / geo.size_mm[1]);
    a.pix_scale[3] = (float)(det.trans_nx / geo.size_mm[0]);
    a.quiet_steps = rn.max_steps > (uint32_t)kQuietSteps ? rn.max_steps - kQuietSteps : 0u;
    a.copy_mask = kCopies - 1;
    a.n_side = (uint32_t)((uint64_t)det.side_nx * det.side_ny);
    a.n_pix_inst = (uint32_t)((uint64_t)det.side_nx * det.side_ny + (uint64_t)det.trans_nx * det.trans_ny);
}

// Per-medium coefficients (Eq. 1 and Eq. 16): s = log2(u0) * neg_ln2_over_mu.
void fill_medium(float &neg_ln2_over_mu, float &albedo, float &absorb, double mu_t, double alb)
{
    neg_ln2_over_mu = mu_t > 0.0 ? (float)(-M_LN2 / mu_t) : -__builtin_huge_valf();
    albedo = (float)alb;
    absorb = (float)(1.0 - alb);
}

// Lower a.quiet_steps to where a photon of this medium cannot yet have met
// roulette.  A weight starts at w0 and is multiplied by the albedo at most once
// per step, each product off by at most 2^-24; the count is rounded down and
// taken a thousandth short, which covers the logarithms' rounding too.
void limit_quiet(WalkArgs &a, float albedo)
{
    const double keep = (double)albedo * (1.0 - 0x1p-23), drop = std::log((double)a.roulette_w / (double)a.w0);
    double steps = 0.0;
    if (a.roulette_w <= 0.f || (albedo > 0.f && drop < 0.0)) {
        steps = a.roulette_w <= 0.f ? 4294967295.0 : std::min(4294967295.0, 0.999 * drop / std::log(keep));
    }
    const uint32_t n = (uint32_t)std::floor(steps);
    a.quiet_steps = std::min(a.quiet_steps, n > kQuietSteps + 1u ? n - kQuietSteps - 1u : 0u);
}

// A medium's coefficients in 1/mm from the form the caller gave them in.
struct MediumCoef {
    double mu_sca, mu_abs, mu_ext, albedo;
};

bool finite_nonneg(double v) { return std::isfinite(v) && v >= 0.0; }

// Eq. 1 (optical depth along the beam axis), Eq. 16 (albedo) or Eq. 17
// (concentration times the cross-sections of Eq. 14), validated.  The optical
// depth form keeps mu_ext = tau / size_z and the given albedo exactly, the
// others form mu_ext as the sum and the albedo as the quotient.
int medium_coefficients(const char *fn, const mc_medium_t &m, double size_z, MediumCoef &c)
{
    const bool sig_ok = finite_nonneg(m.sigma_sca_mm2) && finite_nonneg(m.sigma_abs_mm2);
    if (m.input == MC_MEDIUM_TAU) {
        if (!finite_nonneg(m.tau)) return fail(MC_EINVAL, "%s: tau must be finite and >= 0", fn);
        double alb = m.albedo;
        if (alb < 0.0) {
            if (!sig_ok || !(m.sigma_sca_mm2 + m.sigma_abs_mm2 > 0.0))
                return fail(MC_EINVAL, "%s: albedo < 0 takes sigma_sca / (sigma_sca + sigma_abs), which needs "
                                       "cross-sections >= 0 with a positive sum", fn);
            alb = m.sigma_sca_mm2 / (m.sigma_sca_mm2 + m.sigma_abs_mm2);
        } else if (!(alb <= 1.0)) {
            return fail(MC_EINVAL, "%s: albedo must be in [0, 1] (or < 0 to derive it)", fn);
        }
        c.mu_ext = m.tau / size_z;
        c.albedo = alb;
        c.mu_sca = alb * c.mu_ext;
        c.mu_abs = (1.0 - alb) * c.mu_ext;
        return MC_OK;
    }
    if (m.input == MC_MEDIUM_MU) {
        if (!finite_nonneg(m.mu_sca) || !finite_nonneg(m.mu_abs))
            return fail(MC_EINVAL, "%s: mu_sca and mu_abs must be finite and >= 0", fn);
        c.mu_sca = m.mu_sca;
        c.mu_abs = m.mu_abs;
    } else if (m.input == MC_MEDIUM_CONCENTRATION) {
        if (!finite_nonneg(m.concentration_per_mm3) || !sig_ok || !finite_nonneg(m.mu_abs_host))
            return fail(MC_EINVAL, "%s: concentration, cross-sections and mu_abs_host must be finite and >= 0", fn);
        c.mu_sca = m.concentration_per_mm3 * m.sigma_sca_mm2;
        c.mu_abs = m.concentration_per_mm3 * m.sigma_abs_mm2 + m.mu_abs_host;
        if (!std::isfinite(c.mu_sca) || !std::isfinite(c.mu_abs))
            return fail(MC_EINVAL, "%s: the coefficients overflow", fn);
    } else {
        return fail(MC_EINVAL, "%s: unknown medium input %d", fn, m.input);
    }
    c.mu_ext = c.mu_sca + c.mu_abs;
    if (!std::isfinite(c.mu_ext)) return fail(MC_EINVAL, "%s: the coefficients overflow", fn);
    c.albedo = c.mu_ext > 0.0 ? c.mu_sca / c.mu_ext : 1.0;
    return MC_OK;
}

// A batched launch's schedule is written into the workspace by small kernels
// whose arguments carry up to kInstPerCopy media each (no host buffer has to
// outlive the call).
constexpr int kInstPerCopy = 32;
struct InstChunk {
    BatchInst v[kInstPerCopy];
    uint32_t n, first;
};

__global__ void set_schedule(BatchInst *dst, InstChunk c)
{
    if (threadIdx.x < c.n) dst[c.first + threadIdx.x] = c.v[threadIdx.x];
}

// Enqueue init, walk and finalize for n_inst media (a single medium, or a
// batch whose schedule `sched` is given) on `st`; path_photons: WalkRequest.
int launch_walk(WalkArgs &a, const mc_detector_t &det, const mc_run_t &rn, const mc_tally_t &t, int phase,
                uint32_t n_inst, uint64_t total_photons, uint64_t path_photons, const std::vector<BatchInst> *sched,
                hipStream_t st)
{
    const bool batch = sched != nullptr;
    int cus = 0;
    if (int rc = device_cu_count(&cus)) return rc;
    const uint64_t n_pix = a.n_pix_inst, n_side = a.n_side, n_trans = n_pix - n_side;
    const uint64_t n_total = n_pix * n_inst;
    unsigned long long *ws = (unsigned long long *)t.workspace;
    // The optical depth along the beam axis (negative for a batch).
    const double tau_z = !batch && a.neg_ln2_over_mu < 0.f && std::isfinite(a.neg_ln2_over_mu)
                             ? -M_LN2 / (double)a.neg_ln2_over_mu * a.size[2]
                             : -1.0;
    const WalkPlan p = plan_walk({batch, phase, a.n_cdf, n_inst, n_pix, det.flags, total_photons, path_photons,
                                  rn.block_size, rn.grid_blocks, rn.chunk, tau_z, cus, (uint64_t)a.copy_mask + 1, t.workspace_bytes});
    const bool use_log = p.use_log;
    const int block = p.block, grid = p.grid;
    const size_t lds = p.lds;
    if (lds > 160 * 1024) return fail(MC_EINVAL, "mc_simulate: %zu bytes of LDS per block do not fit a CU", lds);
    const uint64_t copies = p.copies, chunk = p.chunk;
    const uint32_t parts = p.parts, n_cleared = (uint32_t)p.n_cleared;
    a.ws_scal = ws;
    a.ws_img = ws + kWsScalarWords * n_inst;
    a.ws_img2 = (det.flags & MC_SIGMA) ? a.ws_img + copies * n_total : nullptr;
    a.n_pix = n_total;
    a.n_inst = n_inst;
    a.copy_mask = n_cleared - 1;
    a.spread = p.permuted;
    a.cache_bits = p.cache_bits;
    a.chunk = (uint32_t)chunk;
    a.refill_min = p.refill_min;

    // ---- exit log: a region of log_cap entries per block and key range in
    // its words of the workspace (the walk writes every count, so nothing needs
    // clearing) ----
    // What init clears: the scalar words and every image copy, except when
    // log_bin will run (the exit log and some photons) and store into the
    // copies that take no atomics: then only copy 0 (and copy 0 of the squared weights).
    const bool bin_stores = use_log && n_cleared < copies && total_photons > 0;
    const uint64_t clear_words = bin_stores ? kWsScalarWords * n_inst + n_total : workspace_words(det, n_inst, copies);
    unsigned long long *clear2 = bin_stores && (det.flags & MC_SIGMA) ? a.ws_img2 : nullptr;
    const uint64_t clear2_words = clear2 ? n_total : 0;
    if (use_log) {
        const uint64_t regions = ((uint64_t)1 << p.shape.rbits) * grid;
        a.log_cap = p.log_cap;
        a.log_count = (uint32_t *)(ws + p.log_at);
        a.log = ws + p.log_at + (regions * 4 + 7) / 8;
        a.log_bits = p.shape.bits;
        a.log_rbits = p.shape.rbits;
    }

    const int zero_all = (det.flags & MC_ACCUMULATE) ? 0 : 1;
    const bool sig = (det.flags & MC_SIGMA) != 0, rec = (det.flags & MC_RECORD) != 0;
    // The caller's timing events ride on the dispatches themselves
    // (hipExtLaunchKernel): a separate event record would put a barrier, and
    // several microseconds of idle device, between two kernels.
    hipExtLaunchKernelGGL(init_kernel, dim3(1024), dim3(256), 0, st, (hipEvent_t)rn.sim_events[0], nullptr, 0u, ws,
                          (size_t)clear_words, clear2, (size_t)clear2_words, (size_t)(n_side * n_inst), a.rec_i, a.rec_f,
                          (size_t)a.rec_rows, a.side_wk, a.side_wl, a.side_w2k, a.side_w2l, zero_all);
    MC_HIP_CHECK(hipGetLastError());

    using Kern = void (*)(WalkArgs);
    Kern kern = nullptr;
    uint64_t units = 0;
    if (batch) {
        // The schedule: unit ranges in schedule order, copied after the scalars
        // and images of the workspace (after init has cleared it).
        BatchInst *dst = (BatchInst *)(ws + p.ws_words);
        std::vector<BatchInst> s = *sched;
        for (auto &b : s) {
            b.unit_begin = units;
            units += (b.n_photons + chunk - 1) / chunk;
        }
        for (uint32_t i = 0; i < n_inst; i += kInstPerCopy) {
            InstChunk c{};
            c.first = i;
            c.n = std::min<uint32_t>(kInstPerCopy, n_inst - i);
            for (uint32_t j = 0; j < c.n; ++j) c.v[j] = s[i + j];
            hipLaunchKernelGGL(set_schedule, dim3(1), dim3(kInstPerCopy), 0, st, dst, c);
        }
        MC_HIP_CHECK(hipGetLastError());
        a.insts = dst;
        static const Kern batch_kernels[4] = {
            walk_kernel<MC_PHASE_MIE, kOptBatch>, walk_kernel<MC_PHASE_MIE, kOptBatch | kOptSigma>,
            walk_kernel<MC_PHASE_MIE, kOptBatch | kOptLog>, walk_kernel<MC_PHASE_MIE, kOptBatch | kOptLog | kOptSigma>};
        kern = batch_kernels[(sig ? 1 : 0) + (use_log ? 2 : 0)];
    } else {
        const int opt = (sig ? kOptSigma : 0) | (rec ? kOptRecord : 0) | ((det.flags & MC_MOMENTS) ? kOptMoments : 0);
        static const Kern mie_kernels[8] = {walk_kernel<MC_PHASE_MIE, 0>, walk_kernel<MC_PHASE_MIE, 1>,
                                            walk_kernel<MC_PHASE_MIE, 2>, walk_kernel<MC_PHASE_MIE, 3>,
                                            walk_kernel<MC_PHASE_MIE, 4>, walk_kernel<MC_PHASE_MIE, 5>,
                                            walk_kernel<MC_PHASE_MIE, 6>, walk_kernel<MC_PHASE_MIE, 7>};
        static const Kern hg_kernels[8] = {walk_kernel<MC_PHASE_HG, 0>, walk_kernel<MC_PHASE_HG, 1>,
                                           walk_kernel<MC_PHASE_HG, 2>, walk_kernel<MC_PHASE_HG, 3>,
                                           walk_kernel<MC_PHASE_HG, 4>, walk_kernel<MC_PHASE_HG, 5>,
                                           walk_kernel<MC_PHASE_HG, 6>, walk_kernel<MC_PHASE_HG, 7>};
        kern = phase == MC_PHASE_MIE ? mie_kernels[opt] : hg_kernels[opt];
        if (use_log) {
            // Exit log with optional squared weights and path moments (index
            // sigma + 2 x moments); records take the atomic path.
            static const Kern log_kernels[8] = {
                walk_kernel<MC_PHASE_MIE, kOptLog>, walk_kernel<MC_PHASE_MIE, kOptLog | kOptSigma>,
                walk_kernel<MC_PHASE_MIE, kOptLog | kOptMoments>,
                walk_kernel<MC_PHASE_MIE, kOptLog | kOptMoments | kOptSigma>,
                walk_kernel<MC_PHASE_HG, kOptLog>, walk_kernel<MC_PHASE_HG, kOptLog | kOptSigma>,
                walk_kernel<MC_PHASE_HG, kOptLog | kOptMoments>,
                walk_kernel<MC_PHASE_HG, kOptLog | kOptMoments | kOptSigma>};
            kern = log_kernels[(phase == MC_PHASE_MIE ? 0 : 4) + (sig ? 1 : 0) +
                               ((det.flags & MC_MOMENTS) ? 2 : 0)];
        }
        units = total_photons;
    }
    const Claims c = claims_for(units, (uint64_t)grid, (uint64_t)block, chunk, std::max(tau_z, 0.0), batch);
    a.n_ids = (uint32_t)units;
    a.claim0 = c.claim0;
    a.claim_min = c.claim_min;
    a.claim_shift = c.claim_shift;
    if (units > 0) {
        MC_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), (uint32_t)lds, st, (hipEvent_t)rn.walk_events[0],
                              (hipEvent_t)rn.walk_events[1], 0u, a);
        MC_HIP_CHECK(hipGetLastError());
    } else {
        // No walk: the events mark the (empty) place where it would run.
        if (rn.walk_events[0]) MC_HIP_CHECK(hipEventRecord((hipEvent_t)rn.walk_events[0], st));
        if (rn.walk_events[1]) MC_HIP_CHECK(hipEventRecord((hipEvent_t)rn.walk_events[1], st));
    }
    if (use_log && units > 0) {
        const size_t hist = ((size_t)8 << kLogHistBits) * (sig ? 2 : 1);
        auto bin = sig ? log_bin<true> : log_bin<false>;
        MC_HIP_CHECK(hipFuncSetAttribute((const void *)bin, hipFuncAttributeMaxDynamicSharedMemorySize, (int)hist));
        hipLaunchKernelGGL(bin, dim3((1u << a.log_rbits) * parts * (uint32_t)copies), dim3(1024), hist, st,
                           (const unsigned long long *)a.log, (const uint32_t *)a.log_count, a.log_cap,
                           (uint32_t)grid, a.ws_img, a.ws_img2, (uint32_t)copies, n_cleared, n_total, parts,
                           a.log_bits, a.log_rbits, inverse_mod_2_32(kLogHashMul));
        MC_HIP_CHECK(hipGetLastError());
    }
    // ---- finalize: per-XCD copies to the caller's images, scalars to doubles ----
    const bool fix64 = (det.flags & MC_FIX64) != 0;
    FinArgs f{};
    f.copies[0] = a.ws_img;
    f.copies[1] = a.ws_img2;
    f.side[0] = t.side; f.side[1] = t.side_w2;
    f.trans[0] = t.trans; f.trans[1] = t.trans_w2;
    // The fixed-point weight (and squared weight, an FP32 product as in the
    // walk) of an unscattered first-step exit, as the walk's fix() rounds it.
    const float w0sq = a.w0 * a.w0;
    f.ball_w[0] = (unsigned long long)std::llrint((double)a.w0 * kFix);
    f.ball_w[1] = (unsigned long long)std::llrint((double)w0sq * kFix);
    f.n_copies = (int)copies;
    f.n_total = n_total;
    f.n_pix = (uint32_t)n_pix;
    f.n_side = (uint32_t)n_side;
    f.ws_scal = ws;
    f.scalars = t.scalars;
    f.fix = fix64;
    f.add = !zero_all;
    f.block = a.spread ? fin_block<true>() : fin_block<false>();
    const unsigned fin_x = (unsigned)((n_side + f.block - 1) / f.block + (n_trans + f.block - 1) / f.block);
    hipLaunchKernelGGL(a.spread ? finalize_images<true> : finalize_images<false>, dim3(fin_x, n_inst, sig ? 2 : 1),
                       dim3(a.spread ? fin_threads<true>() : fin_threads<false>()), 0, st, f);
    hipExtLaunchKernelGGL(finalize_scalars, dim3(n_inst), dim3(kScalThreads), 0, st, nullptr,
                          (hipEvent_t)rn.sim_events[1], 0u, f);
    MC_HIP_CHECK(hipGetLastError());
    return MC_OK;
}

// Checks and schedule of a batched launch (items in decreasing estimated
// cost, photons x (1 + tau), so the longest start first).
int prepare_batch(const char *fn, const mc_batch_item_t *items, uint32_t n_items, int32_t n_cdf,
                  const mc_source_t *source, const mc_geometry_t *geometry, const mc_detector_t *detector,
                  const mc_run_t *run, const mc_tally_t *tally, double photon_scale, WalkArgs &a,
                  std::vector<BatchInst> &sched, uint64_t &total, uint64_t &full)
{
    if (!items || !source || !geometry || !detector || !run || !tally) return fail(MC_EINVAL, "%s: null argument", fn);
    if (n_items < 1 || n_items > MC_MAX_BATCH) return fail(MC_EINVAL, "%s: n_items must be in 1..%d", fn, MC_MAX_BATCH);
    if (n_cdf < 2 || n_cdf > MC_MAX_N_CDF) return fail(MC_EINVAL, "%s: n_cdf %d outside 2..%d", fn, n_cdf, MC_MAX_N_CDF);
    const mc_geometry_t &geo = *geometry;
    const mc_detector_t &det = *detector;
    const mc_run_t &rn = *run;
    const mc_tally_t &t = *tally;
    if (int rc = check_geometry(fn, geo)) return rc;
    if (int rc = check_setup(fn, *source, geo, det, rn, t)) return rc;
    if (det.flags & (MC_RECORD | MC_MOMENTS | MC_MOMENTS_PIXEL2))
        return fail(MC_EUNSUPPORTED, "%s: MC_RECORD and MC_MOMENTS are not available for batched launches", fn);
    if (det.flags & ~(MC_ACCUMULATE | MC_SIGMA | MC_FIX64 | MC_EXIT_LOG))
        return fail(MC_EINVAL, "%s: unknown detector flags 0x%x", fn, det.flags);
    const uint64_t n_pix = (uint64_t)det.side_nx * det.side_ny + (uint64_t)det.trans_nx * det.trans_ny;
    if (n_pix * n_items >= 0xFFFFFFFFull)
        return fail(MC_EINVAL, "%s: images exceed 2^32 - 2 pixels over all items", fn);
    if (!t.workspace || ((uintptr_t)t.workspace & 7) || t.workspace_bytes < batch_workspace_words(det, n_items) * 8)
        return fail(MC_EINVAL, "%s: workspace needs %llu bytes, 8-byte aligned", fn,
                    (unsigned long long)(batch_workspace_words(det, n_items) * 8));
    sched.clear();
    total = full = 0;
    std::vector<double> cost;
    for (uint32_t i = 0; i < n_items; ++i) {
        const mc_batch_item_t &it = items[i];
        if (!(it.tau >= 0.0) || !std::isfinite(it.tau)) return fail(MC_EINVAL, "%s: item %u: tau must be >= 0", fn, i);
        if (!(it.albedo >= 0.0 && it.albedo <= 1.0))
            return fail(MC_EINVAL, "%s: item %u: albedo must be in [0, 1]", fn, i);
        if (!it.inv_cdf) return fail(MC_EINVAL, "%s: item %u: inv_cdf is required", fn, i);
        uint64_t n = it.n_photons;
        full += n;
        if (photon_scale < 1.0 && n > 0) n = std::max<uint64_t>(1, (uint64_t)std::llround((double)n * photon_scale));
        if (int rc = check_overflow(fn, n, det, rn)) return rc;
        BatchInst b{};
        fill_medium(b.neg_ln2_over_mu, b.albedo, b.absorb, it.tau / geo.size_mm[2], it.albedo);
        b.inv_cdf = it.inv_cdf;
        b.n_photons = n;
        b.counter = it.instance;
        b.slot = i;
        sched.push_back(b);
        cost.push_back((double)n * (1.0 + it.tau));
        total += n;
    }
    std::vector<uint32_t> order(n_items);
    for (uint32_t i = 0; i < n_items; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return cost[x] > cost[y]; });
    std::vector<BatchInst> sorted;
    for (uint32_t i : order) sorted.push_back(sched[i]);
    sched.swap(sorted);

    a = WalkArgs{};
    fill_common(a, *source, geo, det, rn);
    a.n_cdf = n_cdf;
    a.inv_cdf = nullptr;
    a.instance = 0;
    a.photon_offset = 0;
    a.record_stride = 1;
    for (const BatchInst &b : sched) limit_quiet(a, b.albedo);
    return MC_OK;
}

}  // namespace
}  // namespace mcmie

namespace mcmie {
namespace {

// The walk of mc_simulate.  With `scratch_ws` set, the caller's workspace is
// ignored: the images are tallied in as many fixed-point copies as fit that device
// array (noalloc callers) instead of in the workspace's.
int simulate(const char *fn, const mc_medium_t *medium, const mc_source_t *source, const mc_geometry_t *geometry,
             const mc_detector_t *detector, const mc_run_t *run, const mc_tally_t *tally, void *scratch_ws,
             void *stream)
{
    clear_error();
    if (!medium || !source || !geometry || !detector || !run || !tally)
        return fail(MC_EINVAL, "%s: null argument", fn);
    const mc_medium_t m = *medium;
    const mc_geometry_t geo = *geometry;
    const mc_detector_t det = *detector;
    const mc_run_t rn = *run;
    mc_tally_t t = *tally;

    // ---- parameter checks (Sec. 3.1.1) ----
    if (int rc = check_geometry(fn, geo)) return rc;
    MediumCoef coef{};
    if (int rc = medium_coefficients(fn, m, geo.size_mm[2], coef)) return rc;
    if (m.phase == MC_PHASE_MIE) {
        if (m.n_cdf < 2 || m.n_cdf > MC_MAX_N_CDF)
            return fail(MC_EINVAL, "%s: n_cdf %d outside 2..%d", fn, m.n_cdf, MC_MAX_N_CDF);
        if (!m.inv_cdf) return fail(MC_EINVAL, "%s: inv_cdf is required for MC_PHASE_MIE", fn);
    } else if (m.phase == MC_PHASE_HG) {
        if (!(m.g > -1.0 && m.g < 1.0)) return fail(MC_EINVAL, "%s: HG g must be in (-1, 1)", fn);
    } else {
        return fail(MC_EINVAL, "%s: unknown phase %d", fn, m.phase);
    }
    if (scratch_ws) {
        // The library's array stands in for the workspace (checked by check_setup).
        t.workspace = scratch_ws;
        t.workspace_bytes = kNoAllocWords * 8;
    }
    if (int rc = check_setup(fn, *source, geo, det, rn, t)) return rc;
    if ((det.flags & MC_RECORD) && (rn.record_stride < 1 || (t.rec_rows > 0 && (!t.rec_i || !t.rec_f))))
        return fail(MC_EINVAL, "%s: MC_RECORD needs record_stride >= 1 and, for rec_rows > 0, rec_i and rec_f", fn);
    if (rn.photon_offset > UINT64_MAX - rn.n_photons) return fail(MC_EINVAL, "%s: photon ids overflow", fn);
    if (det.flags & ~(MC_ACCUMULATE | MC_SIGMA | MC_RECORD | MC_FIX64 | MC_MOMENTS | MC_MOMENTS_PIXEL2 | MC_EXIT_LOG))
        return fail(MC_EINVAL, "%s: unknown detector flags 0x%x", fn, det.flags);
    if ((det.flags & MC_EXIT_LOG) && (det.flags & MC_RECORD))
        return fail(MC_EINVAL, "%s: MC_EXIT_LOG does not combine with MC_RECORD", fn);
    if ((det.flags & MC_MOMENTS) && (!t.side_wk || !t.side_wl))
        return fail(MC_EINVAL, "%s: MC_MOMENTS needs side_wk and side_wl", fn);
    if ((det.flags & MC_MOMENTS_PIXEL2) && (!(det.flags & MC_MOMENTS) || !t.side_w2k || !t.side_w2l))
        return fail(MC_EINVAL, "%s: MC_MOMENTS_PIXEL2 needs MC_MOMENTS, side_w2k and side_w2l", fn);
    // The image copies the workspace has room for: all, or in the library's
    // scratch as many as fit (1e8 photons at tau = 1, one copy and these: 128 x 128
    // 3.96 / 1.92 ms, 512 x 512 4.74 / 3.47).
    uint64_t copies = kCopies;
    while (scratch_ws && copies > 1 && workspace_words(det, 1, copies) > kNoAllocWords) copies >>= 1;
    if (!t.workspace || ((uintptr_t)t.workspace & 7) || t.workspace_bytes < workspace_words(det, 1, copies) * 8) {
        if (scratch_ws)
            return fail(MC_EINVAL, "%s: the images need %llu bytes of scratch, more than the library's %llu "
                        "(at most 2^21 pixels over both images, 2^20 with MC_SIGMA)", fn,
                        (unsigned long long)(workspace_words(det, 1, copies) * 8),
                        (unsigned long long)(kNoAllocWords * 8));
        return fail(MC_EINVAL, "%s: workspace needs %llu bytes, 8-byte aligned", fn,
                    (unsigned long long)(workspace_words(det) * 8));
    }
    if (int rc = check_overflow(fn, rn.n_photons, det, rn)) return rc;
    const uint64_t n_pix = (uint64_t)det.side_nx * det.side_ny + (uint64_t)det.trans_nx * det.trans_ny;
    if (n_pix >= 0xFFFFFFFFull) return fail(MC_EINVAL, "%s: images exceed 2^32 - 2 pixels in total", fn);

    WalkArgs a{};
    fill_common(a, *source, geo, det, rn);
    fill_medium(a.neg_ln2_over_mu, a.albedo, a.absorb, coef.mu_ext, coef.albedo);
    limit_quiet(a, a.albedo);
    a.copy_mask = (uint32_t)(copies - 1);
    a.n_cdf = m.phase == MC_PHASE_MIE ? m.n_cdf : 0;
    a.inv_cdf = m.inv_cdf;
    a.hg_a = (float)(1.0 + m.g);
    a.hg_b = (float)(2.0 * m.g);
    a.hg_c = (float)(1.0 - m.g * m.g);
    a.hg_d = (float)(1.0 - m.g);
    a.instance = rn.instance;
    a.photon_offset = rn.photon_offset;
    a.rec_i = t.rec_i; a.rec_f = t.rec_f;
    a.side_wk = (det.flags & MC_MOMENTS) ? t.side_wk : nullptr;
    a.side_wl = (det.flags & MC_MOMENTS) ? t.side_wl : nullptr;
    a.side_w2k = (det.flags & MC_MOMENTS_PIXEL2) ? t.side_w2k : nullptr;
    a.side_w2l = (det.flags & MC_MOMENTS_PIXEL2) ? t.side_w2l : nullptr;
    a.rec_rows = (det.flags & MC_RECORD) ? t.rec_rows : 0;
    a.record_stride = rn.record_stride >= 1 ? rn.record_stride : 1;
    return launch_walk(a, det, rn, t, m.phase, 1, rn.n_photons, rn.n_photons, nullptr, (hipStream_t)stream);
}

// Address of this device's copy of `scratch`, looked up once per device
// with the device current (the array's name is a host-side stand-in).
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {nullptr};

int device_scratch(const char *fn, void **out)
{
    int dev = 0;
    MC_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(MC_EDEVICE, "%s: device index %d out of range", fn, dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(MC_EDEVICE, "%s: hipGetSymbolAddress(scratch) failed: %s", fn, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MC_OK;
}

}  // namespace
}  // namespace mcmie

extern "C" int mc_simulate(const mc_medium_t *medium, const mc_source_t *source, const mc_geometry_t *geometry,
                           const mc_detector_t *detector, const mc_run_t *run, const mc_tally_t *tally,
                           void *stream)
{
    return mcmie::simulate("mc_simulate", medium, source, geometry, detector, run, tally, nullptr, stream);
}

extern "C" int mc_simulate_noalloc(const mc_medium_t *medium, const mc_source_t *source,
                                   const mc_geometry_t *geometry, const mc_detector_t *detector, const mc_run_t *run,
                                   const mc_tally_t *tally, void *stream)
{
    using namespace mcmie;
    const char *fn = "mc_simulate_noalloc";
    clear_error();
    if (!detector || !tally) return fail(MC_EINVAL, "%s: null argument", fn);
    if (detector->flags & MC_EXIT_LOG)
        return fail(MC_EINVAL, "%s: MC_EXIT_LOG needs a caller workspace (use mc_simulate)", fn);
    if (!dims_ok(*detector)) return fail(MC_EINVAL, "%s: image dimensions must be >= 1", fn);
    if (workspace_words(*detector, 1, 1) > kNoAllocWords)
        return fail(MC_EINVAL, "%s: the images need %llu bytes of scratch, more than the library's %llu "
                    "(at most 2^21 pixels over both images, 2^20 with MC_SIGMA)", fn,
                    (unsigned long long)(workspace_words(*detector, 1, 1) * 8),
                    (unsigned long long)(kNoAllocWords * 8));
    void *ws = nullptr;
    if (int rc = device_scratch(fn, &ws)) return rc;
    return simulate(fn, medium, source, geometry, detector, run, tally, ws, stream);
}

extern "C" int mc_medium_coefficients(const mc_medium_t *medium, const mc_geometry_t *geometry, double out[4])
{
    using namespace mcmie;
    clear_error();
    if (!medium || !geometry || !out) return fail(MC_EINVAL, "mc_medium_coefficients: null argument");
    if (int rc = check_geometry("mc_medium_coefficients", *geometry)) return rc;
    MediumCoef c{};
    if (int rc = medium_coefficients("mc_medium_coefficients", *medium, geometry->size_mm[2], c)) return rc;
    out[0] = c.mu_sca;
    out[1] = c.mu_abs;
    out[2] = c.mu_ext;
    out[3] = c.albedo;
    return MC_OK;
}

extern "C" uint64_t mc_workspace_bytes(const mc_detector_t *detector)
{
    if (!detector || !mcmie::dims_ok(*detector)) return 0;
    return mcmie::workspace_words(*detector) * 8;
}

extern "C" uint64_t mc_workspace_bytes_log(const mc_detector_t *detector, uint64_t n_photons)
{
    if (!detector || !mcmie::dims_ok(*detector) || !(detector->flags & MC_EXIT_LOG)) return 0;
    using namespace mcmie;
    const mc_detector_t &d = *detector;
    const uint64_t n_keys = (uint64_t)d.side_nx * d.side_ny + (uint64_t)d.trans_nx * d.trans_ny;
    // The table-in-LDS shape: at most as many ranges as the HG walk takes.
    const uint64_t regions = ((uint64_t)1 << log_shape(n_keys, true).rbits) * kLogSizingBlocks;
    return workspace_words(d) * 8 + log_bytes_for(n_photons, regions);
}

extern "C" uint64_t mc_workspace_bytes_batch(const mc_detector_t *detector, uint32_t n_items)
{
    if (!detector || !mcmie::dims_ok(*detector) || n_items < 1 || n_items > MC_MAX_BATCH) return 0;
    return mcmie::batch_workspace_words(*detector, n_items) * 8;
}

extern "C" uint64_t mc_workspace_bytes_batch_log(const mc_detector_t *detector, uint32_t n_items,
                                                 uint64_t total_photons)
{
    using namespace mcmie;
    if (!detector || !dims_ok(*detector) || !(detector->flags & MC_EXIT_LOG) || n_items < 1 ||
        n_items > MC_MAX_BATCH)
        return 0;
    const mc_detector_t &d = *detector;
    const uint64_t n_keys = ((uint64_t)d.side_nx * d.side_ny + (uint64_t)d.trans_nx * d.trans_ny) * n_items;
    const uint64_t regions = ((uint64_t)1 << log_shape(n_keys, false).rbits) * kLogSizingBlocks;
    return batch_workspace_words(d, n_items) * 8 + log_bytes_for(total_photons, regions);
}

extern "C" int mc_simulate_batch(const mc_batch_item_t *items, uint32_t n_items, int32_t n_cdf,
                                 const mc_source_t *source, const mc_geometry_t *geometry,
                                 const mc_detector_t *detector, const mc_run_t *run, const mc_tally_t *tally,
                                 void *stream)
{
    using namespace mcmie;
    clear_error();
    WalkArgs a{};
    std::vector<BatchInst> sched;
    uint64_t total = 0, full = 0;
    if (int rc = prepare_batch("mc_simulate_batch", items, n_items, n_cdf, source, geometry, detector, run, tally,
                               1.0, a, sched, total, full))
        return rc;
    return launch_walk(a, *detector, *run, *tally, MC_PHASE_MIE, n_items, total, full, &sched, (hipStream_t)stream);
}

extern "C" int mc_autotune_batch(const mc_batch_item_t *items, uint32_t n_items, int32_t n_cdf,
                                 const mc_source_t *source, const mc_geometry_t *geometry,
                                 const mc_detector_t *detector, const mc_run_t *run, const mc_tally_t *tally,
                                 double sample_fraction, int32_t *block_size, uint32_t *chunk, double *best_ms,
                                 double *candidate_ms, void *stream)
{
    using namespace mcmie;
    clear_error();
    if (!block_size || !chunk || !best_ms) return fail(MC_EINVAL, "mc_autotune_batch: null output");
    if (!(sample_fraction > 0.0 && sample_fraction <= 1.0))
        return fail(MC_EINVAL, "mc_autotune_batch: sample_fraction must be in (0, 1]");
    WalkArgs a0{};
    std::vector<BatchInst> sched;
    uint64_t total = 0, full = 0;
    if (int rc = prepare_batch("mc_autotune_batch", items, n_items, n_cdf, source, geometry, detector, run, tally,
                               sample_fraction, a0, sched, total, full))
        return rc;
    static const int32_t blocks[3] = {256, 512, 1024};
    static const uint32_t chunks[5] = {256, 512, 1024, 2048, 4096};
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    MC_HIP_CHECK(hipEventCreate(&e0));
    MC_HIP_CHECK(hipEventCreate(&e1));
    double best = INFINITY;
    int32_t bb = 0;
    uint32_t bc = 0;
    int rc = MC_OK;
    for (int i = 0; i < 3 && rc == MC_OK; ++i) {
        for (int j = 0; j < 5 && rc == MC_OK; ++j) {
            mc_run_t rn = *run;
            rn.block_size = blocks[i];
            rn.chunk = chunks[j];
            rn.grid_blocks = 0;
            float ms = 0.f;
            for (int rep = 0; rep < 2 && rc == MC_OK; ++rep) {
                WalkArgs a = a0;
                if (rep == 1 && hipEventRecord(e0, st) != hipSuccess) rc = fail(MC_EDEVICE, "hipEventRecord failed");
                if (rc == MC_OK) rc = launch_walk(a, *detector, rn, *tally, MC_PHASE_MIE, n_items, total, full, &sched, st);
                if (rc == MC_OK && rep == 1) {
                    if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                        hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
                        rc = fail(MC_EDEVICE, "mc_autotune_batch: event timing failed");
                }
            }
            if (rc != MC_OK) break;
            if (candidate_ms) candidate_ms[i * 5 + j] = ms;
            if (ms < best) {
                best = ms;
                bb = blocks[i];
                bc = chunks[j];
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != MC_OK) return rc;
    *block_size = bb;
    *chunk = bc;
    *best_ms = best;
    return MC_OK;
}

extern "C" int mc_grad(const mc_medium_t *medium, const mc_geometry_t *geometry, const mc_detector_t *detector,
                       const mc_tally_t *tally, const double *dloss_dside, const double *d2loss_dside2,
                       double d2loss_uniform, double out_grad[3], void *stream)
{
    using namespace mcmie;
    clear_error();
    if (!medium || !geometry || !detector || !tally || !dloss_dside || !out_grad)
        return fail(MC_EINVAL, "mc_grad: null argument");
    const mc_medium_t m = *medium;
    const mc_geometry_t geo = *geometry;
    const mc_detector_t det = *detector;
    const mc_tally_t t = *tally;
    if (!finite_pos(geo.size_mm[2])) return fail(MC_EINVAL, "mc_grad: size_mm[2] must be > 0");
    MediumCoef coef{};
    if (int rc = medium_coefficients("mc_grad", m, geo.size_mm[2], coef)) return rc;
    if (!(coef.mu_sca > 0.0)) return fail(MC_EINVAL, "mc_grad: needs mu_sca > 0");
    if (det.side_nx < 1 || det.side_ny < 1) return fail(MC_EINVAL, "mc_grad: side image dimensions must be >= 1");
    if (!t.side_wk || !t.side_wl || !t.scalars)
        return fail(MC_EINVAL, "mc_grad: the tally has no moment images (MC_MOMENTS)");
    if (d2loss_dside2 && (!t.side_w2k || !t.side_w2l))
        return fail(MC_EINVAL, "mc_grad: a per-pixel second derivative needs the MC_MOMENTS_PIXEL2 images");
    if (!std::isfinite(d2loss_uniform))
        return fail(MC_EINVAL, "mc_grad: d2loss_uniform must be finite");
    if (d2loss_dside2 && d2loss_uniform != 0.0)
        return fail(MC_EINVAL, "mc_grad: give either d2loss_dside2 or d2loss_uniform, not both");
    if (!t.workspace || ((uintptr_t)t.workspace & 7) || t.workspace_bytes < (kWsScalarWords + 4) * 8)
        return fail(MC_EINVAL, "mc_grad: workspace of at least %llu bytes required",
                    (unsigned long long)((kWsScalarWords + 4) * 8));
    const double mu_s = coef.mu_sca;
    hipStream_t st = (hipStream_t)stream;
    HostResult host;
    double *dots = host ? host.data() : (double *)t.workspace + 24;    // scalar words 24..27
    const uint64_t n = (uint64_t)det.side_nx * det.side_ny;
    // The blocks' partials go after the scalar words, where mc_simulate keeps
    // its image copies (consumed by then), as many as the workspace holds.
    double *part = (double *)t.workspace + kWsScalarWords;
    const uint64_t room = t.workspace_bytes / 8 - kWsScalarWords;
    const uint32_t n_blocks = d2loss_dside2 ? sum_blocks<4>(n, room) : sum_blocks<2>(n, room);
    hipLaunchKernelGGL(d2loss_dside2 ? grad_partial<true> : grad_partial<false>, dim3(n_blocks), dim3(kSumThreads), 0,
                       st, dloss_dside, d2loss_dside2, (const double *)t.side_wk, (const double *)t.side_wl,
                       (const double *)t.side_w2k, (const double *)t.side_w2l, n, part);
    hipLaunchKernelGGL(d2loss_dside2 ? grad_final<true> : grad_final<false>, dim3(1), dim3(kSumBlocks), 0, st,
                       (const double *)part, n_blocks, d2loss_uniform, (const double *)t.scalars, dots);
    MC_HIP_CHECK(hipGetLastError());
    double d[4];
    MC_HIP_CHECK(wait_result(d, 4, dots, host, st));
    // D = M_k / mu_s - M_L (mu_sca), -M_L (mu_abs); Q likewise from the w^2 moments.
    const double gq_s = d[2] / mu_s - d[3], gq_a = -d[3];
    out_grad[0] = (d[0] / mu_s - d[1]) - gq_s;
    out_grad[1] = -d[1] - gq_a;
    const bool have_sigma = m.sigma_sca_mm2 != 0.0 || m.sigma_abs_mm2 != 0.0;
    out_grad[2] = have_sigma ? m.sigma_sca_mm2 * out_grad[0] + m.sigma_abs_mm2 * out_grad[1] : NAN;
    return MC_OK;
}

extern "C" int mc_side_l2(const mc_detector_t *detector, const mc_tally_t *tally, const double *target,
                          double *dloss_dside, double *loss, void *stream)
{
    using namespace mcmie;
    clear_error();
    if (!detector || !tally || !target || !dloss_dside || !loss) return fail(MC_EINVAL, "mc_side_l2: null argument");
    const mc_detector_t det = *detector;
    const mc_tally_t t = *tally;
    if (det.side_nx < 1 || det.side_ny < 1) return fail(MC_EINVAL, "mc_side_l2: side image dimensions must be >= 1");
    if (det.flags & MC_FIX64) return fail(MC_EINVAL, "mc_side_l2: needs a double side image (no MC_FIX64)");
    if (!t.side || !t.scalars) return fail(MC_EINVAL, "mc_side_l2: the tally has no side image or scalars");
    if (!t.workspace || ((uintptr_t)t.workspace & 7) || t.workspace_bytes < (kWsScalarWords + 1) * 8)
        return fail(MC_EINVAL, "mc_side_l2: workspace of at least %llu bytes required",
                    (unsigned long long)((kWsScalarWords + 1) * 8));
    hipStream_t st = (hipStream_t)stream;
    const uint64_t n = (uint64_t)det.side_nx * det.side_ny;
    double *part = (double *)t.workspace + kWsScalarWords;   // as mc_grad's
    const uint32_t n_blocks = sum_blocks<1>(n, t.workspace_bytes / 8 - kWsScalarWords);
    hipLaunchKernelGGL(l2_partial, dim3(n_blocks), dim3(kSumThreads), 0, st, (const double *)t.side, target, n,
                       dloss_dside, part);
    hipLaunchKernelGGL(l2_final, dim3(1), dim3(kSumBlocks), 0, st, (const double *)part, n_blocks,
                       (const double *)t.scalars, loss);
    MC_HIP_CHECK(hipGetLastError());
    return MC_OK;
}

extern "C" int mc_philox_blocks(uint64_t seed, uint32_t instance, const uint64_t *ids, uint64_t n_ids,
                                uint32_t step0, uint32_t n_steps, uint32_t *out, void *stream)
{
    using namespace mcmie;
    clear_error();
    if (n_ids == 0 || n_steps == 0) return MC_OK;
    if (!ids || !out) return fail(MC_EINVAL, "mc_philox_blocks: null buffer");
    if ((uint64_t)step0 + n_steps > (1ull << 32)) return fail(MC_EINVAL, "mc_philox_blocks: step range overflows");
    const uint64_t total = n_ids * (uint64_t)n_steps;
    if (total / n_steps != n_ids || total > (1ull << 40)) return fail(MC_EINVAL, "mc_philox_blocks: too many blocks");
    const uint64_t grid = (total + 255) / 256;
    hipLaunchKernelGGL(philox_blocks_kernel, dim3((uint32_t)grid), dim3(256), 0, (hipStream_t)stream,
                       (uint32_t)seed, (uint32_t)(seed >> 32), instance, ids, n_ids, step0, n_steps, out);
    MC_HIP_CHECK(hipGetLastError());
    return MC_OK;
}
