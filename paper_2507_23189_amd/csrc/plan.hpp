// The launch plan of a walk: workspace layout, launch shape, tally path and the
// rules they follow, as host code without a device, so that it can be checked
// for any size without a launch.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "mcmie.h"

namespace mcmie {

constexpr int kCopies = 8;                 // per-XCD image copies in the workspace (at most)
constexpr uint64_t kFewPhotons = 1 << 20;  // launches up to here take no exit log and fewer image copies
constexpr uint64_t kLogBinBlocks = 512;    // log_bin blocks that fill the chip (two per CU)
constexpr int kQueue = 64;                 // queued image exits per wave
constexpr int kBatchScal = 16;             // LDS scalar words per medium in a batched launch
// LDS scalar words (of the first medium) that tally nothing, the totals of the
// imaged faces being taken from their images, and hold what the block keeps beside
// its tallies: its pool of photon ids and the exits that found the log full.  (Words
// of their own would cost the largest batch, whose scalars and queues fill half a
// CU's LDS to the byte, the second block of every CU.)
constexpr int kLdsPool = MC_S_FACE + 1, kLdsFull = MC_S_FACE + 5;
constexpr uint64_t kWsScalarWords = 32;    // workspace scalar words per medium
constexpr uint32_t kLogMinRangeBits = 6;
constexpr uint32_t kLogHistBits = 13;      // keys per binning block: 2^13 (64 KB of int64 sums)
constexpr size_t kBatchInstBytes = 48;     // a batched launch's schedule entry (BatchInst)

// Workspace layout: per medium kWsScalarWords uint64 scalar words (0..14
// fixed-point scalar sums, 15 the photon work counter (first medium), 16..18
// FP64 second-order side moments, 24..27 mc_grad's dot products), then
// kCopies fixed-point copies of the images of every medium (and of the
// squared-weight images with MC_SIGMA); a batched launch appends its schedule
// (one BatchInst per medium).
inline uint64_t workspace_words(const mc_detector_t &d, uint64_t n_inst = 1, uint64_t copies = kCopies)
{
    const uint64_t n_pix = (uint64_t)d.side_nx * d.side_ny + (uint64_t)d.trans_nx * d.trans_ny;
    return kWsScalarWords * n_inst + copies * n_pix * n_inst * ((d.flags & MC_SIGMA) ? 2 : 1);
}

// The exit log (MC_EXIT_LOG) follows the workspace words (and a batched
// launch's schedule): the counts of 2^rbits x blocks regions (uint32, padded
// to 8 bytes), then the regions of cap entries each, with cap the largest
// the caller's workspace holds.  The key width and range bits follow from
// the number of keys: a range of at most 2^kLogHistBits keys where the LDS
// takes 2^rbits counters (up to 2^8 beside a Mie table, 2^12 otherwise).
constexpr uint64_t kLogSizingBlocks = 256 * 2;   // resident blocks of a full MI355X launch
struct LogShape {
    uint32_t bits, rbits;
};
inline LogShape log_shape(uint64_t n_keys, bool table_in_lds)
{
    const uint64_t groups = (n_keys + 7) / 8;
    uint32_t bits = 1;
    while ((1ull << bits) < groups) ++bits;
    const uint32_t max_r = table_in_lds ? 8u : 12u;
    const uint32_t want = bits > kLogHistBits - 3 ? bits - (kLogHistBits - 3) : 0u;
    const uint32_t rbits = std::min(max_r, std::max(kLogMinRangeBits, want));
    return {std::max(bits, rbits), rbits};
}
// Region capacities are whole granules of entries: 256 (2 KiB of region
// stride) from 1024 entries up, else 64.  The binning pass streams thousands
// of regions at once, one per wave, and its read rate depends on their
// stride: at 512 blocks x 64 regions of 2100 entries, every capacity of a
// multiple of 256 entries from 2304 to 8192 read at 5.5-5.9 TB/s, while some
// other capacities lost up to a quarter of that (4640 or 4641 entries:
// 4.6 TB/s; 8128: 4.3 TB/s).
inline uint64_t log_cap_granule(uint64_t cap) { return cap >= 1024 ? 256 : 64; }
inline uint32_t log_cap_for(uint64_t extra_bytes, uint64_t regions)
{
    const uint64_t count_bytes = (regions * 4 + 7) / 8 * 8;
    if (regions == 0 || extra_bytes < count_bytes) return 0;
    uint64_t cap = (extra_bytes - count_bytes) / (regions * 8);
    // Entry positions are 32-bit.
    cap = std::min<uint64_t>(cap, 0x7FFFFF00ull);
    if (cap >= 64) cap -= cap % log_cap_granule(cap);
    return (uint32_t)cap;
}
// Log bytes for n_photons over `regions` regions: each photon leaves through an
// image at most once; spread evenly over the ranges and the blocks of a full
// launch, a region gets about n / regions entries, and holds half as many again
// (for uneven spread and unequal shares of photons) plus 64, rounded up to a
// whole granule (so that log_cap_for gives back exactly this capacity).
inline uint64_t log_bytes_for(uint64_t n_photons, uint64_t regions)
{
    uint64_t cap = std::min<uint64_t>((n_photons + n_photons / 2 + regions - 1) / regions + 64, 0x7FFFFF00ull);
    const uint64_t gr = log_cap_granule(cap);
    cap = (cap + gr - 1) / gr * gr;
    return (regions * 4 + 7) / 8 * 8 + regions * cap * 8;
}

inline uint64_t batch_workspace_words(const mc_detector_t &d, uint64_t n_items)
{
    return workspace_words(d, n_items) + (n_items * kBatchInstBytes + 7) / 8;
}

constexpr uint32_t kRefillMin = 28;        // lanes of a wave not walking that trigger a round (batched)

// The same for a single medium of optical depth tau along the beam axis.  A
// high threshold shares a round among more photons, a low one keeps more lanes
// walking.  From a sweep of thresholds 8..58 at tau = 0.5..16 (mc_simulate,
// 1e8 photons, 512 x 512, exit log; ms at 12 / 20 / 24 / 28 / 34 (mean of 32
// and 36) / 40): tau = 1 1.42 / 1.41 / 1.42 / 1.39 / 1.33 / 1.32; tau = 2 2.09 /
// 1.94 / 1.79 / 1.76 / 1.76 / 1.77; tau = 4 2.87 / 2.51 / 2.45 / 2.42 / 2.41 /
// 2.42; tau = 8 4.20 / 3.79 / 3.76 / 3.79 / 3.86 / 3.98; tau = 12 5.50 / 5.22 /
// 5.14 / 5.21 / 5.44 / 5.74; tau = 16 6.92 / 6.59 / 6.68 / 6.83 / 7.12 / 7.53.
// HG and path-moment walks have the same optima.
inline uint32_t refill_min_for(double tau)
{
    if (!(tau >= 0.0)) return kRefillMin;
    return tau < 5.0 ? 34 : (tau < 14.0 ? 24 : 20);
}

// Photon ids a wave takes from its block's pool at once (single medium, when
// the caller leaves it to the library), or photons of a batch's work unit.  A
// large chunk leaves fewer rounds short of ids, a small one shares the end of
// the launch better: mc_simulate at 256 / 512 ids, 1e8 photons, 512 x 512: tau
// = 0.5 1.028 / 1.001 ms, tau = 1 1.254 / 1.238, tau = 4 2.328 / 2.318; 1e7
// photons, tau = 16: 0.842 / 0.901.  A batch of 256 media at units of 128 / 256
// / 512 photons: 18.9 / 18.6 / 18.9 ms, with 1/256 of its photons 0.790 / 0.806 /
// 0.837.
inline uint64_t chunk_for(uint64_t total_photons, uint64_t waves_total, bool batch)
{
    const uint64_t chunk = std::min<uint64_t>(batch ? 256 : 512,
                                              total_photons / std::max<uint64_t>(1, waves_total * (batch ? 16 : 6)));
    return std::max<uint64_t>(64, (chunk + 63) / 64 * 64);
}

// How the blocks of a walk get their ids (or a batch's work units): see
// Claims, WalkArgs::claim0 and kPoolFilling.  Every claim from the global counter is one
// device-scope atomic on one word, which takes about 78 million per second.
// When each wave claimed for itself that rate set the time of any launch up
// to 1e7 photons (tau = 4: 1e5 0.19 ms, 1e6 0.37, 1e7 1.13); with a pool per
// block these take 0.05, 0.11 and 0.33.
//   * Up to four photons per lane, the ids are dealt out in equal shares and
//     nothing is claimed (2e6 photons, shares / claims: tau = 1 0.116 / 0.132
//     ms, tau = 4 0.140 / 0.150, tau = 16 0.309 / 0.305).
//   * Beyond that a block starts with a quarter of its share and claims a
//     fixed part of what it last saw left, down to four chunks: many claims
//     where there is time for them, small ones at the end.  Parts of 1/4, 1/8
//     and 1/16 of a share: tau = 4, 1e8 2.328 / 2.339 / 2.389 ms; tau = 16,
//     1e8 6.61 / 6.55 / 6.56; tau = 16, 1e9 64.5 / 63.7 / 63.5.
//   * A batch takes its units in order, eight at a time, so that all blocks
//     work on the same few media at any time: claimed by shares, each block's
//     exits were those of one medium, overflowed its regions of the log, and
//     256 media took 48 ms instead of 18.6.
struct Claims {
    uint32_t claim0, claim_min, claim_shift;
};
inline Claims claims_for(uint64_t units, uint64_t grid, uint64_t block, uint64_t chunk, double tau_z, bool batch)
{
    Claims a{};
    if (batch) {
        a.claim_shift = 31;
        a.claim_min = 8;
        a.claim0 = (uint32_t)std::min<uint64_t>(8, (units + grid - 1) / grid);
        return a;
    }
    const double work = (double)units * (1.0 + tau_z);
    const uint64_t parts = grid * (work < 1e9 ? 4 : (work < 1e10 ? 8 : 16));
    a.claim_shift = 2;
    while (a.claim_shift < 31 && (1ull << a.claim_shift) < parts) ++a.claim_shift;
    a.claim_min = (uint32_t)(4 * chunk);
    const uint64_t even = (units + grid - 1) / grid;
    a.claim0 = (uint32_t)(even <= 4 * block ? even : std::max<uint64_t>(even / 4, chunk));
    return a;
}


// A CU's LDS is handed out in granules (measured: 9 blocks of 17,908 bytes run at
// once but only 8 of 18,036, 5 of 31,960 but 4 of 32,088, 3 of 53,677 but 2 of 53,805).
constexpr size_t kCuLds = 160 * 1024, kLdsGranule = 1280;
// Blocks of `block` lanes and `lds` bytes that run on a CU at once.
inline size_t blocks_on_cu(size_t lds, int block)
{
    const size_t granules = (lds + kLdsGranule - 1) / kLdsGranule;
    return std::max<size_t>(1, std::min<size_t>(kCuLds / kLdsGranule / granules, 32 / (block / 64)));
}

// The countdown to a wave's next look at roulette and the step cap, at a round: 0
// when a photon took a step there (the look is due), else never below 0, so that
// the steps between two rounds, at most 2^24, cannot carry it past the least
// integer, where it would turn into a long stretch without looks.
constexpr int calm_at_round(int calm, bool stepped) { return stepped || calm < 0 ? 0 : calm; }

// What a walk's plan depends on.
struct WalkRequest {
    bool batch;
    int phase, n_cdf;             // n_cdf: 0 without a table
    uint32_t n_inst;
    uint64_t n_pix;               // pixels of one medium's images
    uint32_t flags;               // of the detector
    uint64_t photons;             // over all media
    // Photons of the launch whose tally path is taken (log or not, copies, their
    // order, slots): more than `photons` when a sample of a launch is timed for it.
    uint64_t path_photons;
    int block_size, grid_blocks;  // the caller's, 0: the library's choice
    uint32_t chunk;
    double tau_z;                 // optical depth along the beam axis (negative: a batch)
    int cus;
    uint64_t max_copies;          // image copies the workspace has room for
    uint64_t ws_bytes;
};

struct WalkPlan {
    bool use_log;
    int block, grid, cache_bits;
    size_t lds;
    LogShape shape;
    uint32_t parts;               // log_bin blocks per range and copy
    uint64_t copies, n_cleared;   // image copies in use; those that take the walk's atomics under the log
    bool permuted;                // the copies' pixels are permuted (spread_pixel)
    uint64_t ws_words, log_at;    // words of the scalars and copies; first word of the log
    uint32_t log_cap;             // entries of a log region
    uint64_t chunk;
    uint32_t refill_min;
};

inline WalkPlan plan_walk(const WalkRequest &q)
{
    WalkPlan p{};
    const bool batch = q.batch;
    const uint64_t total_photons = q.path_photons, n_total = q.n_pix * q.n_inst, copy_words = n_total * ((q.flags & MC_SIGMA) ? 2 : 1);
    // A batched launch keeps its schedule after the workspace words; the exit
    // log follows: its counts, then the regions.  A workspace without room for
    // the counts takes the atomic path (the same sums).
    const uint64_t sched_words = batch ? (q.n_inst * kBatchInstBytes + 7) / 8 : 0;
    const LogShape shape = p.shape = log_shape(n_total, !batch && q.phase == MC_PHASE_MIE);
    // Keys of a range have indices below 2^(bits - rbits + 3); log_bin takes
    // them in parts of 2^kLogHistBits.
    const uint64_t per_range = 1ull << (shape.bits - shape.rbits + 3);
    p.parts = (uint32_t)((per_range + (1u << kLogHistBits) - 1) >> kLogHistBits);
    // With the exit log the image copies take log_bin's sums (and the rare
    // fallback atomics): as many copies as give it kLogBinBlocks blocks, so
    // that fine key ranges (large images, batches) leave fewer copies to clear
    // and to sum.  Without it, one per XCD for the image atomics, or one or two
    // in all where the atomics are too few to make up for clearing and summing
    // the others, which takes about 3 ps per pixel and copy (a single copy costs
    // up to 20 ps per photon in waiting).  1, 2 and 8 copies, us, tau = 1: 1e5
    // photons, 512 x 512 49.2 / 51.3 / 66.5; 1e6, 256 x 256 80.9 / 70.6 / 74.5; 1e6, 1024 x
    // 1024 91.5 / 91.7 / 111.9; 3e6, 512 x 512 196 / 197 / 150.  The
    // workspace layout keeps room for all of them either way (the schedule and
    // the log start at the same place); the copies in use come first.
    auto copies_for = [&](bool log) -> uint64_t {
        if (!log) {
            if (total_photons > std::max<uint64_t>(kFewPhotons, n_total)) return q.max_copies;
            return std::min<uint64_t>(q.max_copies, total_photons > kFewPhotons / 2 ? 2 : 1);
        }
        const uint64_t bin_blocks = ((uint64_t)1 << shape.rbits) * p.parts;
        uint64_t c = 1;
        while (c < q.max_copies && bin_blocks * c < kLogBinBlocks) c <<= 1;
        return c;
    };

    // ---- launch shape: 1024-lane blocks (768 with path moments), two per CU, each with
    // the table (single medium), the scalar words, the per-wave exit queues and
    // as large a tally cache as fits in half the CU's 160 KB LDS, or, with the exit
    // log, the block's append counters and a cache for what overflows it ----
    // Path-moment kernels are built for six waves per SIMD: 768-lane blocks,
    // two per CU.
    const int own_block = (q.flags & MC_MOMENTS) ? 768 : 1024;
    const int block = p.block = q.block_size ? q.block_size : own_block;
    const size_t table_bytes = batch ? 0 : (size_t)((q.n_cdf + 3) & ~3) * sizeof(float);
    const size_t scal_bytes = (batch ? (size_t)q.n_inst * kBatchScal : MC_N_SCALARS) * sizeof(double);
    const size_t queue_arrays = batch ? 4 : 3;
    const size_t slot_bytes = sizeof(uint32_t) + sizeof(double) * ((q.flags & MC_SIGMA) ? 2 : 1);
    const size_t lds_half_cu = 80 * 1024;
    const double tau_z = q.tau_z;
    // Few photons take one block per CU: half the tables to load, half the
    // shares to finish, and the same lanes with twice the photons each.  Up to
    // three photons per lane of such a launch, four from depth 3 and five from
    // depth 6 (deep walks hide more of each photon's end); but below half a
    // photon per lane at depth 12 and more two blocks spread the
    // long walks over more waves.  Times in us of two blocks and of one: 1e5
    // tau = 4 57.6 / 53.4, 3e5 tau = 2 63.2 / 58.2, 7e5 tau = 0.25 109.7 / 104.9, tau = 16
    // 209 / 167; 1e6 tau = 1 73.9 / 76.0, tau = 4 88.7 / 83.9, tau = 16 219 / 194; 2e6
    // tau = 4 117.5 / 118.5; 1e4 tau = 16 94.7 / 97.9.  (All with the library's block.)
    const uint64_t lanes_one = (uint64_t)q.cus * block;
    const bool few = !batch && block == own_block && q.photons <= lanes_one * (tau_z > 6.0 ? 5 : (tau_z > 3.0 ? 4 : 3)) &&
                     !(tau_z > 12.0 && q.photons < lanes_one / 2);
    // Slots of the tally cache at most (log2), where the LDS holds them.  At the end
    // every block adds its slots to the images, many of them to the same words, so
    // few photons, or few pixels, pay for more slots than they use, and squared weights
    // double what a slot saves.  Us at 8 / 10 / 12, HG: 1e6 photons, tau = 4, 512 x 512
    // 84.7 / 87.0 / 101.3, tau = 1 70.0 / 80.5 / 83.5.  At 10 / 11 / 12, tau = 1, HG (4096 entries,
    // tau = 4, in brackets), by pixels of both images: 9e6 photons, 16200 177 / 200 / 219 (281 /
    // 294 / 322), 65522 225 / 216 / 228 (297 / 293 / 324), 131072 255 / 243 / 233 (325 / 324 / 330; tau = 8,
    // HG, 11 and 12 436 / 480); 2e7, 8192 286 / 309 / 336 (523 / 534 / 557), 16200 367 / 325 / 358 (571 /
    // 543 / 569), 131072 469 / 435 / 405 (641 / 615 / 581; tau = 8 897 / 925),
    // 524288 515 / 503 / 495 (681 / 684 / 684); 5e7, 32768 795 / 653 / 664 (1220 /
    // 1200 / 1221), 65522 985 / 881 / 703 (1429 / 1288 / 1230), 524288 1160 / 1118 / 1070 (1545 / 1535 / 1503);
    // 2e8, 8192 2265 / 2276 / 2300 (4529 / 4531 / 4554), 16200 3150 / 2293 / 2309 (5255 / 4535 / 4560), 65522
    // 3798 / 3255 / 2547 (5566 / 5062 / 4568).  Batches (whose first media fill the slots)
    // and the exit log's overflow do not tell 10 from 12, and smaller blocks would fit
    // a CU in smaller numbers.
    auto slots_for = [&](bool log) -> int {
        if (log || batch || block != own_block) return 10;
        if (total_photons <= 1u << 20) return (q.flags & MC_SIGMA) ? 10 : 8;
        if (total_photons < 1u << 23) return 10;
        if (total_photons < 1u << 24) return n_total > 1u << 16 ? 11 : 10;
        return n_total <= 1u << 13 ? 10 : (n_total <= 1u << (total_photons < 1u << 25 ? 18 : 15) ? 11 : 12);
    };
    auto launch_shape = [&](bool log) {
        const size_t lds_fixed = table_bytes + scal_bytes + (size_t)(block / 64) * queue_arrays * kQueue * sizeof(float) +
                                 (log ? ((size_t)4 << shape.rbits) : 0);
        // (Under the log the cache, for its overflow alone, takes only LDS that no
        // further block could use: blocks of 64 lanes with a 4096-entry table, 5e7
        // photons, tau = 1, 1.41 ms with 32 slots and 8 blocks a CU, 1.15 with 16 and 9.)
        const size_t fit = std::max<size_t>(1, std::min<size_t>(kCuLds / lds_fixed, 32 / (block / 64)));
        const size_t granules = kCuLds / kLdsGranule / blocks_on_cu(lds_fixed, block);
        const size_t lds_most = log ? std::min({lds_half_cu, kCuLds / fit, granules * kLdsGranule}) : lds_half_cu;
        p.cache_bits = 0;
        for (int b = slots_for(log); b >= 4; --b)
            if (lds_fixed + (slot_bytes << b) <= lds_most) { p.cache_bits = b; break; }
        p.lds = lds_fixed + (p.cache_bits ? (slot_bytes << p.cache_bits) : 0);
        const int blocks_per_cu = std::max(1, std::min((int)(kCuLds / p.lds), 32 / (block / 64)));
        p.grid = q.grid_blocks > 0 ? q.grid_blocks : q.cus * (few ? 1 : blocks_per_cu);
    };
    const uint64_t ws_words = p.ws_words = kWsScalarWords * q.n_inst + q.max_copies * copy_words;
    // So few exits are not worth the log's second pass over them (log and
    // atomics, us, tau = 4: 1e5 photons, 512 x 512 74.9 / 53.8, 1024 x 1024 83.2 / 68.2;
    // 1e6 103.4 / 85.6 and 116.4 / 97.6; 3e6, tau = 1, 512 x 512 134 / 150).  A
    // caller that sets the grid keeps the log: these are times of full launches.
    bool use_log = (q.flags & MC_EXIT_LOG) != 0 && (total_photons > kFewPhotons || q.grid_blocks > 0);
    launch_shape(use_log);
    if (use_log && q.ws_bytes / 8 < ws_words + sched_words + (((uint64_t)p.grid << shape.rbits) * 4 + 7) / 8) {
        use_log = false;
        launch_shape(false);
    }
    // The log's place: words [log_at, log_end) of the workspace, what the caller
    // gave beyond the scalar words, the copies and the schedule.
    p.log_at = ws_words + sched_words;
    uint64_t log_end = q.ws_bytes / 8;
    // Without the flag, large images and batches leave most of their eight copies
    // unused if the exits go through a log: where that room takes three exits of
    // five or more, they do (us with atomics / so: 1e7 photons, tau = 1, 1024 x 1024
    // 335 / 221, 850 x 850 386 / 225, tau = 4 408 / 340; 223 media of 191 x 294 and
    // 5.8e7 photons with squares 5015 / 3080; room for two of three 6540 / 5560, for
    // two of five 1470 / 1795).  Below 2^21 photons it is even, or loses up to 6 %
    // (1.5e6, 725 x 725, tau = 0.5 124 / 129, tau = 1 117 / 111; 3e6 165 / 148).  Where the
    // log's counters cost the second block of every CU (batches from 385 media) it takes
    // room for nine of ten, unless squares double the atomics (450 to 511 media, so /
    // with atomics: room for 0.66 0.96 to 1.58, for 0.75 0.93 to 1.11, for 0.98 0.91 to 0.96, for 1.12
    // 0.88 to 0.95, for 1.4 0.89 to 0.92; squares, 0.7 0.86 to 1.0, 0.8 0.76 to 0.86, 1.0 0.63).
    if (!(q.flags & (MC_EXIT_LOG | MC_RECORD)) && q.grid_blocks <= 0 &&
        total_photons > std::max<uint64_t>(1u << 21, n_total)) {
        const uint64_t at = kWsScalarWords * q.n_inst + copies_for(true) * copy_words;
        const int grid = p.grid;
        launch_shape(true);
        const uint64_t regions = ((uint64_t)1 << shape.rbits) * p.grid;
        const uint64_t tenths = p.grid < grid && !(q.flags & MC_SIGMA) ? 9 : 6;
        use_log = at < ws_words && 10 * regions * log_cap_for((ws_words - at) * 8, regions) >= tenths * total_photons;
        if (use_log) {
            p.log_at = at;
            log_end = ws_words;
        } else {
            launch_shape(false);
        }
    }
    p.use_log = use_log;
    p.copies = copies_for(use_log);
    // With the exit log the walk's only image atomics are its fallback ones
    // (an exit whose region is full and whose pixel has no slot in the cache):
    // all of them go to copy 0, the only one to be cleared.  Many photons in
    // small images leave so many that they take a copy per XCD as well (1e8 at
    // optical depth 1, 128 x 128: 6.0 ms on copy 0, 1.44 spread; 1e7: 196.5 us
    // and 199.4, of which clearing is the difference; 256 x 256 and 1e8: 1.26
    // and 1.23 ms).
    const bool spread = n_total <= (1u << 17) && total_photons >= (1u << 24);
    p.n_cleared = use_log && !spread ? 1 : p.copies;
    // Permuted copies pay where many exits meet (tau = 1, in order and
    // permuted, us: 1e7 photons, 150 x 150 295 / 230, 512 x 512 335 / 303, 700 x 700
    // 384 / 332, but 1024 x 1024 340 / 346; 1e8 2505 / 1847, 2523 / 2317, 3208 / 2540, 2585 /
    // 2434; 3e6, 150 x 150 122 / 127, 700 x 700 154 / 155; batches of 37 to 250 media 2
    // to 9 % less).
    p.permuted = !use_log && total_photons > std::max<uint64_t>(1u << 22, 8 * n_total);
    const uint64_t waves_total = (uint64_t)p.grid * (block / 64);
    p.chunk = q.chunk;
    if (p.chunk == 0) p.chunk = chunk_for(q.photons, waves_total, batch);
    // Work units are counted in 31 bits.
    if (batch) p.chunk = std::max<uint64_t>(p.chunk, q.photons >> 29);
    // Refill threshold from the optical depth; batched launches take the
    // fixed one (256 media, ms at 12 / 20 / 24 / 28 / 32 / 40: 20.5 / 19.3 /
    // 19.05 / 18.97 / 19.01 / 19.5).
    p.refill_min = batch ? kRefillMin : refill_min_for(tau_z >= 0.0 ? tau_z : 0.0);

    if (use_log) p.log_cap = log_end > p.log_at ? log_cap_for((log_end - p.log_at) * 8, ((uint64_t)1 << shape.rbits) * p.grid) : 0;
    return p;
}

}  // namespace mcmie
