// Mie phase-function table on the device, FP64 (Sec. 2.2-2.6, Sec. 3.1.2).
//
// Two kernels build one table:
//   mie_phase_kernel, four lanes per angle, 256-lane workgroups:
//   1. every workgroup runs the Bohren-Huffman series (Sec. 2.5) for itself:
//      one lane runs the logarithmic derivative D_n(mx) by downward
//      recurrence (in homogeneous form, D_n = P_n / Q_n, so the serial chain
//      holds no division; from 256 steps all lanes of its wave share them)
//      while a lane of another wave runs psi_n(x) and chi_n(x) upward; then every
//      lane forms a_n and b_n for its n (Eqs. 7-8 divided through by psi_n(mx)),
//      and Q_ext (Eq. 13), Q_sca and the asymmetry sums (Eq. 12) are added in a
//      fixed order;
//   2. four lanes evaluate S1, S2 (Eqs. 5-6) at an angle, one each of their real
//      and imaginary parts, with the angular functions pi_n, tau_n by upward
//      recurrence (the per-n divisions done once beforehand), giving the phase
//      function normalised so that (1/4pi) int P dOmega = 1 (Eqs. 9-10);
//      P sin(theta) goes to a device buffer of n_angles doubles;
//   mie_inverse_kernel, one lane per inverse-table entry, 1024-lane groups:
//   3. every workgroup reads the whole P sin(theta) grid into LDS and forms
//      its trapezoid CDF by a block scan;
//   4. each inverse-table entry u_i = i/(N-1) finds the first angle with
//      F >= u_i by binary search and interpolates theta linearly; the table
//      stores v = 1 - cos(theta) = 2 sin^2(theta/2) in FP32.
// A size distribution has a workgroup per bin and 256 angles, one lane each
// (mie_bin_kernel): there the series of many bins fills the chip, and four times
// the workgroups would repeat it four times as often (58 us for 64 bins against
// 22).
//
// All of it is bound by the serial chains: a dependent FP64 fma takes about 33
// cycles on a lone wave, four of them a downward step (two for a real index),
// two a term of a sum.  The 100 um absorbing sphere (x = 785) took 57 us of
// downward steps one after the other, hidden behind them 18 of upward ones (33
// with a division in each), and 30 of sums; with the downward steps shared it is
// the upward ones and the sums, 57 us for the kernel from 105.  The 5 um sphere
// takes 4.7 and 2.9 of the kernel's 12.  Before (one lane per angle, factors
// formed in the steps, eight fma in every downward step) mie_phase_kernel took
// 14.4 us at 5 um and 133 at 100 um, the 64 bins 26.5.
// Arrays live in LDS (coefficients 32 KB, pi_n recurrence coefficients 16 KB,
// psi and chi 16 KB, factors 6 KB, angle grid 24 KB at the limits; gfx950 gives
// a workgroup up to 160 KB).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "common.hpp"

namespace mcmie {
namespace {

constexpr int kPhaseThreads = 256;    // phase kernels
constexpr int kAngles = kPhaseThreads / 4;   // angles of a workgroup of mie_phase_kernel
constexpr int kInvThreads = 1024;     // CDF and inverse: one entry per lane, 1..3 angles per lane in the scan

struct cplx {
    double re, im;
};
__device__ __forceinline__ cplx operator-(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cplx operator*(cplx a, cplx b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cplx operator*(double s, cplx a) { return {s * a.re, s * a.im}; }
__device__ __forceinline__ cplx operator+(cplx a, double s) { return {a.re + s, a.im}; }
// Smith's division: no overflow of |b|^2 for large operands.
__device__ __forceinline__ cplx operator/(cplx a, cplx b)
{
    if (fabs(b.re) >= fabs(b.im)) {
        const double r = b.im / b.re, den = b.re + b.im * r;
        return {(a.re + a.im * r) / den, (a.im - a.re * r) / den};
    }
    const double r = b.re / b.im, den = b.re * r + b.im;
    return {(a.re * r + a.im) / den, (a.im * r - a.re) / den};
}
__device__ __forceinline__ double norm2(cplx a) { return a.re * a.re + a.im * a.im; }

// sin(t) for |t| <= pi/2 from its Taylor series through t^19/19!, in Horner
// form in t^2 (truncation below (pi/2)^21/21! < 3e-16): no range reduction is
// needed on this interval.
__device__ __forceinline__ double sin_half_pi(double t)
{
    const double s = t * t;
    double p = 1.0 / 121645100408832000.0;               // 1/19!
    p = fma(p, s, -1.0 / 355687428096000.0);             // -1/17!
    p = fma(p, s, 1.0 / 1307674368000.0);                // 1/15!
    p = fma(p, s, -1.0 / 6227020800.0);                  // -1/13!
    p = fma(p, s, 1.0 / 39916800.0);                     // 1/11!
    p = fma(p, s, -1.0 / 362880.0);                      // -1/9!
    p = fma(p, s, 1.0 / 5040.0);                         // 1/7!
    p = fma(p, s, -1.0 / 120.0);                         // -1/5!
    p = fma(p, s, 1.0 / 6.0);                            // 1/3! (subtracted below)
    return t - t * s * p;
}
// sin and cos of theta in [0, pi].  sin by reflection onto [0, pi/2];
// cos as 1 - 2 sin^2(theta/2) (or its mirror about pi/2), which keeps full
// accuracy where cos is near +-1 and the angular functions are most sensitive.
__device__ __forceinline__ double sin_0_pi(double th) { return sin_half_pi(th <= 0.5 * M_PI ? th : M_PI - th); }
__device__ __forceinline__ double cos_0_pi(double th)
{
    const bool back = th > 0.5 * M_PI;
    const double h = sin_half_pi(0.5 * (back ? M_PI - th : th));
    const double c = 1.0 - 2.0 * h * h;
    return back ? -c : c;
}

struct MieArgs {
    double x, m_re, m_im;
    int n_terms, n_start, n_angles, n_cdf;
    float *inv_cdf;
    double *phase, *cdf, *coef;
    double *result;          // q_ext, q_sca, g, n_terms
    double *host_result;     // the same again, pinned host memory (optional)
    double *work;            // n_angles: P(theta_j) sin(theta_j), from the phase kernel to the inverse kernel
};

// The serial recurrences run on one lane of a wave of their own, whose
// instruction count is their time (a lone wave issues one instruction every
// four cycles or more).  So its 64 lanes first form the factors of kChunk
// steps into LDS, and the lane's steps are the recurrence's own fma, a store,
// and a read of two factors ahead of their use, in groups of eight without
// branches.
// Downward recurrences of this many steps and more are taken by all lanes of the
// wave (downward_scan): below, the steps one after the other end at most a few
// us after the upward recurrence beside them (whole call, us, one after the other
// / shared, 1801 angles: x = 190 real 49.1 / 42.2, absorbing 56.9 / 42.3; x = 440
// 70.1 / 57.1 and 85.9 / 57.8; x = 785 101.7 / 78.4 and 127.9 / 79.4).
constexpr int kScanFrom = 256;
constexpr int kChunk = 256, kAhead = 16;   // kAhead: entries before the first that reading ahead may touch

// Orders LDS accesses of a wave's lanes: those before it come before those after
// it, for every lane (the hardware keeps a wave's accesses in order; this keeps the
// compiler from moving them past each other).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A vector (P, Q) of the downward recurrence, its step from n to n - 1 with
// k = n/(mx), and its scaling by a power of two (see mie_series_block).  With a
// real index the imaginary parts are zero and left out.
struct Ratio {
    cplx P, Q;
};
template <bool REAL>
__device__ __forceinline__ void down_step(Ratio &v, cplx k)
{
    if (REAL) {
        const double Q1 = fma(k.re, v.Q.re, v.P.re);
        v.P.re = fma(k.re, Q1, -v.Q.re);
        v.Q.re = Q1;
    } else {
        const cplx Q1 = {fma(k.re, v.Q.re, fma(-k.im, v.Q.im, v.P.re)), fma(k.re, v.Q.im, fma(k.im, v.Q.re, v.P.im))};
        v.P = {fma(k.re, Q1.re, fma(-k.im, Q1.im, -v.Q.re)), fma(k.re, Q1.im, fma(k.im, Q1.re, -v.Q.im))};
        v.Q = Q1;
    }
}
template <bool REAL>
__device__ __forceinline__ double largest(const Ratio &v)
{
    const double top = fmax(fabs(v.P.re), fabs(v.Q.re));
    return REAL ? top : fmax(fmax(top, fabs(v.P.im)), fabs(v.Q.im));
}
template <bool REAL>
__device__ __forceinline__ void scale_by(Ratio &v, int e)
{
    v.P.re = ldexp(v.P.re, e);
    v.Q.re = ldexp(v.Q.re, e);
    if (!REAL) {
        v.P.im = ldexp(v.P.im, e);
        v.Q.im = ldexp(v.Q.im, e);
    }
}

// The downward recurrence (see downward, below) by all lanes of a wave, for long
// series: its steps are matrices of determinant 1, so each lane multiplies
// those of its 64th of the steps (both columns at once), a scan over the lanes
// joins the products, and each lane takes its steps again from the vector that
// reaches them.  The chain is 2/64 of the steps and six products.  Errors of a_n
// and b_n against an 80-bit evaluation, 70 spheres of x = 165 to 801 with real
// and absorbing indices of 1.4 to 2.4: 1.5e-13 root mean square, 8e-13 at most
// (1.8e-13 and 1.1e-12 one after the other), two thirds of those in the geometric
// mean.
template <bool REAL>
__device__ __forceinline__ void downward_scan(double x, cplx m, int N, int n_start, cplx *s_a, cplx *s_b)
{
    const int lane = threadIdx.x & 63;
    const int len = (n_start + 63) / 64, top = n_start - lane * len;   // this lane's steps: n = top, top - 1, .. (n >= 1)
    const int steps = min(max(top, 0), len);
    // 1/(mx) as a sum of two doubles: its rounding would turn every step the same
    // way.  1 - mx h is exact up to the second order: its products are split by
    // fma, and the differences of their near-equal leading parts are exact.
    const cplx mx = {x * m.re, x * m.im};
    const cplx h = REAL ? cplx{1.0 / mx.re, 0.0} : cplx{1.0, 0.0} / mx;
    cplx l;
    {
        const double lr = fma(x, m.re, -mx.re), li = fma(x, m.im, -mx.im);
        const double p1 = mx.re * h.re, p2 = mx.im * h.im, p3 = mx.re * h.im, p4 = mx.im * h.re;
        const double e1 = fma(mx.re, h.re, -p1), e2 = fma(mx.im, h.im, -p2);
        const double e3 = fma(mx.re, h.im, -p3), e4 = fma(mx.im, h.re, -p4);
        const cplx r = {((1.0 - p1) + p2) + ((e2 - e1) + (li * h.im - lr * h.re)),
                        (-p3 - p4) - ((e3 + e4) + (lr * h.im + li * h.re))};
        l = REAL ? cplx{r.re * h.re, 0.0} : r * h;
    }
    auto factor = [&](int n) {
        const double d = n;
        return cplx{fma(d, h.re, d * l.re), REAL ? 0.0 : fma(d, h.im, d * l.im)};
    };
    // Columns of the product: where the steps take (1, 0) and (0, 1).
    Ratio c0 = {{1.0, 0.0}, {0.0, 0.0}}, c1 = {{0.0, 0.0}, {1.0, 0.0}};
    auto rescale = [&]() {
        int e;
        (void)frexp(fmax(largest<REAL>(c0), largest<REAL>(c1)), &e);
        scale_by<REAL>(c0, -e);
        scale_by<REAL>(c1, -e);
    };
    for (int i = 0; i < steps; ++i) {
        const cplx k = factor(top - i);
        down_step<REAL>(c0, k);
        down_step<REAL>(c1, k);
        if ((i & 7) == 7) rescale();
    }
    rescale();
    auto shifted = [&](const Ratio &v, int by) {
        Ratio r = {{__shfl_up(v.P.re, by), 0.0}, {__shfl_up(v.Q.re, by), 0.0}};
        if (!REAL) {
            r.P.im = __shfl_up(v.P.im, by);
            r.Q.im = __shfl_up(v.Q.im, by);
        }
        return r;
    };
    auto apply = [&](const Ratio &v) {   // (c0 c1) v
        if (REAL)
            return Ratio{{fma(c0.P.re, v.P.re, c1.P.re * v.Q.re), 0.0}, {fma(c0.Q.re, v.P.re, c1.Q.re * v.Q.re), 0.0}};
        auto dot = [](cplx a, cplx x, cplx b, cplx y) {
            return cplx{fma(a.re, x.re, fma(-a.im, x.im, fma(b.re, y.re, -b.im * y.im))),
                        fma(a.re, x.im, fma(a.im, x.re, fma(b.re, y.im, b.im * y.re)))};
        };
        return Ratio{dot(c0.P, v.P, c1.P, v.Q), dot(c0.Q, v.P, c1.Q, v.Q)};
    };
    for (int by = 1; by < 64; by *= 2) {
        const Ratio b0 = shifted(c0, by), b1 = shifted(c1, by);
        if (lane >= by) {
            const Ratio n0 = apply(b0), n1 = apply(b1);
            c0 = n0;
            c1 = n1;
            rescale();
        }
    }
    Ratio v = shifted(c1, 1);   // of D_{n_start} = 0: (0, 1)
    if (lane == 0) v = Ratio{{0.0, 0.0}, {1.0, 0.0}};
    for (int i = 0; i < steps; ++i) {
        const int n = top - i;
        if (n <= N) {
            s_a[n - 1] = REAL ? cplx{v.P.re, v.Q.re} : v.P;
            if (!REAL) s_b[n - 1] = v.Q;
        }
        down_step<REAL>(v, factor(n));
        if ((i & 7) == 7) {
            int e;
            (void)frexp(largest<REAL>(v), &e);
            scale_by<REAL>(v, -e);
        }
    }
}

// One wave's downward recurrence of D_n(mx) = P_n / Q_n from n_start (see
// mie_series_block): P_n to s_a and Q_n to s_b, index n - 1, for n = N..1.  For a
// real index all imaginary parts are zero and the steps leave them out: two fma
// instead of eight, P_n and Q_n stored as the pair s_a.
// s_k holds kAhead + kChunk factors n/(mx).
template <bool REAL>
__device__ __forceinline__ void downward(cplx inv_mx, int N, int n_start, double2 *s_k, cplx *s_a, cplx *s_b)
{
    const int lane = threadIdx.x & 63;
    Ratio v = {{0.0, 0.0}, {1.0, 0.0}};   // D_{n_start} = 0
    auto step = [&](cplx k) { down_step<REAL>(v, k); };
    auto rescale = [&]() {   // after each step from a multiple of 8
        int e;
        (void)frexp(largest<REAL>(v), &e);
        scale_by<REAL>(v, -e);
    };
    auto keep = [&](int n) {   // D_n = P_n / Q_n
        if (REAL) {
            s_a[n - 1] = cplx{v.P.re, v.Q.re};
        } else {
            s_a[n - 1] = v.P;
            s_b[n - 1] = v.Q;
        }
    };
    struct Eight {
        cplx k[8];   // of n, n - 1, .., n - 7
    };
    double *const s_kr = (double *)s_k;
    for (int top = n_start; top >= 1;) {
        // Steps top..bot of this chunk; bot is one past a multiple of 8.
        const int bot = (top - 1) / kChunk * kChunk + 1;
        for (int i = lane; i <= top - bot; i += 64) {
            const cplx k = (double)(bot + i) * inv_mx;
            if (REAL) s_kr[kAhead + i] = k.re;
            else s_k[kAhead + i] = double2{k.re, k.im};
        }
        wave_lds_order();
        if (lane == 0) {
            auto factor = [&](int n) -> cplx {
                if (REAL) return cplx{s_kr[kAhead + n - bot], 0.0};
                const double2 k = s_k[kAhead + n - bot];
                return cplx{k.x, k.y};
            };
            auto eight = [&](int n) {
                Eight e;
#pragma unroll
                for (int u = 0; u < 8; ++u) e.k[u] = factor(n - u);
                return e;
            };
            int n = top;
            auto one = [&]() {
                if (n <= N) keep(n);
                step(factor(n));
                if ((n & 7) == 0) rescale();
                --n;
            };
            auto group = [&](const Eight &e, bool kept) {   // n, a multiple of 8, .. n - 7
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (kept) keep(n - u);
                    step(e.k[u]);
                    if (u == 0) rescale();
                }
                n -= 8;
            };
            while (n >= bot && ((n & 7) || (n > N && n - 7 <= N))) one();
            // Two groups at a time, each reading the next one's factors first.
            // (Those beyond the chunk's end are not used.)
            Eight a = eight(n);
            while (n >= bot) {
                if (n > N && n - 7 <= N) {   // the group in which keeping starts
                    for (int u = 0; u < 8; ++u) one();
                    a = eight(n);
                    continue;
                }
                const Eight b = eight(n - 8);
                if (n <= N) group(a, true);
                else group(a, false);
                if (n < bot || (n > N && n - 7 <= N)) {
                    a = b;
                    continue;
                }
                a = eight(n - 8);
                if (n <= N) group(b, true);
                else group(b, false);
            }
        }
        wave_lds_order();
        top = bot - 1;
    }
}

// One wave's upward recurrences psi_n = (2n - 1)/x psi_{n-1} - psi_{n-2}, chi_n
// likewise, into s_rec at index n = 0..N.  s_f holds kChunk factors.
__device__ __forceinline__ void upward(double x, int N, double *s_f, double2 *s_rec)
{
    const int lane = threadIdx.x & 63;
    double psi_prev = cos(x), psi = sin(x);        // psi_{-1}, psi_0
    double chi_prev = -sin(x), chi = cos(x);       // chi_{-1}, chi_0
    if (lane == 0) s_rec[0] = double2{psi, chi};
    for (int n0 = 1; n0 <= N; n0 += kChunk) {
        const int steps = min(kChunk, N + 1 - n0);
        for (int i = lane; i < steps; i += 64) s_f[i] = (2.0 * (n0 + i) - 1.0) / x;
        wave_lds_order();
        if (lane == 0) {
            auto up = [&](int i, double f) {
                const double psi_n = f * psi - psi_prev;
                const double chi_n = f * chi - chi_prev;
                s_rec[n0 + i] = double2{psi_n, chi_n};
                psi_prev = psi;
                psi = psi_n;
                chi_prev = chi;
                chi = chi_n;
            };
            struct Eight {
                double f[8];
            };
            auto eight = [&](int i) {
                Eight e;
#pragma unroll
                for (int u = 0; u < 8; ++u) e.f[u] = s_f[min(i, kChunk - 8) + u];
                return e;
            };
            int i = 0;
            Eight a = eight(0);
            for (; i + 16 <= steps; i += 16) {
                const Eight b = eight(i + 8);
#pragma unroll
                for (int u = 0; u < 8; ++u) up(i + u, a.f[u]);
                a = eight(i + 16);
#pragma unroll
                for (int u = 0; u < 8; ++u) up(i + 8 + u, b.f[u]);
            }
            for (; i < steps; ++i) up(i, s_f[i]);
        }
        wave_lds_order();
    }
}

// v + its value 32, 16, .. 1 lanes across: the sum over the wave, in every lane,
// in that order.  Without LDS: halves and rows are exchanged by the permlane
// swaps; within a row of 16 a rotation by 8 is the lane 8 across, and after
// that step a rotation by 4 the lane 4 across.
__device__ __forceinline__ double wave_sum(double v)
{
    auto halves = [](double v, auto swap) {
        const int2 x = __builtin_bit_cast(int2, v);
        const auto lo = swap(x.x), hi = swap(x.y);
        return __builtin_bit_cast(double, int2{(int)lo[0], (int)hi[0]}) +
               __builtin_bit_cast(double, int2{(int)lo[1], (int)hi[1]});
    };
    auto row = [](double v, auto move) {
        const int2 x = __builtin_bit_cast(int2, v);
        return v + __builtin_bit_cast(double, int2{move(x.x), move(x.y)});
    };
    v = halves(v, [](int x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
    v = halves(v, [](int x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    v = row(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true); });   // row_ror:8
    v = row(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x124, 0xF, 0xF, true); });   // row_ror:4
    v = row(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true); });    // quad_perm 2301
    return row(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true); }); // quad_perm 1032
}

// Step 1 by every lane of a workgroup: the series for size parameter x and relative
// index m.  The two recurrences are serial and run at once on lanes of two
// different waves: D_n(mx) downward from n_start and psi_n(x), chi_n(x)
// upward (into s_psi, s_chi at index n, n = 0..N).  One downward step
//     D_{n-1} = n/(mx) - 1/(D_n + n/(mx))
// is the Moebius map of the matrix [[k, k^2 - 1], [1, k]], k = n/(mx), so it
// runs on D_n = P_n / Q_n as Q' = P + k Q, P' = k Q' - Q: eight FMAs and no
// division on the serial chain (one wave runs it, so its instruction count
// is its time).  One step grows or shrinks max(|P|, |Q|) by at most
// (1 + |k|)^2, with |k| < 2e9 for every size and index this library accepts
// (n_start <= ~1100 where |mx| < n_terms, |mx| >= 1e-6), so rescaling (P, Q)
// by a power of two every 8 steps keeps both far inside the FP64 range; the
// scale is exact and cancels in P / Q.  Its rounding matches that of the
// direct form (checked against a 50-digit evaluation of the recurrence).
// P_n and Q_n go to s_a and s_b (n = 1..N at index n - 1), and each lane
// forms D_n = P_n / Q_n for its n.  Then each lane forms a_n and b_n (in
// place of P_n and Q_n),
// and the sums of Q_ext (Eq. 13), Q_sca and the asymmetry (Eq. 12) are
// added per lane, per wave and over the waves in a fixed order.  On return
// (after a barrier) s_sums holds Q_ext, Q_sca and g for every lane.
__device__ __forceinline__ void mie_series_block(double x, double m_re, double m_im, int N, int n_start, cplx *s_a, cplx *s_b,
                                                 double2 *s_rec, double2 *s_fac, double *s_red, double *s_sums)
{
    const int tid = threadIdx.x;
    const cplx m = {m_re, m_im};
    const bool real = m_im == 0.0;
    if (tid < 64) {
        const cplx mx = x * m;
        const cplx inv_mx = cplx{1.0, 0.0} / mx;
        if (n_start >= kScanFrom) {
            if (real) downward_scan<true>(x, m, N, n_start, s_a, s_b);
            else downward_scan<false>(x, m, N, n_start, s_a, s_b);
        } else {
            if (real) downward<true>(inv_mx, N, n_start, s_fac, s_a, s_b);
            else downward<false>(inv_mx, N, n_start, s_fac, s_a, s_b);
        }
    } else if (tid < 128) {
        upward(x, N, (double *)(s_fac + kAhead + kChunk), s_rec);
    }
    __syncthreads();
    const cplx inv_m = cplx{1.0, 0.0} / m;
    for (int n = tid + 1; n <= N; n += blockDim.x) {
        const double psi_n = s_rec[n].x, psi = s_rec[n - 1].x;
        const cplx xi_n = {psi_n, -s_rec[n].y};
        const cplx xi_nm1 = {psi, -s_rec[n - 1].y};
        const cplx Pn = s_a[n - 1];
        const cplx Dn = real ? cplx{Pn.re / Pn.im, 0.0} : Pn / s_b[n - 1];
        const double nx = (double)n / x;
        const cplx da = Dn * inv_m + nx;
        const cplx db = m * Dn + nx;
        s_a[n - 1] = (psi_n * da - cplx{psi, 0.0}) / (da * xi_n - xi_nm1);
        s_b[n - 1] = (psi_n * db - cplx{psi, 0.0}) / (db * xi_n - xi_nm1);
    }
    __syncthreads();
    double sum_ext = 0.0, sum_sca = 0.0, sum_g = 0.0;
    for (int n = tid + 1; n <= N; n += blockDim.x) {
        const cplx an = s_a[n - 1], bn = s_b[n - 1];
        const double w = 2.0 * n + 1.0;
        sum_ext += w * (an.re + bn.re);
        sum_sca += w * (norm2(an) + norm2(bn));
        // asymmetry: (n-1)(n+1)/n Re(a_{n-1} a_n* + b_{n-1} b_n*) + (2n+1)/(n(n+1)) Re(a_n b_n*)
        if (n > 1) {
            const cplx ap = s_a[n - 2], bp = s_b[n - 2];
            const double c = (double)(n - 1) * (n + 1) / n;
            sum_g += c * (ap.re * an.re + ap.im * an.im + bp.re * bn.re + bp.im * bn.im);
        }
        sum_g += w / ((double)n * (n + 1)) * (an.re * bn.re + an.im * bn.im);
    }
    sum_ext = wave_sum(sum_ext);
    sum_sca = wave_sum(sum_sca);
    sum_g = wave_sum(sum_g);
    const int waves = blockDim.x >> 6;
    if ((tid & 63) == 0) {
        s_red[3 * (tid >> 6) + 0] = sum_ext;
        s_red[3 * (tid >> 6) + 1] = sum_sca;
        s_red[3 * (tid >> 6) + 2] = sum_g;
    }
    __syncthreads();
    if (tid == 0) {
        double e = 0.0, q = 0.0, g = 0.0;
        for (int w = 0; w < waves; ++w) {
            e += s_red[3 * w + 0];
            q += s_red[3 * w + 1];
            g += s_red[3 * w + 2];
        }
        const double inv_x2 = 1.0 / (x * x);
        const double q_sca = 2.0 * inv_x2 * q;
        s_sums[0] = 2.0 * inv_x2 * e;
        s_sums[1] = q_sca;
        s_sums[2] = 4.0 * inv_x2 * g / q_sca;
    }
    __syncthreads();
}

// Before step 2: fold the angular weight (2n + 1)/(n(n + 1)) of Eqs. 5-6 into
// a_n and b_n (in place) and tabulate the coefficients (2n - 1)/(n - 1) and
// n/(n - 1) of the pi_n recurrence, so the per-angle loop neither divides nor
// converts n.  Ends with a barrier.
__device__ void prepare_angular(int N, cplx *s_a, cplx *s_b, double2 *s_pi)
{
    for (int n = threadIdx.x + 1; n <= N; n += blockDim.x) {
        const double c = (2.0 * n + 1.0) / ((double)n * (n + 1));
        s_a[n - 1] = c * s_a[n - 1];
        s_b[n - 1] = c * s_b[n - 1];
        s_pi[n - 1] = n > 1 ? double2{(2.0 * n - 1.0) / (double)(n - 1), (double)n / (double)(n - 1)}
                            : double2{0.0, 0.0};
    }
    __syncthreads();
}

// Step 2 at an angle of cosine mu: S1 and S2 (Eqs. 5-6) with the angular functions
// upward, pi_n = ((2n - 1) mu pi_{n-1} - n pi_{n-2}) / (n - 1) from pi_0 = 0, pi_1
// = 1, and tau_n = n mu pi_n - (n + 1) pi_{n-1}, on the coefficients prepared
// above.  PART says what the lane adds up: kAll both sums, S[0..3] = Re S1, Im S1,
// Re S2, Im S2; kFirst or kSecond only the real part (im = 0) or imaginary part
// (1) of S1 or S2, S[0].  The loop runs a single wave on its SIMD and each sum
// takes two dependent fma a term, about 33 cycles each; the next terms'
// coefficients are read while four are worked on.
enum SumPart { kAll, kFirst, kSecond };
template <SumPart PART>
__device__ __forceinline__ void mie_sums(double mu, int N, const cplx *s_a, const cplx *s_b, const double2 *s_pi, int im,
                                         double *S)
{
    struct Term {
        double2 c;
        cplx a, b;
    };
    auto read = [&](int i) -> Term {
        if (PART == kAll) return {s_pi[i], s_a[i], s_b[i]};
        return {s_pi[i], {((const double *)(s_a + i))[im], 0.0}, {((const double *)(s_b + i))[im], 0.0}};
    };
    double pi_prev = 0.0, pi_n = 1.0;              // pi_0, pi_1
    {   // n = 1: tau_1 = mu
        const Term t = read(0);
        if (PART == kAll) {
            S[0] = fma(mu, t.b.re, t.a.re); S[1] = fma(mu, t.b.im, t.a.im);
            S[2] = fma(mu, t.a.re, t.b.re); S[3] = fma(mu, t.a.im, t.b.im);
        } else {
            S[0] = PART == kFirst ? fma(mu, t.b.re, t.a.re) : fma(mu, t.a.re, t.b.re);
        }
    }
    double dn = 2.0;
    auto add = [&](const Term &t) {
        const double p = fma(t.c.x * mu, pi_n, -t.c.y * pi_prev);
        pi_prev = pi_n;
        pi_n = p;
        const double dmu = dn * mu;
        dn += 1.0;
        const double tau_n = fma(dmu, pi_n, -dn * pi_prev);
        if (PART == kAll) {
            S[0] = fma(pi_n, t.a.re, fma(tau_n, t.b.re, S[0]));
            S[1] = fma(pi_n, t.a.im, fma(tau_n, t.b.im, S[1]));
            S[2] = fma(tau_n, t.a.re, fma(pi_n, t.b.re, S[2]));
            S[3] = fma(tau_n, t.a.im, fma(pi_n, t.b.im, S[3]));
        } else if (PART == kFirst) {
            S[0] = fma(pi_n, t.a.re, fma(tau_n, t.b.re, S[0]));
        } else {
            S[0] = fma(tau_n, t.a.re, fma(pi_n, t.b.re, S[0]));
        }
    };
    constexpr int G = 4;
    struct Four {
        Term t[G];
    };
    auto four = [&](int n) {   // (terms beyond N are read but not used)
        Four f;
#pragma unroll
        for (int u = 0; u < G; ++u) f.t[u] = read(min(n, MC_MAX_TERMS - G + 1) + u - 1);
        return f;
    };
    int n = 2;
    Four f = four(n);
    for (; n + 2 * G <= N + 1; n += 2 * G) {
        const Four g = four(n + G);
#pragma unroll
        for (int u = 0; u < G; ++u) add(f.t[u]);
        f = four(n + 2 * G);
#pragma unroll
        for (int u = 0; u < G; ++u) add(g.t[u]);
    }
    for (; n <= N; ++n) add(read(n - 1));
}

// |S1|^2 + |S2|^2 and its halves, rounded the same way wherever the sums come from.
__device__ __forceinline__ double square(double re, double im) { return fma(re, re, im * im); }
__device__ __forceinline__ double plus(double x, double y)
{
#pragma clang fp contract(off)
    return x + y;
}

// Step 2 at angle j of the na-point grid: scale x (|S1|^2 + |S2|^2) to
// phase_out[j] and, times sin(theta_j), to ang[j] (each if given).
__device__ __forceinline__ void put_phase(int j, double th, double P, double *phase_out, double *ang)
{
    if (phase_out) phase_out[j] = P;
    if (ang) ang[j] = P * sin_0_pi(th);
}

// One lane per angle.
__device__ __forceinline__ void phase_at(int j, int na, int N, double scale, const cplx *s_a, const cplx *s_b,
                                         const double2 *s_pi, double *phase_out, double *ang)
{
    const double th = (double)j * (M_PI / (double)(na - 1));
    double S[4];
    mie_sums<kAll>(cos_0_pi(th), N, s_a, s_b, s_pi, 0, S);
    put_phase(j, th, scale * plus(square(S[0], S[1]), square(S[2], S[3])), phase_out, ang);
}

// Four lanes per angle, one for each sum: waves 0 and 1 take S1, 2 and 3 S2, of the
// workgroup's kAngles angles; even lanes the real part, odd ones the imaginary.
// s_half holds kAngles doubles.
__device__ __forceinline__ void phase_split(int na, int N, double scale, const cplx *s_a, const cplx *s_b,
                                            const double2 *s_pi, double *s_half, double *phase_out, double *ang)
{
    const int tid = threadIdx.x, at = (tid & (kPhaseThreads / 2 - 1)) >> 1, j = blockIdx.x * kAngles + at;
    const double th = (double)j * (M_PI / (double)(na - 1));
    const bool first = tid < kPhaseThreads / 2;
    double S;
    if (first) mie_sums<kFirst>(cos_0_pi(th), N, s_a, s_b, s_pi, tid & 1, &S);
    else mie_sums<kSecond>(cos_0_pi(th), N, s_a, s_b, s_pi, tid & 1, &S);
    const int2 x = __builtin_bit_cast(int2, S);   // the neighbour's part (quad_perm 1032)
    const double im = __builtin_bit_cast(double, int2{__builtin_amdgcn_mov_dpp(x.x, 0xB1, 0xF, 0xF, true),
                                                      __builtin_amdgcn_mov_dpp(x.y, 0xB1, 0xF, 0xF, true)});
    const double half = square(S, im);
    if (!first && !(tid & 1)) s_half[at] = half;
    __syncthreads();
    if (first && !(tid & 1) && j < na) put_phase(j, th, scale * plus(half, s_half[at]), phase_out, ang);
}

__device__ __forceinline__ void put_result(double *to, double q_ext, double q_sca, double g, double n_terms)
{
    if (!to) return;
    to[0] = q_ext;
    to[1] = q_sca;
    to[2] = g;
    to[3] = n_terms;
}

// Steps 1-2 for one size: workgroup b runs the series, workgroup 0 writes the
// scalar results (and the coefficients if asked), and lane t evaluates angle
// j = 256 b + t into work[j] = P sin(theta_j) (and phase[j] = P if asked).
__global__ __launch_bounds__(kPhaseThreads) void mie_phase_kernel(MieArgs a)
{
    __shared__ cplx s_a[MC_MAX_TERMS];
    __shared__ cplx s_b[MC_MAX_TERMS];
    __shared__ double2 s_rec[MC_MAX_TERMS + 1];         // psi_n, chi_n
    __shared__ double2 s_fac[kAhead + kChunk + kChunk / 2];   // factors of the recurrences
    __shared__ double2 s_pi[MC_MAX_TERMS];              // pi_n recurrence coefficients
    __shared__ double s_red[3 * (kPhaseThreads / 64)];
    __shared__ double s_sums[3];                       // Q_ext, Q_sca, g
    __shared__ double s_half[kAngles];                 // |S2|^2

    const int tid = threadIdx.x;
    const int N = a.n_terms;
    const double x = a.x;
    mie_series_block(x, a.m_re, a.m_im, N, a.n_start, s_a, s_b, s_rec, s_fac, s_red, s_sums);
    if (blockIdx.x == 0) {
        if (tid == 0) {
            put_result(a.result, s_sums[0], s_sums[1], s_sums[2], (double)N);
            put_result(a.host_result, s_sums[0], s_sums[1], s_sums[2], (double)N);
        }
        if (a.coef) {
            for (int n = tid; n < N; n += kPhaseThreads) {
                a.coef[4 * n + 0] = s_a[n].re;
                a.coef[4 * n + 1] = s_a[n].im;
                a.coef[4 * n + 2] = s_b[n].re;
                a.coef[4 * n + 3] = s_b[n].im;
            }
        }
    }
    __syncthreads();
    prepare_angular(N, s_a, s_b, s_pi);
    // Phase function normalised as Eq. 10: P = 2 (|S1|^2 + |S2|^2) / (x^2 Q_sca).
    phase_split(a.n_angles, N, 2.0 / (x * x * s_sums[1]), s_a, s_b, s_pi, s_half, a.phase, a.work);
}

__device__ int first_at_least(const double *f, int l, int r, double u)
{
    while (l < r) {
        const int mid = (l + r) >> 1;
        if (f[mid] < u) l = mid + 1;
        else r = mid;
    }
    return l;
}

// Steps 3-4: ang holds P sin(theta) on the na-point grid.  Every workgroup
// reads it into LDS and forms the trapezoid CDF F_j in place (F = 1 at pi):
// each lane adds the increments of its run of at most three angles, a
// shuffle scan within each wave and a scan of the wave totals give every run
// the sum before it, and each run is then accumulated in order and divided
// by the total.  Workgroup 0 writes F to cdf_out (if given).  Then lane i of
// the grid takes inverse-table entry u_i = i / (nc - 1): the first angle with
// F >= u_i by binary search, theta interpolated linearly in F, and
// v = 1 - cos(theta) = 2 sin^2(theta/2) stored in FP32.
__global__ __launch_bounds__(kInvThreads) void mie_inverse_kernel(const double *ang, int na, int nc, float *inv_cdf,
                                                                  double *cdf_out)
{
    __shared__ double s_ang[MC_MAX_N_ANGLES];
    __shared__ double s_wave[kInvThreads / 64];
    __shared__ double s_total;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int j = tid; j < na; j += kInvThreads) s_ang[j] = ang[j];
    __syncthreads();

    const double dth = M_PI / (double)(na - 1);
    const int per = (na + kInvThreads - 1) / kInvThreads;
    const int lo = min(tid * per, na), hi = min(lo + per, na);
    const double f_left = lo >= 1 && lo < na ? s_ang[lo - 1] : 0.0;
    double local = 0.0;
    for (int j = max(lo, 1); j < hi; ++j) {
        const double th_j = (double)j * dth, th_p = (double)(j - 1) * dth;
        local += 0.5 * (th_j - th_p) * (s_ang[j - 1] + s_ang[j]);
    }
    double incl = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double v = __shfl_up(incl, off, 64);
        if (lane >= off) incl += v;
    }
    double excl = __shfl_up(incl, 1, 64);
    if (lane == 0) excl = 0.0;
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    if (tid == 0) {   // exclusive scan of the wave totals
        double run = 0.0;
        for (int w = 0; w < kInvThreads / 64; ++w) {
            const double v = s_wave[w];
            s_wave[w] = run;
            run += v;
        }
        s_total = run;
    }
    __syncthreads();
    double acc = s_wave[wave] + excl;
    const double total = s_total;
    double prev = f_left;
    for (int j = lo; j < hi; ++j) {
        const double f = s_ang[j];
        if (j >= 1) {
            const double th_j = (double)j * dth, th_p = (double)(j - 1) * dth;
            acc += 0.5 * (th_j - th_p) * (prev + f);
        }
        prev = f;
        s_ang[j] = (j == na - 1) ? 1.0 : acc / total;
    }
    __syncthreads();
    if (cdf_out && blockIdx.x == 0)
        for (int j = tid; j < na; j += kInvThreads) cdf_out[j] = s_ang[j];

    const int i = blockIdx.x * kInvThreads + tid;
    if (i >= nc) return;
    const double u = (double)i / (double)(nc - 1);
    // u <= 1 = F at pi, so only rounding could leave an entry past the grid.
    const int l = min(first_at_least(s_ang, 0, na, u), na - 1);
    double th = 0.0;
    if (l > 0) {
        const double th_j = (double)l * dth, th_p = (double)(l - 1) * dth;
        th = th_p + (u - s_ang[l - 1]) / (s_ang[l] - s_ang[l - 1]) * (th_j - th_p);
    }
    const double sh = sin_half_pi(0.5 * th);
    inv_cdf[i] = (float)(2.0 * sh * sh);
}

// ---- polydisperse: the bins, the mixture, then the same inverse ----------

struct PolyArgs {
    double x[MC_MAX_BINS];         // size parameter of each bin
    double c[MC_MAX_BINS];         // probability x geometric cross-section (mm^2) of each bin
    int n_terms[MC_MAX_BINS], n_start[MC_MAX_BINS];
    double m_re, m_im;
    int n_bins, n_angles, n_cdf;
    double geo_median;             // geometric cross-section of the median diameter (mm^2)
    double *rows;                  // n_bins x n_angles: c_k Q_sca,k P_k(theta_j)
    double *bins;                  // n_bins x 4: Q_ext,k, Q_sca,k, g_k, N_k
    double *ang;                   // n_angles: P(theta_j) sin(theta_j) of the mixture
    double *phase;
    double *result;                // q_ext, q_sca (over geo_median), g, max N
    double *host_result;           // the same again, pinned host memory (optional)
};

// Workgroup (s, k) runs bin k's series (workgroup (0, k) writes its scalars to
// bins) and its lanes evaluate row k at the 256 angles of slice s.
__global__ __launch_bounds__(kPhaseThreads) void mie_bin_kernel(PolyArgs a)
{
    __shared__ cplx s_a[MC_MAX_TERMS];
    __shared__ cplx s_b[MC_MAX_TERMS];
    __shared__ double2 s_rec[MC_MAX_TERMS + 1];         // psi_n, chi_n
    __shared__ double2 s_fac[kAhead + kChunk + kChunk / 2];   // factors of the recurrences
    __shared__ double2 s_pi[MC_MAX_TERMS];              // pi_n recurrence coefficients
    __shared__ double s_red[3 * (kPhaseThreads / 64)];
    __shared__ double s_sums[3];
    const int k = blockIdx.y, tid = threadIdx.x;
    const double x = a.x[k];
    const int N = a.n_terms[k];
    mie_series_block(x, a.m_re, a.m_im, N, a.n_start[k], s_a, s_b, s_rec, s_fac, s_red, s_sums);
    if (blockIdx.x == 0 && tid == 0) {
        a.bins[4 * k + 0] = s_sums[0];
        a.bins[4 * k + 1] = s_sums[1];
        a.bins[4 * k + 2] = s_sums[2];
        a.bins[4 * k + 3] = (double)N;
    }
    prepare_angular(N, s_a, s_b, s_pi);
    // c_k Q_sca,k P_k with P_k = 2 (|S1|^2 + |S2|^2) / (x^2 Q_sca,k): the Q_sca,k cancel.
    const int j = blockIdx.x * kPhaseThreads + tid;
    if (j < a.n_angles)
        phase_at(j, a.n_angles, N, a.c[k] * 2.0 / (x * x), s_a, s_b, s_pi, a.rows + (uint64_t)k * a.n_angles,
                 nullptr);
}

// Lane t of workgroup b mixes the rows at angle j = 256 b + t into ang[j]
// (and phase[j]); every workgroup sums the bins' cross-sections itself, in
// bin order, and workgroup 0 writes the scalar results.
__global__ __launch_bounds__(kPhaseThreads) void mie_mix_kernel(PolyArgs a)
{
    __shared__ double s_sca, s_bins[4 * MC_MAX_BINS], s_c[MC_MAX_BINS];
    const int tid = threadIdx.x;
    static_assert(4 * MC_MAX_BINS <= kPhaseThreads, "a lane per bin value");
    if (tid < 4 * a.n_bins) s_bins[tid] = a.bins[tid];
    if (tid < a.n_bins) s_c[tid] = a.c[tid];
    const int na = a.n_angles;
    const int j = blockIdx.x * kPhaseThreads + tid;
    const bool in = j < na;
    const double *row = a.rows + (in ? j : 0);
    // The rows added in bin order, their loads issued 32 at a time (8 at a time,
    // and bins read by the lane that adds them, took 10.4 us at 64 bins).
    constexpr int kRows = 32;
    double v[kRows];
    auto read = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kRows; ++u) v[u] = row[(uint64_t)min(k0 + u, a.n_bins - 1) * na];
    };
    read(0);
    __syncthreads();
    if (tid == 0) {
        // Number-averaged cross-sections and the C_sca-weighted asymmetry, in bin order.
        double ext = 0.0, sca = 0.0, gs = 0.0, nmax = 0.0;
#pragma unroll 8
        for (int k = 0; k < a.n_bins; ++k) {
            const double q_ext = s_bins[4 * k + 0], q_sca = s_bins[4 * k + 1];
            const double g = s_bins[4 * k + 2], n = s_bins[4 * k + 3];
            ext += s_c[k] * q_ext;
            sca += s_c[k] * q_sca;
            gs += s_c[k] * q_sca * g;
            nmax = fmax(nmax, n);
        }
        s_sca = sca;
        if (blockIdx.x == 0) {
            put_result(a.result, ext / a.geo_median, sca / a.geo_median, gs / sca, nmax);
            put_result(a.host_result, ext / a.geo_median, sca / a.geo_median, gs / sca, nmax);
        }
    }
    double mix = 0.0;
    for (int k0 = 0;;) {
#pragma unroll
        for (int u = 0; u < kRows; ++u)
            if (k0 + u < a.n_bins) mix += v[u];
        k0 += kRows;
        if (k0 >= a.n_bins) break;
        read(k0);
    }
    __syncthreads();
    if (!in) return;
    const double dth = M_PI / (double)(na - 1);
    const double P = mix * (1.0 / s_sca);
    if (a.phase) a.phase[j] = P;
    a.ang[j] = P * sin_0_pi((double)j * dth);
}

// Per-device scratch for the scalar results (8 doubles) and the angle grid
// (MC_MAX_N_ANGLES doubles) of synchronous builds whose caller passes none
// (allocated once per device, kept until the process ends).
constexpr size_t kScratchDoubles = 8 + MC_MAX_N_ANGLES;
std::mutex g_scratch_mu;
double *g_scratch[64] = {nullptr};

// Validate the spec and derive x, m and the series length (no device work).
int prepare_table(const mie_spec_t *spec, const mie_table_t *table, MieArgs *args, const char *who)
{
    if (!spec || !table) return fail(MC_EINVAL, "%s: null spec or table", who);
    const mie_spec_t s = *spec;
    if (!(s.n_medium > 0) || !(s.m_re > 0) || !(s.m_im >= 0) || !(s.diameter_um > 0) ||
        !(s.wavelength_nm > 0) || !std::isfinite(s.n_medium * s.m_re * s.m_im * s.diameter_um *
                                                   s.wavelength_nm))
        return fail(MC_EINVAL, "%s: indices, diameter and wavelength must be finite, positive (m_im >= 0)", who);
    if (s.n_angles < 3 || s.n_angles > MC_MAX_N_ANGLES)
        return fail(MC_EINVAL, "%s: n_angles %d outside 3..%d", who, s.n_angles, MC_MAX_N_ANGLES);
    if (s.n_cdf < 2 || s.n_cdf > MC_MAX_N_CDF)
        return fail(MC_EINVAL, "%s: n_cdf %d outside 2..%d", who, s.n_cdf, MC_MAX_N_CDF);
    if (!table->inv_cdf) return fail(MC_EINVAL, "%s: inv_cdf buffer is required", who);

    // Parameter processing (Sec. 3.1.1): x = pi d n_med / lambda0 (Eq. 3 with
    // the wavelength in the medium), m relative to the medium (Eq. 4).
    const double x = M_PI * s.diameter_um * 1e3 * s.n_medium / s.wavelength_nm;
    const double m_re = s.m_re / s.n_medium, m_im = s.m_im / s.n_medium;
    const double mx_abs = x * std::hypot(m_re, m_im);
    if (!(x >= 1e-6)) return fail(MC_EINVAL, "%s: size parameter %g below 1e-6", who, x);
    if (!(mx_abs >= 1e-6)) return fail(MC_EINVAL, "%s: |m| x = %g below 1e-6", who, mx_abs);
    const int n_terms = (int)std::lround(x + 4.0 * std::cbrt(x) + 2.0);   // Wiscombe 1980
    if (n_terms > MC_MAX_TERMS)
        return fail(MC_EINVAL, "%s: %d series terms exceed %d (x = %g)", who, n_terms, MC_MAX_TERMS, x);
    if (table->coef && table->coef_capacity < n_terms)
        return fail(MC_EINVAL, "%s: coef holds %d terms, %d needed", who, table->coef_capacity, n_terms);
    // Downward start: the start error decays slowly across the turning point
    // n ~ |mx|, whose width grows like |mx|^(1/3).
    const int n_start = (int)std::ceil(std::max((double)n_terms, mx_abs)) + 16 +
                        (int)std::ceil(8.0 * std::cbrt(mx_abs));

    *args = MieArgs{x, m_re, m_im, n_terms, n_start, s.n_angles, s.n_cdf,
                    table->inv_cdf, table->phase, table->cdf, table->coef, nullptr, nullptr, nullptr};
    return MC_OK;
}

// Launch the prepared table kernels on `st`: scalar results to `result`,
// the angle grid through `work` (both device).
int launch_table(MieArgs args, mie_table_t *table, hipStream_t st, double *result, double *work,
                 double *host_result = nullptr)
{
    args.result = result;
    args.host_result = host_result;
    args.work = work;
    const int g_phase = (args.n_angles + kAngles - 1) / kAngles;
    const int g_inv = (args.n_cdf + kInvThreads - 1) / kInvThreads;
    hipLaunchKernelGGL(mie_phase_kernel, dim3(g_phase), dim3(kPhaseThreads), 0, st, args);
    hipLaunchKernelGGL(mie_inverse_kernel, dim3(g_inv), dim3(kInvThreads), 0, st, (const double *)work, args.n_angles,
                       args.n_cdf, args.inv_cdf, args.cdf);
    MC_HIP_CHECK(hipGetLastError());
    table->x = args.x;
    table->m_rel_re = args.m_re;
    table->m_rel_im = args.m_im;
    table->n_terms = args.n_terms;
    table->n_cdf = args.n_cdf;
    return MC_OK;
}

void set_scalars(mie_table_t *table, const mie_spec_t &s, const double res[3])
{
    const double geo_mm2 = M_PI * (s.diameter_um * 1e-3) * (s.diameter_um * 1e-3) / 4.0;   // Eq. 14
    table->q_ext = res[0];
    table->q_sca = res[1];
    table->q_abs = res[0] - res[1];
    table->g = res[2];
    table->sigma_ext_mm2 = res[0] * geo_mm2;
    table->sigma_sca_mm2 = res[1] * geo_mm2;
    table->sigma_abs_mm2 = (res[0] - res[1]) * geo_mm2;
}

// The caller's result buffer and (if `work` is not null) angle-grid buffer,
// or for each one missing the library's per-device scratch (then `lock`
// holds the scratch until the results are back on the host).
int scratch_buffers(const mie_table_t *table, std::unique_lock<std::mutex> &lock, double **result, double **work,
                    const char *who)
{
    *result = table->result;
    if (work) *work = table->work;
    if (*result && (!work || *work)) return MC_OK;
    int dev = 0;
    MC_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(MC_EDEVICE, "device index %d out of range", dev);
    lock.lock();
    if (!g_scratch[dev]) {
        void *p = nullptr;
        if (hipMalloc(&p, kScratchDoubles * sizeof(double)) != hipSuccess)
            return fail(MC_ENOMEM, "%s: scratch allocation failed", who);
        g_scratch[dev] = (double *)p;
    }
    if (!*result) *result = g_scratch[dev];
    if (work && !*work) *work = g_scratch[dev] + 8;
    return MC_OK;
}

// Orthonormal Hermite polynomial h_n(t) for the weight exp(-t^2), by the
// three-term recurrence h_{j+1} = sqrt(2/(j+1)) t h_j - sqrt(j/(j+1)) h_{j-1}
// from h_0 = pi^(-1/4), together with sum_{j<n} h_j(t)^2.
struct HermiteCoef {
    double h0;                               // pi^(-1/4)
    double a[MC_MAX_BINS], b[MC_MAX_BINS];   // sqrt(2 / (j + 1)), sqrt(j / (j + 1))
};

// kLanes arguments at once, as independent chains that fill the vector units
// (one argument's chain of n steps leaves them idle).
constexpr int kLanes = 8;
struct Lanes {
    double v[kLanes];
};

template <bool SUM>
Lanes hermite_lanes(const HermiteCoef &c, int n, const Lanes &t, Lanes *sum_sq, Lanes *h_last)
{
    typedef double Pair __attribute__((vector_size(16)));
    constexpr int kPairs = kLanes / 2;
    Pair x[kPairs], h_prev[kPairs], h[kPairs], s[kPairs];
    for (int l = 0; l < kPairs; ++l) {
        x[l] = Pair{t.v[2 * l], t.v[2 * l + 1]};
        h_prev[l] = s[l] = Pair{0.0, 0.0};
        h[l] = Pair{c.h0, c.h0};
    }
    for (int j = 0; j < n; ++j) {
        const Pair a = {c.a[j], c.a[j]}, b = {c.b[j], c.b[j]};
#pragma unroll
        for (int l = 0; l < kPairs; ++l) {
            if (SUM) s[l] += h[l] * h[l];
            const Pair h_next = a * x[l] * h[l] - b * h_prev[l];
            h_prev[l] = h[l];
            h[l] = h_next;
        }
    }
    Lanes out;
    for (int l = 0; l < kLanes; ++l) {
        out.v[l] = h[l / 2][l & 1];
        if (SUM) sum_sq->v[l] = s[l / 2][l & 1];
        if (h_last) h_last->v[l] = h_prev[l / 2][l & 1];   // h_{n-1}
    }
    return out;
}
Lanes hermite_orthonormal(const HermiteCoef &c, int n, const Lanes &t, Lanes *sum_sq, Lanes *h_last = nullptr)
{
    return sum_sq ? hermite_lanes<true>(c, n, t, sum_sq, h_last) : hermite_lanes<false>(c, n, t, sum_sq, h_last);
}

// Gauss-Hermite rule for the weight exp(-t^2): the nodes are the n roots of
// h_n, all inside (-sqrt(2n+1), sqrt(2n+1)); each is bracketed by a sign
// change on a grid far finer than the root spacing and bisected to machine
// precision.  The weights are the Christoffel numbers 1 / sum_{j<n} h_j(t)^2.
//
// The grid's cells are found from every kStride-th point, then by halving, and
// kLanes roots are refined at a time: 64 nodes from the whole grid and one by one
// took 370 of the 430 us of mie_table_build_poly; this takes 28 of its 84.
int gauss_hermite(int n, double *t, double *w)
{
    if (n == 1) {
        t[0] = 0.0;
        w[0] = std::sqrt(M_PI);
        return MC_OK;
    }
    HermiteCoef c;
    c.h0 = std::pow(M_PI, -0.25);
    for (int j = 0; j < n; ++j) {
        c.a[j] = std::sqrt(2.0 / (j + 1));
        c.b[j] = std::sqrt((double)j / (j + 1));
    }
    // The grid step 2R / (40 n) is below a seventeenth of the smallest spacing
    // of neighbouring roots (about pi / sqrt(2n + 1)): no kStride cells hold two.
    constexpr int kStride = 8;
    const double R = std::sqrt(2.0 * n + 1.0) + 1.0;
    const int steps = 40 * n;
    auto grid = [&](int i) { return -R + 2.0 * R * (double)i / steps; };
    auto at_grid = [&](const int *i, double *h) {   // h_n at kLanes grid points
        Lanes x;
        for (int l = 0; l < kLanes; ++l) x.v[l] = i[l] == 0 ? -R : grid(i[l]);
        const Lanes v = hermite_orthonormal(c, n, x, nullptr);
        for (int l = 0; l < kLanes; ++l) h[l] = v.v[l];
    };
    // Strides (at[k] - kStride, at[k]] with a root: the sign of h_n changes over
    // them, or h_n is 0 at their end (it then has the other sign after it).
    static_assert(40 % kStride == 0, "whole strides");
    int at[MC_MAX_BINS + kLanes] = {0};
    bool neg[MC_MAX_BINS + kLanes] = {false};   // h_n < 0 before the root
    int found = 0;
    bool before = false;
    for (int i0 = 0; i0 <= steps && found < n; i0 += kLanes * kStride) {
        int i[kLanes];
        double h[kLanes];
        for (int l = 0; l < kLanes; ++l) i[l] = std::min(i0 + l * kStride, steps);
        at_grid(i, h);
        for (int l = 0; l < kLanes && i0 + l * kStride <= steps && found < n; ++l) {
            if (i[l] == 0) {
                before = h[l] < 0.0;
                continue;
            }
            if ((h[l] < 0.0) != before || h[l] == 0.0) {
                at[found] = i[l];
                neg[found] = before;
                ++found;
                before = !before;
            }
        }
    }
    if (found != n) return fail(MC_EINVAL, "Gauss-Hermite: found %d of %d nodes", found, n);
    for (int r0 = 0; r0 < n; r0 += kLanes) {
        // The stride's first point at or past the root, by halving.  (Selects, not
        // branches: which half holds a root cannot be predicted.)
        int lo_i[kLanes], up_i[kLanes];
        bool minus[kLanes];
        double h[kLanes], h_up[kLanes];
        for (int l = 0; l < kLanes; ++l) {
            const int r = std::min(r0 + l, n - 1);
            lo_i[l] = at[r] - kStride;
            up_i[l] = at[r];
            minus[l] = neg[r];
        }
        at_grid(up_i, h_up);
        for (int width = kStride; width > 1; width /= 2) {
            int mid[kLanes];
            for (int l = 0; l < kLanes; ++l) mid[l] = (lo_i[l] + up_i[l]) / 2;
            at_grid(mid, h);
            for (int l = 0; l < kLanes; ++l) {
                const bool past = ((h[l] < 0.0) != minus[l]) | (h[l] == 0.0);
                up_i[l] = past ? mid[l] : up_i[l];
                h_up[l] = past ? h[l] : h_up[l];
                lo_i[l] = past ? lo_i[l] : mid[l];
            }
        }
        // The cell, by halving to neighbouring doubles (a root on the grid is one).
        // Newton's steps (h_n' = sqrt(2n) h_{n-1}; from a cell's middle the error
        // falls as 3e-4, 8e-7, 7e-12, rounding) say where the root is, so that
        // h_n itself is needed only within 1e-12 of it: beyond, |h_n| is a hundred
        // times what its recurrence rounds and has the sign of its side.
        Lanes lo, up, mid, near;
        for (int l = 0; l < kLanes; ++l) {
            lo.v[l] = h_up[l] == 0.0 ? grid(up_i[l]) : (lo_i[l] == 0 ? -R : grid(lo_i[l]));
            up.v[l] = grid(up_i[l]);
            near.v[l] = 0.5 * (lo.v[l] + up.v[l]);
        }
        const double slope = std::sqrt(2.0 * n);
        for (int it = 0; it < 4; ++it) {
            Lanes last;
            const Lanes hn = hermite_orthonormal(c, n, near, nullptr, &last);
            for (int l = 0; l < kLanes; ++l) near.v[l] -= hn.v[l] / (slope * last.v[l]);
        }
        // (A step that left the cell would be no guide: every sign is then taken
        // from h_n.)
        double margin[kLanes];
        for (int l = 0; l < kLanes; ++l)
            margin[l] = near.v[l] > lo.v[l] && near.v[l] < up.v[l] ? 1e-12 * std::max(1.0, std::fabs(near.v[l])) : INFINITY;
        for (int it = 0; it < 200; ++it) {
            int open = 0, ask = 0;
            bool inside[kLanes];
            for (int l = 0; l < kLanes; ++l) {
                mid.v[l] = 0.5 * (lo.v[l] + up.v[l]);
                inside[l] = (mid.v[l] > lo.v[l]) & (mid.v[l] < up.v[l]);
                open |= inside[l];
                ask |= inside[l] & !(std::fabs(mid.v[l] - near.v[l]) > margin[l]);
            }
            if (!open) break;
            Lanes hm{};
            if (ask) hm = hermite_orthonormal(c, n, mid, nullptr);
            for (int l = 0; l < kLanes; ++l) {
                const bool below = ask ? (hm.v[l] < 0.0) == minus[l] : mid.v[l] < near.v[l];
                lo.v[l] = (inside[l] & below) ? mid.v[l] : lo.v[l];
                up.v[l] = (inside[l] & !below) ? mid.v[l] : up.v[l];
            }
        }
        Lanes root, sum;
        for (int l = 0; l < kLanes; ++l) root.v[l] = h_up[l] == 0.0 ? up.v[l] : 0.5 * (lo.v[l] + up.v[l]);
        (void)hermite_orthonormal(c, n, root, &sum);
        for (int l = 0; l < kLanes && r0 + l < n; ++l) {
            t[r0 + l] = root.v[l];
            w[r0 + l] = 1.0 / sum.v[l];
        }
    }
    return MC_OK;
}

int lognormal_bins(double median_um, double sigma_ln, int n, double *d, double *p)
{
    if (!(median_um > 0.0) || !std::isfinite(median_um) || !(sigma_ln >= 0.0) || !std::isfinite(sigma_ln))
        return fail(MC_EINVAL, "lognormal bins: median must be > 0 and sigma_ln >= 0, both finite");
    if (n < 1 || n > MC_MAX_BINS) return fail(MC_EINVAL, "lognormal bins: n_bins %d outside 1..%d", n, MC_MAX_BINS);
    double t[MC_MAX_BINS], w[MC_MAX_BINS];
    if (int rc = gauss_hermite(n, t, w)) return rc;
    for (int k = 0; k < n; ++k) {
        d[k] = median_um * std::exp(std::sqrt(2.0) * sigma_ln * t[k]);
        p[k] = w[k] / std::sqrt(M_PI);
    }
    return MC_OK;
}

uint64_t poly_work_words(int n_angles, int n_bins) { return (uint64_t)n_bins * n_angles + 4ull * n_bins + n_angles; }

}  // namespace
}  // namespace mcmie

extern "C" int mc_lognormal_bins(double median_um, double sigma_ln, int32_t n_bins, double *diameters_um,
                                 double *probs)
{
    using namespace mcmie;
    clear_error();
    if (!diameters_um || !probs) return fail(MC_EINVAL, "mc_lognormal_bins: null output");
    return lognormal_bins(median_um, sigma_ln, n_bins, diameters_um, probs);
}

extern "C" uint64_t mie_poly_work_bytes(const mie_spec_t *spec, const mie_poly_t *poly)
{
    if (!spec || !poly || spec->n_angles < 3 || spec->n_angles > MC_MAX_N_ANGLES || poly->n_bins < 1 ||
        poly->n_bins > MC_MAX_BINS)
        return 0;
    return mcmie::poly_work_words(spec->n_angles, poly->n_bins) * 8;
}

extern "C" int mie_table_build_poly(const mie_spec_t *spec, const mie_poly_t *poly, mie_table_t *table, void *stream)
{
    using namespace mcmie;
    clear_error();
    const char *who = "mie_table_build_poly";
    MieArgs med;
    if (int rc = prepare_table(spec, table, &med, who)) return rc;
    if (!poly) return fail(MC_EINVAL, "%s: null poly", who);
    const mie_spec_t s = *spec;
    const mie_poly_t q = *poly;
    if (table->coef) return fail(MC_EINVAL, "%s: coef is not produced for a size distribution (set it to NULL)", who);
    if (!q.work || ((uintptr_t)q.work & 7) || q.work_bytes < poly_work_words(s.n_angles, q.n_bins) * 8)
        return fail(MC_EINVAL, "%s: work needs %llu bytes, 8-byte aligned", who,
                    (unsigned long long)(poly_work_words(s.n_angles, std::max(1, q.n_bins)) * 8));
    double d[MC_MAX_BINS], p[MC_MAX_BINS];
    if (int rc = lognormal_bins(s.diameter_um, q.sigma_ln, q.n_bins, d, p)) return rc;
    PolyArgs a{};
    a.m_re = med.m_re;
    a.m_im = med.m_im;
    a.n_bins = q.n_bins;
    a.n_angles = s.n_angles;
    a.n_cdf = s.n_cdf;
    for (int k = 0; k < q.n_bins; ++k) {
        // Each bin's parameters as prepare_table derives them for one size.
        const double x = M_PI * d[k] * 1e3 * s.n_medium / s.wavelength_nm;
        const double mx_abs = x * std::hypot(med.m_re, med.m_im);
        const int n_terms = (int)std::lround(x + 4.0 * std::cbrt(x) + 2.0);
        if (n_terms > MC_MAX_TERMS)
            return fail(MC_EINVAL, "%s: bin %d needs %d series terms, more than %d", who, k, n_terms, MC_MAX_TERMS);
        a.x[k] = x;
        a.n_terms[k] = n_terms;
        a.n_start[k] = (int)std::ceil(std::max((double)n_terms, mx_abs)) + 16 + (int)std::ceil(8.0 * std::cbrt(mx_abs));
        a.c[k] = p[k] * M_PI * (d[k] * 1e-3) * (d[k] * 1e-3) / 4.0;
    }
    a.geo_median = M_PI * (s.diameter_um * 1e-3) * (s.diameter_um * 1e-3) / 4.0;
    a.rows = q.work;
    a.bins = q.work + (uint64_t)q.n_bins * s.n_angles;
    a.ang = a.bins + 4ull * q.n_bins;
    a.phase = table->phase;
    std::unique_lock<std::mutex> lock(g_scratch_mu, std::defer_lock);
    if (int rc = scratch_buffers(table, lock, &a.result, nullptr, who)) return rc;
    HostResult host;
    a.host_result = host ? host.data() : nullptr;
    hipStream_t st = (hipStream_t)stream;
    const int slices = (s.n_angles + kPhaseThreads - 1) / kPhaseThreads;
    hipLaunchKernelGGL(mie_bin_kernel, dim3(slices, q.n_bins), dim3(kPhaseThreads), 0, st, a);
    hipLaunchKernelGGL(mie_mix_kernel, dim3(slices), dim3(kPhaseThreads), 0, st, a);
    hipLaunchKernelGGL(mie_inverse_kernel, dim3((s.n_cdf + kInvThreads - 1) / kInvThreads), dim3(kInvThreads), 0, st,
                       (const double *)a.ang, s.n_angles, s.n_cdf, table->inv_cdf, table->cdf);
    MC_HIP_CHECK(hipGetLastError());
    double res[4];
    MC_HIP_CHECK(wait_result(res, 4, a.result, host, st));
    table->x = med.x;
    table->m_rel_re = med.m_re;
    table->m_rel_im = med.m_im;
    table->n_terms = (int)res[3];
    table->n_cdf = s.n_cdf;
    set_scalars(table, s, res);
    return MC_OK;
}

extern "C" int mie_table_build(const mie_spec_t *spec, mie_table_t *table, void *stream)
{
    using namespace mcmie;
    clear_error();
    hipStream_t st = (hipStream_t)stream;
    MieArgs args;
    if (int rc = prepare_table(spec, table, &args, "mie_table_build")) return rc;
    double *result = nullptr, *work = nullptr;
    std::unique_lock<std::mutex> lock(g_scratch_mu, std::defer_lock);
    if (int rc = scratch_buffers(table, lock, &result, &work, "mie_table_build")) return rc;
    HostResult host;
    if (int rc = launch_table(args, table, st, result, work, host ? host.data() : nullptr)) return rc;
    double res[4];
    MC_HIP_CHECK(wait_result(res, 4, result, host, st));
    set_scalars(table, *spec, res);
    return MC_OK;
}

extern "C" int mie_table_enqueue(const mie_spec_t *spec, mie_table_t *table, void *stream)
{
    using namespace mcmie;
    clear_error();
    MieArgs args;
    if (int rc = prepare_table(spec, table, &args, "mie_table_enqueue")) return rc;
    if (!table->result) return fail(MC_EINVAL, "mie_table_enqueue: result buffer is required");
    if (!table->work) return fail(MC_EINVAL, "mie_table_enqueue: work buffer (n_angles doubles) is required");
    if (int rc = launch_table(args, table, (hipStream_t)stream, table->result, table->work)) return rc;
    const double nan3[3] = {NAN, NAN, NAN};
    set_scalars(table, *spec, nan3);
    return MC_OK;
}
