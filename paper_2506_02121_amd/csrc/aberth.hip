// Critical-curve root finder: parallel Aberth-Ehrlich sweeps (Sec. 3.2)
// over the phase grid, warm-started along phi and grown centre-out in
// subchains (Sec. 4.3), in plain FP64 or in a mixed-precision form.
//
// Layout and scheduling (gfx950):
//  * One lane per root; a wave takes a block of 64 consecutive roots of one
//    "front" (a growing end of a subchain).  Star positions and the other
//    roots stream through LDS in tiles of the wave's own and are read back as
//    wave-uniform broadcasts.  Work groups have one wave in the round schedule
//    and the expansion kernel, and up to eight in the persistent launch.
//  * A block with only a few unconverged roots left (the last sweep of a row)
//    works on them one at a time with the whole wave.
//  * Jacobi double buffering: every pass reads one iterate and writes the
//    other; a round alternates them for all fronts, the persistent launch for
//    each front by itself.
//  * Each front carries a phase.  FP64 mode: every row is FP64 Aberth sweeps.
//    Mixed mode: cold starts are FP32 Aberth sweeps until the roots settle;
//    warm rows with a chain prediction start directly with FP64 Newton
//    polish passes (the paper's cutoffs on each Newton step, row identities
//    for the row), warm rows without one with a single FP32 sweep; a row the
//    polish does not settle gets one FP32 sweep of the whole row and the
//    polish again, then FP64 Aberth sweeps.
//  * A warm row's first pass may start each root from an extrapolation
//    along its chain instead of its previous-row value.
//  * Warm rows with a chain prediction, in either form, are solved from the
//    star field's Taylor expansion about a point of each root's chain by a
//    kernel of their own, in which every block of 64 roots goes through the
//    rows of its front by itself (expand_rows); passes take the cold starts,
//    the rows next to them and the roots an expansion leaves open.
//    expand_check then tests the rows they finished, whose roots nothing kept
//    apart, by their row identities, and expand_control moves the fronts on.
//    Coarse phase grids take no expansions.
//  * A control kernel after every round advances the fronts (device-side; the
//    host polls a status block one batch ahead); in the persistent launch the
//    work group that finishes a front's pass does.
//  * Converged roots are mapped to the caustic in the same kernel.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "mlcc_internal.h"
#include "term_groups.h"

namespace mlcc {

// The hardware estimate v_rcp_f64 has relative error ~2^-24.4; one
// refinement step takes it below 2^-47, a few units in the last place of a
// double.  Star terms and root-root terms both take that step, so every sum
// of an FP64 Aberth sweep is formed at double precision (the paper's program
// is double precision throughout, Sec. 4.4).
constexpr int RCP_STAR = 1;
constexpr int RCP_ROOT = 1;

// Streams the records p[0..n) through body(i, rec) for one wave.  Tiles of 64 records (one per lane) are fetched with coalesced
// vector loads, the next tile while the current one is consumed, converted
// by cvt and parked in LDS, and read back with one wave-uniform (broadcast)
// LDS read per record; tile_end() runs after each tile.  Vector loads retire
// in order, so waiting for the older tile never waits for the prefetch
// behind it.  Indices past n-1 are clamped on load, so nothing outside the
// array is read.  `lds` holds two tiles of the wave's own.
template <class Src, class L, class Cvt, class Body, class End>
__device__ __forceinline__ void stream_tiles_ex(const Src p, int n, L *lds, Cvt &&cvt,
                                                Body &&body, End &&tile_end)
{
    if (n <= 0) return;
    const int lane = threadIdx.x & 63;
    const int ntiles = (n + 63) >> 6;
    auto reg = p[min(lane, n - 1)];
    for (int t = 0; t < ntiles; ++t) {
        L *buf = lds + ((t & 1) << 6);
        buf[lane] = cvt(reg);
        wave_sync();
        if (t + 1 < ntiles) reg = p[min(((t + 1) << 6) + lane, n - 1)];
        const int base = t << 6;
        const int cnt = min(64, n - base);
        if (cnt == 64) {
#pragma unroll 8
            for (int k = 0; k < 64; ++k) body(base + k, buf[k]);
        } else {
            for (int k = 0; k < cnt; ++k) body(base + k, buf[k]);
        }
        tile_end();
    }
    wave_sync();
}

// Calls body(i, p[i]) for i = lane, lane + 64, ... < n, four loads in flight:
// the few roots of a straggler block, often a wave alone on its SIMD, would else
// wait out the latency of every record.  (Left to `#pragma unroll 4` the compiler
// put each load behind the record before it, in some of the kernels.)  2,500
// stars, whose last block of 8 roots is such a block in every sweep: a sweep of
// the round schedule 209 -> 137 us with multipole sums, 234 -> 197 without;
// whole calls N = 1,000 6.2 -> 5.7 ms, N = 3,000 with multipole sums 12.0 -> 10.8.
template <class T, class Body>
__device__ __forceinline__ void each_strided(const T *__restrict__ p, int n, int lane, Body &&body)
{
    int i = lane;
    for (int t = n >> 8; t; --t, i += 256) {
        const T r[4] = {p[i], p[i + 64], p[i + 128], p[i + 192]};
#pragma unroll
        for (int j = 0; j < 4; ++j) body(i + 64 * j, r[j]);
    }
    for (; i < n; i += 64) body(i, p[i]);
}

struct Same {
    template <class T> __device__ __forceinline__ T operator()(const T &v) const { return v; }
};
struct NoEnd {
    __device__ __forceinline__ void operator()() const {}
};

template <class Src, class T, class Body>
__device__ __forceinline__ void stream_tiles(const Src p, int n, T *lds, Body &&body)
{
    stream_tiles_ex(p, n, lds, Same{}, body, NoEnd{});
}

// Star records: (x, y) when all masses are equal (the common mass is applied
// once at the end), (x, y, m, 0) otherwise.
template <bool EQUAL> struct StarRec;
template <> struct StarRec<true> {
    using T = double2;
    static __device__ __forceinline__ double mass(const double2 &) { return 1.0; }
};
template <> struct StarRec<false> {
    using T = double4;
    static __device__ __forceinline__ double mass(const double4 &s) { return s.z; }
};

__device__ __forceinline__ void wave_sum(double &v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
}

// Agent-scope atomic loads: what another work group published reaches this
// one through them whichever XCD (and L2) each runs on.
__device__ __forceinline__ unsigned long long load_acquire(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t load_acquire(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_relaxed(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t load_relaxed(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// FP64 Aberth sweep
// ---------------------------------------------------------------------------

// Running sums for one root z, u_i = 1/(z - z_i):
//   s1 = sum u_i                (for P'/P = F'/F + 2 s1)
//   s0 = sum m_i u_i            (lens mapping; equals m0 s1 for equal masses)
//   s2 = sum m_i u_i^2          (F = gamma + s2 - (1 - kappa_s) e^{-i phi});
//                               while accumulating, s2i holds sum m_i ux uy
//                               and finish() turns it into Im s2 = -2 that
//   s3 = sum m_i u_i^3          (F' = -2 s3)
//   R  = sum_{r != k} 1/(z - z_r)
// For equal masses the m_i factors are left out and applied once at the end.
struct Sums {
    double s1r, s1i, s0r, s0i, s2r, s2i, s3r, s3i, Rr, Ri;
};

__device__ __forceinline__ void zero(Sums &S)
{
    S.s1r = S.s1i = S.s0r = S.s0i = S.s2r = S.s2i = S.s3r = S.s3i = S.Rr = S.Ri = 0.0;
}

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star_inv(Sums &S, double dx, double dy, double inv,
                                             const T &s);

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star(Sums &S, double zr, double zi, const T &s)
{
    const double dx = zr - s.x;
    const double dy = zi - s.y;
    add_star_inv<EQUAL>(S, dx, dy, rcp_refined<RCP_STAR>(fma(dx, dx, dy * dy)), s);
}

// G consecutive star terms sharing one refined reciprocal (rcp_group), in
// the order add_star would take them.
template <bool EQUAL, int G, class T>
__device__ __forceinline__ void add_star_group(Sums &S, double zr, double zi, const T *r)
{
    double dx[G], dy[G], q[G], iq[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        dx[j] = zr - r[j].x;
        dy[j] = zi - r[j].y;
        q[j] = fma(dx[j], dx[j], dy[j] * dy[j]);
    }
    rcp_group<G, RCP_STAR>(q, iq);
#pragma unroll
    for (int j = 0; j < G; ++j) add_star_inv<EQUAL>(S, dx[j], dy[j], iq[j], r[j]);
}

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star_inv(Sums &S, double dx, double dy, double inv,
                                             const T &s)
{
    // u = conj(d) / |d|^2 = ux - i uy, with a = ux^2, b = uy^2:
    //   u^2 = (a - b) - 2 i ux uy,   u^3 = ux (a - 3b) + i uy (b - 3a).
    // Since a + b = |u|^2 = inv, only b is squared: t = a - b = inv - 2b,
    // a - 3b = t - 2b and b - 3a = 4b - 3 inv = -2t - inv.  Every
    // coefficient is an inline constant of the three-operand FP64 FMA and the
    // negated inv a source modifier, so u^2 and u^3 take one product and four
    // FMAs instead of two products and four FMAs.
    const double ux = dx * inv;
    const double uy = dy * inv;
    const double b = uy * uy;
    const double t = fma(-2.0, b, inv);
    const double c3r = fma(-2.0, b, t), c3i = fma(-2.0, t, -inv);
    S.s1r += ux;
    S.s1i -= uy;
    if (EQUAL) {
        S.s2r += t;
        S.s2i = fma(ux, uy, S.s2i);
        S.s3r = fma(ux, c3r, S.s3r);
        S.s3i = fma(uy, c3i, S.s3i);
    } else {
        const double mi = StarRec<EQUAL>::mass(s);
        const double mux = mi * ux, muy = mi * uy;
        S.s0r += mux;
        S.s0i -= muy;
        S.s2r = fma(mi, t, S.s2r);
        S.s2i = fma(mux, uy, S.s2i);
        S.s3r = fma(mux, c3r, S.s3r);
        S.s3i = fma(muy, c3i, S.s3i);
    }
}

// Root-root term of the Aberth correction, 1/(z - z_r) = conj(d) / |d|^2.
__device__ __forceinline__ void add_root(Sums &S, double zr, double zi, const double2 &o)
{
    const double dx = zr - o.x, dy = zi - o.y;
    const double inv = rcp_refined<RCP_ROOT>(fma(dx, dx, dy * dy));
    S.Rr = fma(dx, inv, S.Rr);
    S.Ri = fma(-dy, inv, S.Ri);
}

// G root-root terms sharing one refined reciprocal (rcp_group), in the order
// add_root would take them.  Two iterates at one point make every term of the
// group non-finite, as one term alone would be, and the iterate is nudged.
template <int G>
__device__ __forceinline__ void add_root_group(Sums &S, double zr, double zi, const double2 *r)
{
    double dx[G], dy[G], q[G], iq[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        dx[j] = zr - r[j].x;
        dy[j] = zi - r[j].y;
        q[j] = fma(dx[j], dx[j], dy[j] * dy[j]);
    }
    rcp_group<G, RCP_STAR>(q, iq);
#pragma unroll
    for (int j = 0; j < G; ++j) {
        S.Rr = fma(dx[j], iq[j], S.Rr);
        S.Ri = fma(-dy[j], iq[j], S.Ri);
    }
}

// The root-root term with FP32 arithmetic (MLCC_FP64_R32, warm rows).  Each
// coordinate enters as an FP32 pair hi + lo (hi = the FP64 value rounded to
// FP32, lo = the rounded remainder), and the difference is formed as
// (hi_k - hi_r) + (lo_k - lo_r): the first difference is exact for nearby
// roots, so the distance carries FP32 relative accuracy (~2^-24) at any
// separation, as does the FP32 reciprocal; the term runs at the FP32 issue
// rate.
struct SplitRoot {
    __device__ __forceinline__ float4 operator()(const double2 &o) const
    {
        const float hx = (float)o.x, hy = (float)o.y;
        return make_float4(hx, hy, (float)(o.x - (double)hx), (float)(o.y - (double)hy));
    }
};

__device__ __forceinline__ void add_root_hl(float &Rr, float &Ri, const float4 &z,
                                            const float4 &o)
{
    const float dx = (z.x - o.x) + (z.z - o.z);
    const float dy = (z.y - o.y) + (z.w - o.w);
    const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, dy * dy));
    Rr = fmaf(dx, inv, Rr);
    Ri = fmaf(-dy, inv, Ri);
}

struct Update {
    double zr, zi;   // new iterate
    double wr, wi;   // its image under the lens map
    bool flag;       // converged
    double err;      // Newton polish: estimated error of the new iterate
};

// Degenerate iterate (on a star, or two iterates equal): nudge it off.
__device__ __forceinline__ void nudge(Update &u, double zr, double zi, int k)
{
    u.zr = zr + 1e-7 * (1 + (k & 7));
    u.zi = zi + 1e-7 * (1 + (k >> 3 & 7));
    u.flag = false;
}

// One Aberth-Ehrlich update from the sums at z (Sec. 3.2), the convergence
// test of the Sec. 3.2 footnote with the App. C bound on |1/mu|, and the
// lens map at the new iterate.  The map reuses the sums: with
// z' = z - D, sum m_i/(z' - z_i) = s0 + D s2 + D^2 s3 + O(D^3 sum m_i u_i^4),
// and D is below the convergence cutoffs once a root is flagged.
// Rectangular field (Sec. 4.2, App. B): the sheet adds -P(z) to F and
// -P'(z) to F', with P(z) = sum_{k=1..n} d_2k z^2k (real d_2k, see
// sheet_poly): P = w h(w), P' = 2 z g(w), w = z^2, h = sum d_2k w^(k-1),
// g = sum k d_2k w^(k-1), both by Horner's rule.
__device__ __forceinline__ void sheet_terms(const double *__restrict__ d, int n, double zr,
                                            double zi, double &Pr, double &Pi, double &Qr,
                                            double &Qi)
{
    const double wr = zr * zr - zi * zi, wi = 2.0 * zr * zi;
    double hr = d[n - 1], hi = 0.0, gr = n * d[n - 1], gi = 0.0;
    for (int k = n - 2; k >= 0; --k) {
        const double th = hr * wr - hi * wi + d[k];
        hi = hr * wi + hi * wr;
        hr = th;
        const double tg = gr * wr - gi * wi + (k + 1) * d[k];
        gi = gr * wi + gi * wr;
        gr = tg;
    }
    Pr = hr * wr - hi * wi;
    Pi = hr * wi + hi * wr;
    Qr = 2.0 * (gr * zr - gi * zi);
    Qi = 2.0 * (gr * zi + gi * zr);
}

// Its term of the lens map: sum_k d_2k / (2k + 1) z^(2k+1) = z^3 H(z^2) with
// H = sum (d_2k / (2k + 1)) w^(k-1); the map subtracts its conjugate.
__device__ __forceinline__ void sheet_map_term(const double *__restrict__ dm, int n, double zr,
                                               double zi, double &Qr, double &Qi)
{
    const double wr = zr * zr - zi * zi, wi = 2.0 * zr * zi;
    double hr = dm[n - 1], hi = 0.0;
    for (int k = n - 2; k >= 0; --k) {
        const double th = hr * wr - hi * wi + dm[k];
        hi = hr * wi + hi * wr;
        hr = th;
    }
    const double qr = hr * wr - hi * wi, qi = hr * wi + hi * wr;   // z^2 H
    Qr = qr * zr - qi * zi;
    Qi = qr * zi + qi * zr;
}

// F and F' at an iterate.
struct FieldAt {
    double Fr, Fi, Fpr, Fpi;
};

// F and F' from the sums at z, which are completed in place: the common mass
// and the sign of Im s2.
template <bool EQUAL>
__device__ __forceinline__ FieldAt field_at(Sums &S, double zr, double zi, double m0, double2 e,
                                            double gamma, const double *sheet, int n_poly)
{
    S.s2i *= -2.0;
    if (EQUAL) {   // every mass equals m0: the sums above left it out
        S.s0r = m0 * S.s1r;
        S.s0i = m0 * S.s1i;
        S.s2r *= m0;
        S.s2i *= m0;
        S.s3r *= m0;
        S.s3i *= m0;
    }
    // F = gamma + S2 - (1 - kappa_s) e^{-i phi}, F' = -2 S3
    FieldAt Q;
    Q.Fr = gamma + S.s2r - e.x;
    Q.Fi = S.s2i - e.y;
    Q.Fpr = -2.0 * S.s3r;
    Q.Fpi = -2.0 * S.s3i;
    if (n_poly > 0) {   // rectangular field: F -= P(z), F' -= P'(z)
        double Pr, Pi, Qr, Qi;
        sheet_terms(sheet, n_poly, zr, zi, Pr, Pi, Qr, Qi);
        Q.Fr -= Pr;
        Q.Fi -= Pi;
        Q.Fpr -= Qr;
        Q.Fpi -= Qi;
    }
    return Q;
}

// The step F / (F' + F G), G = 2 S1 - R (the Aberth step
// 1 / (F'/F + 2 S1 - R)), its tests and the lens map, from completed sums.
__device__ __forceinline__ Update take_step(const Sums &S, const FieldAt &Q, double Gr, double Gi,
                                            double zr, double zi, double gamma, double a,
                                            double a1, double tol_step2, double tol_mu, int k,
                                            const double *sheet, int n_poly)
{
    const double Fr = Q.Fr, Fi = Q.Fi;
    const double Dr = Q.Fpr + (Fr * Gr - Fi * Gi);
    const double Di = Q.Fpi + (Fr * Gi + Fi * Gr);
    const double den = Dr * Dr + Di * Di;
    const double stepr = (Fr * Dr + Fi * Di) / den;
    const double stepi = (Fi * Dr - Fr * Di) / den;
    Update u;
    u.zr = zr - stepr;
    u.zi = zi - stepi;
    const double aF = sqrt(Fr * Fr + Fi * Fi);
    u.flag = (stepr * stepr + stepi * stepi < tol_step2) || (aF * (aF + 2.0 * a1) < tol_mu);
    if (!isfinite(u.zr) || !isfinite(u.zi)) nudge(u, zr, zi, k);
    // T = s0 + D s2 + D^2 s3 with D = step
    const double d2r = stepr * stepr - stepi * stepi, d2i = 2.0 * stepr * stepi;
    const double Tr = S.s0r + (stepr * S.s2r - stepi * S.s2i) + (d2r * S.s3r - d2i * S.s3i);
    const double Ti = S.s0i + (stepr * S.s2i + stepi * S.s2r) + (d2r * S.s3i + d2i * S.s3r);
    // w = (1 - kappa_s) z' + gamma conj(z') - conj(T)
    u.wr = fma(a, u.zr, gamma * u.zr) - Tr;
    u.wi = fma(a, u.zi, -gamma * u.zi) + Ti;
    if (n_poly > 0) {   // rectangular field: - conj(sum_k d_2k / (2k + 1) z'^(2k+1))
        double Qr, Qi;
        sheet_map_term(sheet + n_poly, n_poly, u.zr, u.zi, Qr, Qi);
        u.wr -= Qr;
        u.wi += Qi;
    }
    return u;
}

template <bool EQUAL>
__device__ __forceinline__ Update finish(Sums S, double zr, double zi, double m0, double2 e,
                                         double gamma, double a, double a1, double tol_step2,
                                         double tol_mu, int k, const double *sheet = nullptr,
                                         int n_poly = 0)
{
    const FieldAt Q = field_at<EQUAL>(S, zr, zi, m0, e, gamma, sheet, n_poly);
    return take_step(S, Q, 2.0 * S.s1r - S.Rr, 2.0 * S.s1i - S.Ri, zr, zi, gamma, a, a1,
                     tol_step2, tol_mu, k, sheet, n_poly);
}

__device__ __forceinline__ double2 cdiv(double2 p, double2 q)
{
    const double inv = rcp_refined<2>(fma(q.x, q.x, q.y * q.y));
    return make_double2(fma(p.x, q.x, p.y * q.y) * inv, fma(p.y, q.x, -(p.x * q.y)) * inv);
}

// Resident waves per SIMD the sweep and polish kernels are compiled for
// (register budget 512 / waves); the loops keep their instruction counts.
// MLCC_XCD_MAP 1 keeps every front's blocks on one XCD (one L2 per front's
// iterate).  Measured on n10k it is ~30% slower than the plain order, which
// spreads each front over all eight XCDs: the fronts in a full pass change
// from round to round, and whole fronts per XCD leave XCDs idle.
#ifndef MLCC_XCD_MAP
#define MLCC_XCD_MAP 0
#endif
#ifndef MLCC_SWEEP_WAVES
#define MLCC_SWEEP_WAVES 4
#endif
#ifndef MLCC_POLISH_WAVES
#define MLCC_POLISH_WAVES 4
#endif
// The persistent kernel with multipole sums spends most of its time waiting
// on dependent loads; trading registers for resident waves did not pay on
// n10k mixed (4 waves 331 ms per step, 5: 362, 6: 386, 8: 423: the spills
// cost more than the extra waves hide), so it keeps the sweep's count.
#ifndef MLCC_FMM_WAVES
#define MLCC_FMM_WAVES MLCC_SWEEP_WAVES
#endif

// Blocks with at most this many unconverged roots take the cooperative path.
constexpr int SPARSE_MAX = 16;

// An FP64 cold start still unsettled after this many sweeps (cold starts
// take 11-30) starts again from the second set of start values (the
// default of mlcc_cc_params.cold_restart_sweeps).
constexpr int STALL_START = 100;

// Newton steps a root may take within one polish pass.
constexpr int POLISH_STEPS = 3;

// Resident waves per SIMD the expansion kernel is compiled for: its 28 moment
// sums and the terms of four stars need more than the 168 registers of three.
#ifndef MLCC_EXPAND_WAVES
#define MLCC_EXPAND_WAVES 2
#endif

// ---------------------------------------------------------------------------
// Fast multipole star sums (Sec. 4.1: near stars directly, far stars through
// a local Taylor series)
// ---------------------------------------------------------------------------

// The stars are binned on a G x G grid of square cells of width w covering
// [c0 - 2R, c0 + 2R]^2, R the largest star distance from c0.  For a point z
// in cell C, the stars of C's 3 x 3 neighbourhood are summed directly; every
// other star is at least 1.5 w from C's centre c while |z - c| <= w / sqrt 2,
// and its terms come from C's local expansions
//   f_C(z) = sum_far w_i / (z - z_i) = sum_k a_k (z - c)^k,  a_k = -sum w_i / (z_i - c)^(k+1),
//   g_C(z) = the same with unit weights,
// (w_i = m_i, or 1 when all masses are equal and the kernels apply the mass
// once), whose derivatives give the other sums: sum w/(z - z_i)^2 = -f',
// sum w/(z - z_i)^3 = f''/2.  The ratio |z - c| / |z_i - c| <= 0.47 bounds the
// truncation after order p by ~0.47^(p+1) of each term.  The coefficients
// are stored scaled, b_k = a_k w^k = -(1/w) sum w_i v_i^(k+1) with
// v_i = w / (z_i - c), |v_i| <= 2/3, and the series is evaluated in
// tau = (z - c) / w, |tau| <= 0.71, so no power over- or underflows whatever
// the field's scale; f' and f'' take 1/w and 1/w^2.  Points outside the
// grid (|z - c0| >= 2R) use one expansion about c0 of all stars,
// f = sum_k M_k / (z - c0)^(k+1), M_k = sum w_i (z_i - c0)^k.  The polish's
// bound sum w |u|^4 takes, for the far stars, the per-cell constant
// sum_far w_i / dist(z_i, cell)^4 (or W / (|z - c0| - R)^4 outside).
struct FmmArgs {
    int32_t on, G, p, equal;
    int32_t stride;            // coefficients per cell: p + 1 rounded up to a multiple of 8
    double x0, y0, w, inv_w;   // grid origin (lower-left corner), cell width, 1 / w
    double cx, cy, R, wsum;    // c0, R, sum of the weights
    const int32_t *cell_start; // [G*G + 1]: stars of cell q are fstars[cell_start[q] ..)
    const double4 *fstars;     // stars sorted by cell: (x, y, m, 0)
    const double2 *cf, *cg;    // [G*G][stride]: b_k of f and of g (zero for k > p)
    const double *qfar;        // [G*G]
    const double2 *mf, *mg;    // [p + 1]: M_k about c0, weighted and unit
};

// Horner's rule for sum_k a_k t^k and its first two derivatives, over a
// coefficient row padded with zeros to a multiple of 8 (leading zeros leave
// the result unchanged).  Eight coefficients are loaded at a time, so the
// loads of a chunk are in flight together: the rows live in L2 or beyond,
// and one load per step would wait out that latency p times.
__device__ __forceinline__ void horner2(const double2 *__restrict__ a, int stride, double tr,
                                        double ti, double &fr, double &fi, double &dr, double &di,
                                        double &er, double &ei)
{
    fr = fi = dr = di = er = ei = 0.0;
    for (int c = stride - 8; c >= 0; c -= 8) {
        const double4 *a4 = reinterpret_cast<const double4 *>(a + c);
        double2 q[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double4 v = a4[j];
            q[2 * j] = make_double2(v.x, v.y);
            q[2 * j + 1] = make_double2(v.z, v.w);
        }
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            // e = e t + 2 d, d = d t + f, f = f t + a_k (e = f'', d = f')
            const double ner = er * tr - ei * ti + 2.0 * dr, nei = er * ti + ei * tr + 2.0 * di;
            const double ndr = dr * tr - di * ti + fr, ndi = dr * ti + di * tr + fi;
            const double nfr = fr * tr - fi * ti + q[j].x, nfi = fr * ti + fi * tr + q[j].y;
            er = ner; ei = nei; dr = ndr; di = ndi; fr = nfr; fi = nfi;
        }
    }
}

__device__ __forceinline__ void horner0(const double2 *__restrict__ a, int stride, double tr,
                                        double ti, double &fr, double &fi)
{
    fr = fi = 0.0;
    for (int c = stride - 8; c >= 0; c -= 8) {
        const double4 *a4 = reinterpret_cast<const double4 *>(a + c);
        double2 q[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double4 v = a4[j];
            q[2 * j] = make_double2(v.x, v.y);
            q[2 * j + 1] = make_double2(v.z, v.w);
        }
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            const double nfr = fr * tr - fi * ti + q[j].x, nfi = fr * ti + fi * tr + q[j].y;
            fr = nfr; fi = nfi;
        }
    }
}

// Far-field sums at z: f, f', f'' of the weighted expansion, g of the unit
// one (when want_g; the polish does not use it), and the bound on
// sum_far w |u|^4.  Sets `cell` to the cell index, or -1 outside the grid
// (then every star is far).
__device__ __forceinline__ void fmm_far(const FmmArgs &M, double zr, double zi, int &cell,
                                        double2 &f, double2 &f1, double2 &f2, double2 &g,
                                        double &q, bool want_g)
{
    const double fx = floor((zr - M.x0) / M.w), fy = floor((zi - M.y0) / M.w);
    if (fx >= 0.0 && fy >= 0.0 && fx < (double)M.G && fy < (double)M.G) {
        const int ix = (int)fx, iy = (int)fy;
        cell = iy * M.G + ix;
        const double tr = (zr - (M.x0 + (ix + 0.5) * M.w)) * M.inv_w;
        const double ti = (zi - (M.y0 + (iy + 0.5) * M.w)) * M.inv_w;
        const double2 *a = M.cf + (int64_t)cell * M.stride;
        horner2(a, M.stride, tr, ti, f.x, f.y, f1.x, f1.y, f2.x, f2.y);
        const double iw2 = M.inv_w * M.inv_w;
        f1.x *= M.inv_w; f1.y *= M.inv_w;
        f2.x *= iw2; f2.y *= iw2;
        if (M.equal) {
            g = f;
        } else if (want_g) {
            horner0(M.cg + (int64_t)cell * M.stride, M.stride, tr, ti, g.x, g.y);
        } else {
            g = make_double2(0.0, 0.0);
        }
        q = M.qfar[cell];
        return;
    }
    cell = -1;
    // t = 1 / (z - c0); f = t A(t), f' = -t^2 B(t), f'' = t^3 C(t) with
    // A = sum M_k t^k, B = sum (k+1) M_k t^k, C = sum (k+1)(k+2) M_k t^k
    const double dx = zr - M.cx, dy = zi - M.cy;
    const double r2 = dx * dx + dy * dy;
    const double tr = dx / r2, ti = -dy / r2;
    double Ar = M.mf[M.p].x, Ai = M.mf[M.p].y;
    double Br = (M.p + 1) * Ar, Bi = (M.p + 1) * Ai;
    double Cr = (double)(M.p + 1) * (M.p + 2) * Ar, Ci = (double)(M.p + 1) * (M.p + 2) * Ai;
    double Gr = M.mg[M.p].x, Gi = M.mg[M.p].y;
    for (int k = M.p - 1; k >= 0; --k) {
        const double2 mk = M.mf[k];
        double nr = Ar * tr - Ai * ti + mk.x, ni = Ar * ti + Ai * tr + mk.y;
        Ar = nr; Ai = ni;
        nr = Br * tr - Bi * ti + (k + 1) * mk.x; ni = Br * ti + Bi * tr + (k + 1) * mk.y;
        Br = nr; Bi = ni;
        const double c = (double)(k + 1) * (k + 2);
        nr = Cr * tr - Ci * ti + c * mk.x; ni = Cr * ti + Ci * tr + c * mk.y;
        Cr = nr; Ci = ni;
        const double2 gk = M.mg[k];
        nr = Gr * tr - Gi * ti + gk.x; ni = Gr * ti + Gi * tr + gk.y;
        Gr = nr; Gi = ni;
    }
    const double t2r = tr * tr - ti * ti, t2i = 2.0 * tr * ti;
    const double t3r = t2r * tr - t2i * ti, t3i = t2r * ti + t2i * tr;
    f = make_double2(tr * Ar - ti * Ai, tr * Ai + ti * Ar);
    f1 = make_double2(-(t2r * Br - t2i * Bi), -(t2r * Bi + t2i * Br));
    f2 = make_double2(t3r * Cr - t3i * Ci, t3r * Ci + t3i * Cr);
    g = M.equal ? f : make_double2(tr * Gr - ti * Gi, tr * Gi + ti * Gr);
    const double dd = sqrt(r2) - M.R;
    q = M.wsum / (dd * dd * dd * dd);
}

// One far star's place in a cell's expansion, the next power of v, and the
// cell's centre, as both kernels below form them: each product and sum is
// written out, so that their rows agree to the last bit.
__device__ __forceinline__ void p2l_star(double w, double dx, double dy, double &vr, double &vi)
{
    const double r2 = fma(dx, dx, dy * dy);
    vr = w * dx / r2;
    vi = -w * dy / r2;
}

__device__ __forceinline__ void p2l_next(double vr, double vi, double &pr, double &pi)
{
    const double tr = fma(vr, pr, -(vi * pi));
    pi = fma(vr, pi, vi * pr);
    pr = tr;
}

__device__ __forceinline__ double2 p2l_centre(double x0, double y0, double w, int ix, int iy)
{
    return make_double2(fma(w, ix + 0.5, x0), fma(w, iy + 0.5, y0));
}

// Local expansions of every cell from its far stars, one work group of 64
// lanes per cell.  The stars go by in blocks of 64: lane k takes star k of
// the block, forms v = w / (z_k - c) (0 for a star of the 3 x 3 near cells,
// whose cell index rides in the record's fourth component) and writes its
// powers v^1 .. v^stride to LDS; then lane j adds up power j + 1 over the
// block's stars, weighted (f) and unweighted (g).  Successive products cost
// one complex multiply per power, against ~7 for raising each lane's star
// to its own power.  Lane k also adds its star's term of the bound
// sum_far w_i / dist(z_i, cell)^4.
__global__ void __launch_bounds__(64)
fmm_p2l(int32_t G, int32_t p, int32_t stride, double x0, double y0, double w, int32_t equal,
        int32_t n, const double4 *__restrict__ fstars, double2 *__restrict__ cf,
        double2 *__restrict__ cg, double *__restrict__ qfar)
{
    __shared__ double2 pw[64 * 65];   // pw[j * 65 + k] = v_k^(j+1); the pad spreads the banks
    __shared__ double wk[64];
    const int cell = blockIdx.x;
    const int ix = cell % G, iy = cell / G;
    const double2 ctr = p2l_centre(x0, y0, w, ix, iy);
    const int lane = threadIdx.x;
    double fr = 0.0, fi = 0.0, gr = 0.0, gi = 0.0, q = 0.0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        double vr = 0.0, vi = 0.0, wi = 0.0;
        if (i < n) {
            const double4 st = fstars[i];
            const int sc = (int)st.w;
            const int sx = sc % G, sy = sc / G;
            if (abs(sx - ix) > 1 || abs(sy - iy) > 1) {
                const double dx = st.x - ctr.x, dy = st.y - ctr.y;
                p2l_star(w, dx, dy, vr, vi);
                wi = equal ? 1.0 : st.z;
                const double ex = fmax(fabs(dx) - 0.5 * w, 0.0), ey = fmax(fabs(dy) - 0.5 * w, 0.0);
                const double d2 = ex * ex + ey * ey;
                q += wi / (d2 * d2);
            }
        }
        double pr = vr, pi = vi;
        for (int j = 0; j < stride; ++j) {
            pw[j * 65 + lane] = make_double2(pr, pi);
            p2l_next(vr, vi, pr, pi);
        }
        wk[lane] = wi;
        __syncthreads();
        if (lane < stride) {
#pragma unroll 8
            for (int k = 0; k < 64; ++k) {
                const double2 v = pw[lane * 65 + k];
                const double wt = wk[k];
                fr = fma(-wt, v.x, fr);
                fi = fma(-wt, v.y, fi);
                gr -= v.x;
                gi -= v.y;
            }
        }
        __syncthreads();
    }
    wave_sum(q);
    if (lane < stride) {
        const double s = lane <= p ? 1.0 / w : 0.0;
        cf[(int64_t)cell * stride + lane] = make_double2(fr * s, fi * s);
        cg[(int64_t)cell * stride + lane] = make_double2(gr * s, gi * s);
    }
    if (lane == 0) qfar[cell] = q;
}

// The same coefficients bit for bit, a lane a cell, for many cells: the columns
// of a field are numbered by its cold start, which follows the last bit of these
// sums, so every order adds up its terms star by star as above.  (The bounds
// qfar add theirs in another order: they say how far a series or a Newton step
// is trusted, and enter no FP64 cold start.)  A wave takes 64 cells and KB of the
// orders from k0 on: the stars go by in tiles parked in
// LDS, and their powers, by the same successive products, are added straight
// into registers (6 FP64 instructions per order and star, 8 for unequal masses,
// 4 for the orders before k0).  It is bound by that arithmetic on as many SIMDs
// as there are waves.  N = 10,000 (16,900 cells): 14.9 ms with one work group a
// cell and the powers through LDS, 8.0 with this (4.0 with the stars split too,
// but then the columns came out numbered otherwise); 96 fields of 50 to 600
// stars, 96 launches there and one here: 1.95 -> 0.65 ms; N = 3,000 (5,200
// cells): 1.4 there, 2.4 here by its cost per star.
struct P2lJob {
    int32_t field, cell0, k0, n;   // n: the field's stars
};

template <int KB, bool EQUAL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 8)))
fmm_p2l_lanes(const P2lJob *__restrict__ jobs, const FmmArgs *__restrict__ recs)
{
    __shared__ double4 tile[64];   // x, y, weight, cell column and row
    const P2lJob J = jobs[blockIdx.x];
    const FmmArgs &M = recs[J.field];
    const int n = J.n;
    const double4 *__restrict__ st = M.fstars;
    const int lane = threadIdx.x, G = M.G;
    const int cell = min(J.cell0 + lane, G * G - 1);
    const int ix = cell % G, iy = cell / G;
    const double w = M.w;
    const double2 ctr = p2l_centre(M.x0, M.y0, w, ix, iy);
    double fr[KB], fi[KB], gr[KB], gi[KB], q = 0.0;
#pragma unroll
    for (int k = 0; k < KB; ++k) fr[k] = fi[k] = gr[k] = gi[k] = 0.0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int cnt = min(64, n - i0);
        if (lane < cnt) {
            double4 a = st[i0 + lane];
            const int sc = (int)a.w;
            a.w = __hiloint2double(sc / G, sc % G);
            tile[lane] = a;
        }
        wave_sync();
        // two stars at a time, for two independent chains of products; each sum
        // still takes its terms in star order
        for (int t = 0; t < cnt; t += 2) {
            double vr[2], vi[2], pr[2], pi[2], wi[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double4 a = tile[min(t + c, cnt - 1)];
                const int sx = __double2loint(a.w), sy = __double2hiint(a.w);
                const bool far = t + c < cnt && (abs(sx - ix) > 1 || abs(sy - iy) > 1);
                const double dx = a.x - ctr.x, dy = a.y - ctr.y;
                double br, bi;
                p2l_star(w, dx, dy, br, bi);
                vr[c] = far ? br : 0.0;
                vi[c] = far ? bi : 0.0;
                wi[c] = EQUAL ? 1.0 : a.z;
                pr[c] = vr[c];
                pi[c] = vi[c];
                if (J.k0 == 0 && far) {
                    const double ex = fmax(fabs(dx) - 0.5 * w, 0.0);
                    const double ey = fmax(fabs(dy) - 0.5 * w, 0.0);
                    const double d2 = fma(ex, ex, ey * ey);
                    q += wi[c] / (d2 * d2);
                }
            }
            auto next = [&](int c) { p2l_next(vr[c], vi[c], pr[c], pi[c]); };
#pragma unroll 4
            for (int k = 0; k < J.k0; ++k) {
                next(0);
                next(1);
            }
#pragma unroll
            for (int k = 0; k < KB; ++k) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (EQUAL) {
                        fr[k] -= pr[c];
                        fi[k] -= pi[c];
                    } else {
                        fr[k] = fma(-wi[c], pr[c], fr[k]);
                        fi[k] = fma(-wi[c], pi[c], fi[k]);
                        gr[k] -= pr[c];
                        gi[k] -= pi[c];
                    }
                    next(c);
                }
            }
        }
        wave_sync();
    }
    if (J.cell0 + lane >= G * G) return;
    double2 *cf = const_cast<double2 *>(M.cf) + (int64_t)cell * M.stride + J.k0;
    double2 *cg = const_cast<double2 *>(M.cg) + (int64_t)cell * M.stride + J.k0;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        if (J.k0 + k >= M.stride) continue;
        const double s = J.k0 + k <= M.p ? 1.0 / w : 0.0;
        const double2 f = make_double2(fr[k] * s, fi[k] * s);
        cf[k] = f;
        cg[k] = EQUAL ? f : make_double2(gr[k] * s, gi[k] * s);
    }
    if (J.k0 == 0) const_cast<double *>(M.qfar)[cell] = q;
}

// Calls body(star) for the stars of the 3 x 3 cells around `cell`, in the
// order of the sorted list (the block's three grid rows, each a run of
// adjacent cells), and returns their number.  The records are read
// NEAR_BATCH at a time, all loads of a batch issued before the first body
// runs: lanes of a wave sit in different cells, so every record is a
// gather from L2, and one load per body would wait out that latency for
// each near star.
#ifndef MLCC_NEAR_BATCH
#define MLCC_NEAR_BATCH 4
#endif
constexpr int NEAR_BATCH = MLCC_NEAR_BATCH;

template <class Body>
__device__ __forceinline__ int fmm_near(const FmmArgs &M, int cell, Body &&body)
{
    if (cell < 0) return 0;
    const int ix = cell % M.G, iy = cell / M.G;
    const int xa = max(ix - 1, 0), xb = min(ix + 1, M.G - 1);
    int lo[3], len[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int y = iy - 1 + r;
        // the cells of one grid row are adjacent in the sorted order
        const bool in = y >= 0 && y < M.G;
        const int q0 = (in ? y : iy) * M.G + xa, q1 = (in ? y : iy) * M.G + xb;
        const int i0 = M.cell_start[q0], i1 = M.cell_start[q1 + 1];
        lo[r] = i0;
        len[r] = in ? i1 - i0 : 0;
    }
    const int l01 = len[0] + len[1], n = l01 + len[2];
    for (int j = 0; j < n; j += NEAR_BATCH) {
        double4 rec[NEAR_BATCH];
#pragma unroll
        for (int u = 0; u < NEAR_BATCH; ++u) {
            const int t = j + u;
            const int i = t < len[0] ? lo[0] + t : t < l01 ? lo[1] + (t - len[0]) : lo[2] + (t - l01);
            rec[u] = M.fstars[t < n ? i : 0];   // past the end: a valid record, not used
        }
#pragma unroll
        for (int u = 0; u < NEAR_BATCH; ++u)
            if (j + u < n) body(rec[u]);
    }
    return n;
}

// A wave's multipole tallies (see FMM_STRIPES): near-field star terms,
// far-field evaluations (lanes that updated a root) and those evaluations
// times the field's star count (the direct terms they replace).  The values
// are wave-uniform.
struct FmmTally {
    unsigned long long near = 0, far = 0, far_n = 0;
};

__device__ __forceinline__ void fmm_count(FmmTally &t, bool act, int n_near, int n_stars)
{
    int v = act ? n_near : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    v = __builtin_amdgcn_readfirstlane(v);
    const int n_act = __popcll(__ballot(act));
    t.near += (unsigned long long)v;
    t.far += (unsigned long long)n_act;
    t.far_n += (unsigned long long)n_act * (unsigned long long)n_stars;
}

// Adds a wave's tallies to its work group's copy (kind: FMM_T_*).
__device__ __forceinline__ void fmm_flush(unsigned long long *tally, int kind, const FmmTally &t)
{
    if ((threadIdx.x & 63) == 0 && t.far) {
        unsigned long long *s = tally + (blockIdx.x % FMM_STRIPES) * FMM_STRIPE_U64 + kind;
        atomicAdd(&s[0], t.near);
        atomicAdd(&s[1], t.far);
        atomicAdd(&s[2], t.far_n);
    }
}

// Arguments shared by the kernels of a round.  Stars of every realisation
// are concatenated; each front names its realisation, and the grid maps a
// block to (front, block within the front) through bmap.
template <class T> struct RoundArgs {
    const T *stars;
    const Real *reals;
    const int2 *bmap;
    const Front *fronts;
    int32_t *flagrow;
    const double2 *cur;
    double2 *nxt;
    const double2 *unit;   // (cos phi_j, -sin phi_j)
    double tol_step, tol_step2, tol_mu;
    double *out_re, *out_im, *caus_re, *caus_im;
    double2 *bnd;
    int32_t *counts;
    int32_t *passupd;  // per front: roots updated by this round's pass (the control kernel sums them)
    Control *ctl;
    unsigned long long *fmm_tally;   // multipole tallies (FMM_STRIPES copies)
    double4 *vieta;    // two per block: row sums, and their error terms
    double *errbuf;    // estimated error of each polished root
    int32_t predictor;
    int32_t xfrom;      // finished rows a warm row needs behind it to be expanded (0: none is)
    int32_t persistent; // the persistent scheduler: iterates by per-front parity
    double2 *iter0, *iter1;
    const double *sheet; // rectangular fields' sheet records (Real::sheet_off)
    const FmmArgs *fmm;  // fast multipole star sums: one record per field (kernels built with them)
    int32_t *next_row, *stuck;   // expand_rows: per block its next row, and whether it is stuck there
    int32_t *root_row;           // FP64: per root its own next row
};

// What one block knows about its front and star field.
template <class T> struct BlockCtx {
    int f, q, r, k0, k, lane, n_r, n_stars, row, stamp, dir, pred;
    int n_poly, n_extra;   // rectangular field: sheet terms and extra roots (else 0)
    const double *sheet;   // its record: d_2k, then d_2k / (2k + 1), then extra seeds
    double sheet_c;        // |c|, the distance of its corners
    int vslot;   // this block's slot in the per-block row sums (front order)
    int hist, end_row;   // finished rows behind the current one (<= 3); the front's last row
    bool valid, boundary;
    bool reseed, second;   // restart the row from its start values; from the second seeds
    bool fast;       // root-root terms in FP32 (fast_roots_pass)
    bool fresh;      // first pass over the row (roots flagged by then: expand_rows)
    bool has_bnd;    // the front's end row is a duplicate boundary row
    bool settled;    // its row is finished already (Front::settled)
    int32_t *count, *upd;   // the pass's totals: roots left open (or moving), updates made
    int64_t base_f, out_off, bnd_row_off;
    const T *stars;
    const double2 *zsrc;
    double2 *nxt;
    double m0, gamma, a, a1;
    double2 e;   // (1 - kappa_s) e^{-i phi} of the front's row
};

// Which FP64 Aberth passes take the root-root sum in FP32 (add_root_hl):
// warm rows of a field solved in MLCC_FP64_R32.  Cold starts, where the
// repulsion between the iterates steers global convergence from the seeds,
// MLCC_FP64 and the mixed form's FP64 restarts keep it in FP64.
__device__ __forceinline__ bool fast_roots_pass(const Front &fr, const Real &r)
{
    return r.root32 && fr.dir != 0 && fr.mode == PH_F64;
}

// Context of block q of front f, whose record is F (in LDS under the
// persistent schedule); `count` and `upd` take the pass's totals.
template <class T>
__device__ __forceinline__ void enter_fq(const RoundArgs<T> &A, const Front *F, int f, int q,
                                         int32_t *count, int32_t *upd, BlockCtx<T> &B)
{
    B.f = f;
    B.q = q;
    const Real *R = A.reals + F->real;
    B.r = F->real;
    B.row = F->row;
    B.stamp = F->stamp;
    B.vslot = F->blk0 + B.q;
    B.dir = F->dir;
    B.pred = (F->fresh && F->dir != 0 && F->hist >= 2) ? min(A.predictor, F->hist - 1) : 0;
    B.reseed = F->reseed != 0;
    B.second = F->seedvar > 0;
    B.fast = fast_roots_pass(*F, *R);
    B.fresh = F->fresh != 0;
    B.has_bnd = F->bnd_slot >= 0;
    B.settled = F->settled != 0;
    B.count = count;
    B.upd = upd;
    B.hist = F->hist;
    B.end_row = F->end_row;
    B.n_r = R->n_r;
    B.n_stars = R->n_stars;
    B.n_poly = R->n_poly;
    B.n_extra = R->n_extra;
    B.sheet = R->n_poly > 0 ? A.sheet + R->sheet_off : nullptr;
    B.sheet_c = R->sheet_c;
    B.stars = A.stars + R->star_off;
    B.m0 = R->m0;
    B.gamma = R->gamma;
    B.a = R->a;
    B.a1 = R->a1;
    B.base_f = F->it_off;
    if (A.persistent) {   // every front keeps its own ping-pong parity
        B.zsrc = (F->par ? A.iter1 : A.iter0) + F->it_off;
        B.nxt = F->par ? A.iter0 : A.iter1;
    } else {
        B.zsrc = A.cur + A.fronts[F->src].it_off;
        B.nxt = A.nxt;
    }
    B.out_off = R->out_off;
    B.boundary = B.has_bnd && B.row == F->end_row;
    B.bnd_row_off = R->bnd_off + (int64_t)max(F->bnd_slot, 0) * R->n_r;
    const double2 u = A.unit[B.row];
    B.e = make_double2(B.a * u.x, B.a * u.y);
    B.lane = threadIdx.x & 63;
    B.k0 = B.q * 64;
    B.k = B.k0 + B.lane;
    B.valid = B.k < B.n_r;
}

// Block context of this work group in a round: (front, block) from bmap.
template <class T>
__device__ __forceinline__ bool enter(const RoundArgs<T> &A, int phase, BlockCtx<T> &B)
{
    const int2 fq = A.bmap[blockIdx.x];
    const Front *F = A.fronts + fq.x;
    if (F->state != FRONT_ACTIVE || F->phase != phase) return false;
    enter_fq(A, F, fq.x, fq.y, A.counts + fq.x, A.passupd + fq.x, B);
    return true;
}

// Start of a new row's first pass for root k: extrapolation along its chain
// from the previous row (z1, the converged iterate) and the rows before it,
// which the subchain has already written to the output (same labels):
// linear 2 z1 - z2, quadratic 3 (z1 - z2) + z3.
template <class T>
__device__ __forceinline__ void predict(const RoundArgs<T> &A, const BlockCtx<T> &B, int k,
                                        double &zr, double &zi)
{
    const int64_t o2 = B.out_off + (int64_t)(B.row - 2 * B.dir) * B.n_r + k;
    const double x2 = A.out_re[o2], y2 = A.out_im[o2];
    if (B.pred == 1) {
        zr = 2.0 * zr - x2;
        zi = 2.0 * zi - y2;
    } else {
        const int64_t o3 = o2 - (int64_t)B.dir * B.n_r;
        zr = fma(3.0, zr - x2, A.out_re[o3]);
        zi = fma(3.0, zi - y2, A.out_im[o3]);
    }
}

// Write-back of a converged root: its row of the output (or the duplicate
// boundary row of a subchain) and its caustic image.
template <class T>
__device__ __forceinline__ void put(const RoundArgs<T> &A, const BlockCtx<T> &B, int k,
                                    const Update &u)
{
    if (B.boundary) {
        A.bnd[B.bnd_row_off + k] = make_double2(u.zr, u.zi);
        return;
    }
    const int64_t o = B.out_off + (int64_t)B.row * B.n_r + k;
    A.out_re[o] = u.zr;
    A.out_im[o] = u.zi;
    if (A.caus_re) {
        A.caus_re[o] = u.wr;
        A.caus_im[o] = u.wi;
    }
}

// Root k of the current row where it is accepted already.
template <class T>
__device__ __forceinline__ double2 accepted_root(const RoundArgs<T> &A, const BlockCtx<T> &B, int k)
{
    if (B.boundary) return A.bnd[B.bnd_row_off + k];
    const int64_t o = B.out_off + (int64_t)B.row * B.n_r + k;
    return make_double2(A.out_re[o], A.out_im[o]);
}

// ---------------------------------------------------------------------------
// Star sums of Newton-like steps, and FP64 rows from their chains
// ---------------------------------------------------------------------------

// Sums for the Newton polish: s0 = sum m u, s2 = sum m u^2, s3 = sum m u^3
// (F = gamma + s2 - (1 - kappa_s) e^{-i phi}, F' = -2 s3) and the real
// q = sum m |u|^4, which bounds |F''| = 6 |sum m u^4| <= 6 q.
struct PSums {
    double s0r, s0i, s2r, s2i, s3r, s3i, q;
};

__device__ __forceinline__ void zero(PSums &S)
{
    S.s0r = S.s0i = S.s2r = S.s2i = S.s3r = S.s3i = S.q = 0.0;
}

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star_polish_inv(PSums &S, double dx, double dy, double inv,
                                                    const T &s);

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star_polish(PSums &S, double zr, double zi, const T &s)
{
    const double dx = zr - s.x;
    const double dy = zi - s.y;
    add_star_polish_inv<EQUAL>(S, dx, dy, rcp_refined<RCP_STAR>(fma(dx, dx, dy * dy)), s);
}

// G consecutive polish star terms sharing one refined reciprocal.
template <bool EQUAL, int G, class T>
__device__ __forceinline__ void add_star_polish_group(PSums &S, double zr, double zi, const T *r)
{
    double dx[G], dy[G], q[G], iq[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        dx[j] = zr - r[j].x;
        dy[j] = zi - r[j].y;
        q[j] = fma(dx[j], dx[j], dy[j] * dy[j]);
    }
    rcp_group<G, RCP_STAR>(q, iq);
#pragma unroll
    for (int j = 0; j < G; ++j) add_star_polish_inv<EQUAL>(S, dx[j], dy[j], iq[j], r[j]);
}

template <bool EQUAL, class T>
__device__ __forceinline__ void add_star_polish_inv(PSums &S, double dx, double dy, double inv,
                                                    const T &s)
{
    // u = ux - i uy, a = ux^2, b = uy^2:  u^2 = (a - b) - 2i ux uy,
    // u^3 = ux (a - 3b) + i uy (b - 3a), formed from b alone as in
    // add_star_inv (t = a - b = inv - 2b, a - 3b = t - 2b, b - 3a = -2t - inv);
    // |u|^4 = inv^2
    // (s2i accumulates sum m ux uy; polish_finish turns it into Im s2 = -2 that)
    const double uy = dy * inv;
    const double b = uy * uy;
    const double t = fma(-2.0, b, inv);
    const double c3r = fma(-2.0, b, t), c3i = fma(-2.0, t, -inv);
    if (EQUAL) {
        const double ux = dx * inv;
        S.s0r += ux; S.s0i -= uy;
        S.s2r += t;
        S.s2i = fma(ux, uy, S.s2i);
        S.s3r = fma(ux, c3r, S.s3r);
        S.s3i = fma(uy, c3i, S.s3i);
        S.q = fma(inv, inv, S.q);
    } else {
        // the mass enters through m inv, shared by m u = conj(d) m inv and
        // the bound's m inv^2; u's real part is not needed on its own
        const double mi = StarRec<EQUAL>::mass(s);
        const double minv = mi * inv;
        const double mux = dx * minv, muy = mi * uy;
        S.s0r += mux; S.s0i -= muy;
        S.s2r = fma(mi, t, S.s2r);
        S.s2i = fma(mux, uy, S.s2i);
        S.s3r = fma(mux, c3r, S.s3r);
        S.s3i = fma(muy, c3i, S.s3i);
        S.q = fma(minv, inv, S.q);
    }
}

// Star sums at (zr, zi) for the lanes of `mask` (PSums; what is not read is
// not computed).  Multipole sums: every lane its cell's series and near
// stars, whose number goes to n_near.  Direct sums: the whole wave one root
// after another when the mask holds few, else the star tiles for every lane.
template <bool EQUAL, bool FMM>
__device__ __forceinline__ void newton_sums(const RoundArgs<typename StarRec<EQUAL>::T> &A,
                                            const BlockCtx<typename StarRec<EQUAL>::T> &B,
                                            unsigned long long mask, double zr, double zi,
                                            double4 *tiles, PSums &S, int &n_near)
{
    using T = typename StarRec<EQUAL>::T;
    zero(S);
    n_near = 0;
    if constexpr (FMM) {
        int cell;
        double2 f, f1, f2, g;
        double q;
        fmm_far(A.fmm[B.r], zr, zi, cell, f, f1, f2, g, q, false);
        n_near = fmm_near(A.fmm[B.r], cell, [&](const double4 &s4) {
            if constexpr (EQUAL) add_star_polish<EQUAL>(S, zr, zi, make_double2(s4.x, s4.y));
            else add_star_polish<EQUAL>(S, zr, zi, s4);
        });
        S.s0r += f.x; S.s0i += f.y;
        S.s2r -= f1.x; S.s2i += 0.5 * f1.y;
        S.s3r += 0.5 * f2.x; S.s3i += 0.5 * f2.y;
        S.q += q;
    } else if (__popcll(mask) <= SPARSE_MAX) {
        while (mask) {
            const int l = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            const double xk = __shfl(zr, l, 64), yk = __shfl(zi, l, 64);
            PSums C;
            zero(C);
            each_strided(B.stars, B.n_stars, B.lane,
                         [&](int, const T &st) { add_star_polish<EQUAL>(C, xk, yk, st); });
            wave_sum(C.s0r); wave_sum(C.s0i); wave_sum(C.s2r); wave_sum(C.s2i);
            wave_sum(C.s3r); wave_sum(C.s3i); wave_sum(C.q);
            if (B.lane == l) S = C;
        }
    } else {
        stream_tiles_grouped(B.stars, B.n_stars, reinterpret_cast<T *>(tiles),
                             [&](auto g, const T *r) {
                                 add_star_polish_group<EQUAL, decltype(g)::value>(S, zr, zi, r);
                             });
    }
}

// Sum over the wave of a per-lane count.
__device__ __forceinline__ int wave_count(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return __builtin_amdgcn_readfirstlane(v);
}

// ---------------------------------------------------------------------------
// Rows from expansions
// ---------------------------------------------------------------------------

// A row moves each root by about half a phase step (in units of its distance
// to the nearest star), so the star field around a root is the same function
// row after row, and its Taylor expansion about one point z0 of the chain
// serves many rows:
//   f(z) = sum m_i / (z - z_i) = sum_k s_{k+1} (z0 - z)^k,   s_k = sum m_i u_i^k,
//   u_i = 1 / (z0 - z_i),
// whose derivatives give the other sums (sum m u^2 = -f', sum m u^3 = f''/2,
// sum m u^4 = -f'''/6).  Every star enters the moments s_k directly (with
// multipole sums: the near stars, and the cell's series re-centred on z0), in
// FP64.  With x = |z - z0| max|u_i|, the terms left out of sum m u^2 are at
// most M x^(M-1) sum m |u|^4 / max|u|^2 / (1 - x)^2 for M moments; the
// expansion is used where that is below EXP_TAIL, under the rounding of the
// sum itself (~1e-16 sum m |u|^2).
//
// A direct star term costs ~80 instructions against ~19 (23 for unequal
// masses) for the sums of one row, and a row from the expansion ~600
// instructions a root, whatever N.  14 moments let x reach ~0.04 (each row
// moves x by 1/2 to 3 phase steps): tens of rows at 10,000 phase steps, ~6 at
// 1,000.  Measured with 10 / 12 / 14 / 16 / 20 moments, ms a call: N = 6,000
// FP64 131 / 109 / 102 / 102 / 109; 40 fields mixed 152 / 75 / 65 / 61 / 59;
// N = 10,000 mixed with multipole sums 71 / 66 / 67 / 72 / 79.
#ifndef MLCC_MOMENTS
#define MLCC_MOMENTS 14
#endif
constexpr int NMOM = MLCC_MOMENTS;
constexpr double EXP_TAIL = 2e-17;
// A root takes steps D with the correction G = -F''/(2 F') (what the Aberth
// correction 2 S1 - R equals at a simple zero) while |G F/F'| < EXP_BASIN, deep
// inside its zero's basin; farther out, the mixed form takes plain Newton
// steps (its row identities tell when two columns end at one root) and FP64
// leaves the root to Aberth steps.  It is accepted inside the basin, when it is
// flagged and the step leaves less than EXP_ERR (of the order of |D|^3 |G|^2).
// A root this does not settle in EXP_STEPS steps is left to the row's passes.
constexpr double EXP_BASIN = 0.05;
constexpr double EXP_ERR = 1e-16;
// A new expansion is formed this share of the last one's reach ahead.
// (N = 6,000 FP64: 79 ms a call at 0, 72 at 1/2, 70 at 3/4 and 0.9.)
constexpr double EXP_LEAD = 0.75;
constexpr int EXP_STEPS = 4;
// Phase grids of at least this many steps take their warm rows from expansions
// (FP64 and MLCC_FP64_R32; the mixed form, whose blocks wait for each of their
// open roots).  On coarser ones a root leaves its expansion, or its zero's
// basin, nearly every row, and the passes alone are the faster way.  Time with
// expansions over time without, the mean and the slowest of 13 to 15 fields,
// batches and piece counts from 10 to 2,500 stars at 96 / 160 / 256 / 400 / 512
// steps: FP64 1.25 1.03 0.94 0.75 0.66, slowest 1.8 1.4 1.6 1.7 1.5 (a rectangular
// field of 40 stars), with multipole sums 1.28 1.02 0.88 0.67 0.58 and 1.6 1.4 1.5
// 1.05 1.1; mixed 1.83 1.51 1.19 0.92 0.86 and 4.6 4.1 2.4 1.5 1.2, with multipole
// sums 1.61 1.31 1.08 0.85 0.78 and 3.2 3.0 2.4 1.4 1.2.
constexpr int64_t EXP_MIN_STEPS = 256, EXP_MIN_STEPS_MIXED = 400;

struct Moments {
    double r[NMOM], i[NMOM];   // s_1 .. s_M
    double q, u2;              // sum m |u|^4, max |u|^2
};

__device__ __forceinline__ void zero(Moments &S)
{
#pragma unroll
    for (int k = 0; k < NMOM; ++k) S.r[k] = S.i[k] = 0.0;
    S.q = S.u2 = 0.0;
}

__device__ __forceinline__ void cfma(double &ar, double &ai, double br, double bi, double cr,
                                     double ci)
{
    ar = fma(br, cr, fma(-bi, ci, ar));
    ai = fma(br, ci, fma(bi, cr, ai));
}

// One star's term.  u .. u^4 are formed from |u|^2 as in add_star_inv; the
// higher powers go in fours, m u^(4j) times u, u^2, u^3 being added straight
// into the sums.
template <bool EQUAL>
__device__ __forceinline__ void add_moments(Moments &S, double dx, double dy, double inv, double m)
{
    const double ur = dx * inv, ui = -dy * inv;
    const double b = ui * ui, t = ur * ui;
    const double v2r = fma(-2.0, b, inv), v2i = t + t;
    const double v3r = ur * fma(-2.0, b, v2r), v3i = ui * fma(2.0, v2r, inv);
    const double inv2 = inv * inv;
    const double v4r = fma(-2.0 * v2i, v2i, inv2), v4i = 2.0 * v2r * v2i;
    S.u2 = fmax(S.u2, inv);
    double pr, pi;   // m u^(4j)
    if (EQUAL) {
        S.r[0] += ur;  S.i[0] += ui;
        S.r[1] += v2r; S.i[1] += v2i;
        S.r[2] += v3r; S.i[2] += v3i;
        S.q += inv2;
        pr = v4r; pi = v4i;
    } else {
        S.r[0] = fma(m, ur, S.r[0]);  S.i[0] = fma(m, ui, S.i[0]);
        S.r[1] = fma(m, v2r, S.r[1]); S.i[1] = fma(m, v2i, S.i[1]);
        S.r[2] = fma(m, v3r, S.r[2]); S.i[2] = fma(m, v3i, S.i[2]);
        S.q = fma(m, inv2, S.q);
        pr = m * v4r; pi = m * v4i;
    }
#pragma unroll
    for (int k = 3; k < NMOM; k += 4) {
        S.r[k] += pr;
        S.i[k] += pi;
        if (k + 1 < NMOM) cfma(S.r[k + 1], S.i[k + 1], pr, pi, ur, ui);
        if (k + 2 < NMOM) cfma(S.r[k + 2], S.i[k + 2], pr, pi, v2r, v2i);
        if (k + 3 < NMOM) cfma(S.r[k + 3], S.i[k + 3], pr, pi, v3r, v3i);
        if (k + 4 < NMOM) {
            const double tr = fma(pr, v4r, -pi * v4i);
            pi = fma(pr, v4i, pi * v4r);
            pr = tr;
        }
    }
}

// Four consecutive star terms at most, sharing one refined reciprocal.
template <bool EQUAL, int G, class T>
__device__ __forceinline__ void add_moments_group(Moments &S, double zr, double zi, const T *r)
{
    if constexpr (G > 4) {
        add_moments_group<EQUAL, G / 2>(S, zr, zi, r);
        add_moments_group<EQUAL, G / 2>(S, zr, zi, r + G / 2);
    } else {
        double dx[G], dy[G], q[G], iq[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            dx[j] = zr - r[j].x;
            dy[j] = zi - r[j].y;
            q[j] = fma(dx[j], dx[j], dy[j] * dy[j]);
        }
        rcp_group<G, RCP_STAR>(q, iq);
#pragma unroll
        for (int j = 0; j < G; ++j)
            add_moments<EQUAL>(S, dx[j], dy[j], iq[j], StarRec<EQUAL>::mass(r[j]));
    }
}

template <bool EQUAL, class T>
__device__ __forceinline__ void add_moments_star(Moments &S, double zr, double zi, const T &s)
{
    const double dx = zr - s.x, dy = zi - s.y;
    add_moments<EQUAL>(S, dx, dy, rcp_refined<RCP_STAR>(fma(dx, dx, dy * dy)),
                       StarRec<EQUAL>::mass(s));
}

// The far stars of a point inside the grid, which set the moments: the cell's
// series re-centred on the point (M Horner levels over one read of the row;
// far stars are at least w away).
__device__ __forceinline__ void set_moments_far(Moments &S, const FmmArgs &M, int cell, double tr,
                                                double ti)
{
    const double2 *a = M.cf + (int64_t)cell * M.stride;
    for (int c = M.stride - 8; c >= 0; c -= 8) {
        const double4 *a4 = reinterpret_cast<const double4 *>(a + c);
        double2 w[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double4 v = a4[j];
            w[2 * j] = make_double2(v.x, v.y);
            w[2 * j + 1] = make_double2(v.z, v.w);
        }
#pragma unroll
        for (int j = 7; j >= 0; --j) {
#pragma unroll
            for (int k = NMOM - 1; k >= 0; --k) {
                const double xr = k ? S.r[k - 1] : w[j].x, xi = k ? S.i[k - 1] : w[j].y;
                const double nr = fma(S.r[k], tr, fma(-S.i[k], ti, xr));
                S.i[k] = fma(S.r[k], ti, fma(S.i[k], tr, xi));
                S.r[k] = nr;
            }
        }
    }
    double sc = 1.0;   // (-1 / w)^k
#pragma unroll
    for (int k = 0; k < NMOM; ++k) {
        S.r[k] *= sc;
        S.i[k] *= sc;
        sc *= -M.inv_w;
    }
    S.q = M.qfar[cell];
    S.u2 = M.inv_w * M.inv_w;
}

// A rectangular field's sheet adds the polynomial p(z) = sum_k dmap_k
// z^(2k+1) to f (its map term; the sheet's share of F is -P = -p', as the
// stars' is sum m u^2 = -f').  Its Taylor terms about z0 by synthetic
// division; a second division with |dmap| at max(|z0|, |c| / 2) bounds the
// first one left out, and the ratio of those that follow is at most
// t / (M |z0|).
__device__ __forceinline__ void add_moments_sheet(Moments &S, const double *__restrict__ dmap,
                                                  int n, double cabs, double zr, double zi)
{
    double br[NMOM], bi[NMOM], g[NMOM];
#pragma unroll
    for (int k = 0; k < NMOM; ++k) br[k] = bi[k] = g[k] = 0.0;
    const double az = fmax(sqrt(fma(zr, zr, zi * zi)), 0.5 * cabs);
    for (int d = 2 * n + 1; d >= 0; --d) {
        const double cf = (d & 1) && d >= 3 ? dmap[(d - 3) >> 1] : 0.0;
#pragma unroll
        for (int k = NMOM - 1; k >= 0; --k) {
            const double xr = k ? br[k - 1] : cf, xi = k ? bi[k - 1] : 0.0;
            const double nr = fma(br[k], zr, fma(-bi[k], zi, xr));
            bi[k] = fma(br[k], zi, fma(bi[k], zr, xi));
            br[k] = nr;
            g[k] = fma(g[k], az, k ? g[k - 1] : fabs(cf));
        }
    }
#pragma unroll
    for (int k = 0; k < NMOM; ++k) {
        S.r[k] += (k & 1) ? -br[k] : br[k];
        S.i[k] += (k & 1) ? -bi[k] : bi[k];
    }
    const double u = fmax((2.0 * n + 2.0) / (NMOM * az), sqrt(S.u2));
    double q = g[NMOM - 1];
#pragma unroll
    for (int k = 0; k < NMOM - 4; ++k) q /= u;
    S.q += q;
    S.u2 = u * u;
}

// The wave's sums of its lanes' moments, in every lane.  At each level a lane
// hands half of its values over and adds the other half, so 32 exchanges and
// as many broadcasts do what six exchanges a value did (174).
__device__ __forceinline__ void spread_sums(Moments &S, int lane)
{
    static_assert(2 * NMOM + 1 <= 32, "one value a pair of lanes");
    double v[32];
#pragma unroll
    for (int k = 0; k < NMOM; ++k) {
        v[2 * k] = S.r[k];
        v[2 * k + 1] = S.i[k];
    }
    v[2 * NMOM] = S.q;
#pragma unroll
    for (int k = 2 * NMOM + 1; k < 32; ++k) v[k] = 0.0;
#pragma unroll
    for (int half = 16; half >= 1; half >>= 1) {
        const bool up = lane & (2 * half);
#pragma unroll
        for (int j = 0; j < half; ++j) {
            const double give = up ? v[j] : v[j + half], keep = up ? v[j + half] : v[j];
            v[j] = keep + __shfl_xor(give, 2 * half, 64);
        }
    }
    const double w = v[0] + __shfl_xor(v[0], 1, 64);   // value lane / 2
    auto from = [&](int src) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(w), src),
                                __builtin_amdgcn_readlane(__double2loint(w), src));
    };
#pragma unroll
    for (int k = 0; k < NMOM; ++k) {
        S.r[k] = from(4 * k);
        S.i[k] = from(4 * k + 2);
    }
    S.q = from(4 * NMOM);
}

// Moments about (zr, zi) for the lanes of `mask`; the other lanes keep theirs
// where the mask holds few lanes and no multipole sums are on, and receive
// moments about their own (zr, zi) otherwise, unless they are out of the grid.
// Direct sums: the whole wave one root after another when the mask holds few,
// else the star tiles for every lane.  Multipole sums: each lane its cell's
// series and near stars; a lane of the mask outside the grid sums over all stars.
template <bool EQUAL, bool FMM>
__device__ __forceinline__ void sum_moments(const RoundArgs<typename StarRec<EQUAL>::T> &A,
                                            const BlockCtx<typename StarRec<EQUAL>::T> &B,
                                            unsigned long long mask, double zr, double zi,
                                            double4 *tiles, Moments &S, int &n_near)
{
    using T = typename StarRec<EQUAL>::T;
    auto masses = [&](Moments &C) {   // the common mass
        if (!EQUAL) return;
#pragma unroll
        for (int j = 0; j < NMOM; ++j) {
            C.r[j] *= B.m0;
            C.i[j] *= B.m0;
        }
        C.q *= B.m0;
    };
    if (!FMM && __popcll(mask) > SPARSE_MAX) {
        zero(S);
        stream_tiles_grouped(B.stars, B.n_stars, reinterpret_cast<T *>(tiles),
                             [&](auto g, const T *r) {
                                 add_moments_group<EQUAL, decltype(g)::value>(S, zr, zi, r);
                             });
        masses(S);
        return;
    }
    if constexpr (FMM) {
        const FmmArgs &M = A.fmm[B.r];
        const double fx = floor((zr - M.x0) / M.w), fy = floor((zi - M.y0) / M.w);
        const bool in = fx >= 0.0 && fy >= 0.0 && fx < (double)M.G && fy < (double)M.G;
        zero(S);
        n_near = B.n_stars;
        if (in) {
            const int ix = (int)fx, iy = (int)fy, cell = iy * M.G + ix;
            set_moments_far(S, M, cell, (zr - (M.x0 + (ix + 0.5) * M.w)) * M.inv_w,
                            (zi - (M.y0 + (iy + 0.5) * M.w)) * M.inv_w);
            n_near = fmm_near(M, cell, [&](const double4 &s4) {
                if constexpr (EQUAL) add_moments_star<EQUAL>(S, zr, zi, make_double2(s4.x, s4.y));
                else add_moments_star<EQUAL>(S, zr, zi, s4);
            });
            masses(S);
        }
        mask &= __ballot(!in);
    }
    while (mask) {
        const int l = __ffsll((long long)mask) - 1;
        mask &= mask - 1;
        const double xk = __shfl(zr, l, 64), yk = __shfl(zi, l, 64);
        Moments C;
        zero(C);
        int i = B.lane;
        for (int t = B.n_stars >> 8; t; --t, i += 256) {   // four loads in flight
            const T r[4] = {B.stars[i], B.stars[i + 64], B.stars[i + 128], B.stars[i + 192]};
            add_moments_group<EQUAL, 4>(C, xk, yk, r);
        }
        for (; i < B.n_stars; i += 64) add_moments_star<EQUAL>(C, xk, yk, B.stars[i]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) C.u2 = fmax(C.u2, __shfl_xor(C.u2, off, 64));
        spread_sums(C, B.lane);
        masses(C);
        if (B.lane == l) S = C;
    }
}

// Square of the distance from its centre to which an expansion serves.
__device__ __forceinline__ double moments_reach2(const Moments &S)
{
    // M x^(M-1) q / u2 < EXP_TAIL, x = |z - z0| u, less a share for 1/(1 - x)^2
    const float c = (float)(EXP_TAIL / NMOM * S.u2 / S.q);
    const float x = 0.95f * exp2f(log2f(c) * (1.0f / (NMOM - 1)));
    const float xm = fminf(x, 0.25f);
    const double r2 = (double)(xm * xm) / S.u2;
    return r2 > 0.0 ? r2 : 0.0;   // also an expansion that is not finite
}

// A block's share of its polished row's sums sum r and sum r^2 (row
// identities), and of what bounds their error: the roots' own estimated errors,
// and sum |r|, sum |r|^2 for the rounding of the sums.
template <class T>
__device__ __forceinline__ void put_row_sums(const RoundArgs<T> &A, const BlockCtx<T> &B,
                                             double zr, double zi, double er)
{
    const bool valid = B.valid;
    double s1r = valid ? zr : 0.0, s1i = valid ? zi : 0.0;
    double s2r = valid ? zr * zr - zi * zi : 0.0, s2i = valid ? 2.0 * zr * zi : 0.0;
    const double ab2 = valid ? zr * zr + zi * zi : 0.0, ab = sqrt(ab2);
    const double ev = valid ? er : 0.0;
    double t_e = ev, t_e2 = ev * (2.0 * ab + ev), t_a = ab, t_a2 = ab2;
    wave_sum(s1r); wave_sum(s1i); wave_sum(s2r); wave_sum(s2i);
    wave_sum(t_e); wave_sum(t_e2); wave_sum(t_a); wave_sum(t_a2);
    if (B.lane == 0) {
        A.vieta[2 * B.vslot] = make_double4(s1r, s1i, s2r, s2i);
        A.vieta[2 * B.vslot + 1] = make_double4(t_e, t_e2, t_a, t_a2);
    }
}

// Work of the expansion kernel, added to the striped tallies from FMM_T_EXP on:
// near stars (multipole sums), steps on expansions, expansions formed, and
// those weighted by their fields' star counts.
enum { EXP_NEAR = 0, EXP_STEPS_DONE = 1, EXP_FORMED = 2, EXP_STARS = 3 };

// Rows of a parked front by expansions, one block of 64 roots a work group:
// each root starts a row from the extrapolation of its chain and steps on its
// expansion, which is formed anew about that start once it lies too far from
// the last centre.  Nothing couples the block's roots to other blocks, so it
// goes on through its front's rows by itself, from where it stopped last; a
// row counts when every root of the block is accepted in it.  At the first row
// that leaves a root open the block is stuck: the accepted roots of that row are
// stored, and the row's passes step the others once every other block has come
// to it (expand_control).  In FP64 only the roots left open wait; the others go
// on, each with its own next row, so that what is left to do after the passes
// is one root's rows and not a block's.  In the mixed form the block waits.
//
// A kernel of its own at two waves per SIMD, so that the moments stay in
// registers.  Whole calls, with one sum over the stars per row and with this:
// N = 6,000 FP64 547 -> 101 ms, N = 1,000 27.4 -> 12.9, N = 4,099 mixed 184 ->
// 55, rectangular N = 437 10.5 -> 5.6, N = 3,000 FP64 with multipole sums 28.4 ->
// 22.7, N = 10,000 mixed with them 150 -> 70, 40 fields mixed 130 -> 64 ms (with
// fewer pieces of the phase grid and their nearer starts as well 45, 6.4, 27,
// 4.8, 12.6, 54 and 54).  A single root's expansion takes four stars a lane at a
// time, so that their loads are in flight together (58.8 -> 55.4 ms at N = 6,000),
// and its sums are spread over the lanes in halves (7.8 -> 7.1 at N = 1,000, 57 ->
// 54 for the 40 fields).  Letting the accepted roots of a stuck block go on by
// themselves in FP64 took the call at N = 6,000 from 55.4 to 45.2 ms and at
// N = 1,000 from 7.1 to 6.4.  What bounds the kernel now is its last blocks: those
// whose roots pass close to a star or a critical point form an expansion
// every few steps, one after another.  Splitting the stars over 2 or 4
// waves did not help them (61 and 89 ms at N = 6,000 against 58.8), nor did
// keeping the nearest star out of the expansion (56.3 against 55.4; N = 10,000 with
// multipole sums 60 against 54).
// Errors against 80-bit roots of 8 fields of 10 to 3,000 stars: FP64 as before
// (rms 2e-16 to 2.7e-15), mixed rms 2e-16 to 8e-15 against 2e-14 to
// 2e-13.
template <bool EQUAL, bool FMM, bool POLISH>   // POLISH: the mixed form
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MLCC_EXPAND_WAVES, 8)))
expand_rows(RoundArgs<typename StarRec<EQUAL>::T> A)
{
    __shared__ typename StarRec<EQUAL>::T star_tiles[128];
    double4 *tiles = reinterpret_cast<double4 *>(star_tiles);
    const int2 fq = A.bmap[blockIdx.x];
    const Front *F = A.fronts + fq.x;
    if (F->state != FRONT_PARKED) return;
    BlockCtx<typename StarRec<EQUAL>::T> B;
    enter_fq(A, F, fq.x, fq.y, (int32_t *)nullptr, (int32_t *)nullptr, B);
    constexpr bool polish = POLISH;
    const int front_row = F->row;
    if (B.settled) B.row += B.dir;   // the passes finished this one
    if (!F->redo) {   // on from where the block stopped, or past the row passes finished since
        const int next = A.next_row[B.vslot];
        if ((next - B.row) * B.dir > 0) B.row = next;
    }
    const int k = B.k, n_r = B.n_r;
    const int hist0 = B.hist - front_row * B.dir;   // finished rows behind row j: hist0 + j dir
    const int64_t base_f = B.base_f;
    const bool valid = B.valid;
    // FP64: the root's own next row; blocks of the mixed form stay in step
    int root_row = B.row;
    if (valid && !polish && !F->redo) {
        const int next = A.root_row[base_f + k];
        if ((next - root_row) * B.dir > 0) root_row = next;
    }
    bool goes_on = valid, loaded = false;   // false: left open in a row of this launch
    int stuck_row = 0;
    double2 z1 = make_double2(0.0, 0.0), z2 = z1, z3 = z1;
    Moments Mo;
    zero(Mo);
    double cr = 0.0, ci = 0.0, reach2 = -1.0;   // centre of the expansion, and its reach
    unsigned long long t_steps = 0, t_exp = 0, t_near = 0;   // per lane
    bool is_stuck = false;
    for (; (B.row - B.end_row) * B.dir <= 0; B.row += B.dir) {
        if (!__ballot(goes_on && (root_row - B.end_row) * B.dir <= 0)) break;
        const bool mine = goes_on && root_row == B.row;
        if (mine && !loaded) {
            const int hist = hist0 + B.row * B.dir;
            const int64_t d = (int64_t)B.dir * n_r, o1 = B.out_off + (int64_t)B.row * n_r + k - d;
            z1 = make_double2(A.out_re[o1], A.out_im[o1]);
            if (hist >= 2) z2 = make_double2(A.out_re[o1 - d], A.out_im[o1 - d]);
            if (hist >= 3) z3 = make_double2(A.out_re[o1 - 2 * d], A.out_im[o1 - 2 * d]);
            reach2 = -1.0;
            loaded = true;
        }
        B.boundary = B.has_bnd && B.row == B.end_row;
        const double2 un = A.unit[B.row];
        const double2 e = make_double2(B.a * un.x, B.a * un.y);
        const int pred = min(A.predictor, min(hist0 + B.row * B.dir, 3) - 1);
        double pr = z1.x, pi = z1.y;
        if (pred == 1) {
            pr = 2.0 * z1.x - z2.x;
            pi = 2.0 * z1.y - z2.y;
        } else if (pred == 2) {
            pr = fma(3.0, z1.x - z2.x, z3.x);
            pi = fma(3.0, z1.y - z2.y, z3.y);
        }
        bool going = mine, left = mine;   // left: not accepted in this row
        double xr = pr, xi = pi, err = 0.0;
        Update u{};
        for (int it = 0; it < EXP_STEPS; ++it) {
            if (!__ballot(going)) break;
            // lanes out of reach of their expansion form a new one, ahead of them by
            // most of the last one's reach along their chain, so that it serves
            // from one edge to the other; at their own place if that is still
            // too far
            for (int ahead = it == 0; ahead >= 0; --ahead) {
                const double ox = xr - cr, oy = xi - ci;
                const bool out = going && !(ox * ox + oy * oy <= reach2);
                const unsigned long long mask = __ballot(out);
                if (!mask) break;
                const bool fresh = FMM || __popcll(mask) > SPARSE_MAX ? mine : out;
                const double vx = pr - z1.x, vy = pi - z1.y, v2 = vx * vx + vy * vy;
                const double lead =
                    ahead && reach2 > 0.0 && v2 > 0.0 ? EXP_LEAD * sqrt(reach2 / v2) : 0.0;
                const double tx = fma(lead, vx, xr), ty = fma(lead, vy, xi);
                int near = 0;
                sum_moments<EQUAL, FMM>(A, B, __ballot(fresh), tx, ty, tiles, Mo, near);
                if (fresh) {
                    if (B.n_poly > 0)
                        add_moments_sheet(Mo, B.sheet + B.n_poly, B.n_poly, B.sheet_c, tx, ty);
                    cr = tx;
                    ci = ty;
                    reach2 = moments_reach2(Mo);
                    t_exp += out;   // those formed along with them are not counted
                    t_near += out ? near : 0;
                }
            }
            // f, f', f''/2 and f'''/6 in h = z0 - z by Horner's rule
            const double hr = cr - xr, hi = ci - xi;
            double g0r = 0, g0i = 0, g1r = 0, g1i = 0, g2r = 0, g2i = 0, g3r = 0, g3i = 0;
#pragma unroll
            for (int j = NMOM - 1; j >= 0; --j) {
                double nr, ni;
                nr = fma(g3r, hr, fma(-g3i, hi, g2r)); ni = fma(g3r, hi, fma(g3i, hr, g2i));
                g3r = nr; g3i = ni;
                nr = fma(g2r, hr, fma(-g2i, hi, g1r)); ni = fma(g2r, hi, fma(g2i, hr, g1i));
                g2r = nr; g2i = ni;
                nr = fma(g1r, hr, fma(-g1i, hi, g0r)); ni = fma(g1r, hi, fma(g1i, hr, g0i));
                g1r = nr; g1i = ni;
                nr = fma(g0r, hr, fma(-g0i, hi, Mo.r[j])); ni = fma(g0r, hi, fma(g0i, hr, Mo.i[j]));
                g0r = nr; g0i = ni;
            }
            Sums S;
            zero(S);
            S.s0r = g0r; S.s0i = g0i; S.s2r = g1r; S.s2i = g1i; S.s3r = g2r; S.s3i = g2i;
            FieldAt Q;
            Q.Fr = B.gamma + g1r - e.x;
            Q.Fi = g1i - e.y;
            Q.Fpr = -2.0 * g2r;
            Q.Fpi = -2.0 * g2i;
            // G = -F''/(2 F') with F'' = 6 sum m u^4
            const double2 G = cdiv(make_double2(1.5 * g3r, 1.5 * g3i), make_double2(g2r, g2i));
            // far from its zero a root of the mixed form takes Newton's step, as
            // the polish would
            const double2 n = cdiv(make_double2(Q.Fr, Q.Fi), make_double2(Q.Fpr, Q.Fpi));
            const double g2 = G.x * G.x + G.y * G.y;
            const bool basin = (n.x * n.x + n.y * n.y) * g2 < EXP_BASIN * EXP_BASIN;
            const bool corr = basin || !polish;
            const Update v = take_step(S, Q, corr ? G.x : 0.0, corr ? G.y : 0.0, xr, xi, B.gamma, B.a,
                                       B.a1, A.tol_step2, A.tol_mu, k, nullptr, 0);
            const double sr = xr - v.zr, si = xi - v.zi, d2 = sr * sr + si * si;
            if (going) {
                t_steps += 1;
                going = basin || polish;
                if (basin && v.flag && (d2 * g2) * (d2 * g2) * d2 < EXP_ERR * EXP_ERR) {
                    u = v;
                    err = sqrt(g2) * d2;
                    left = false;
                    going = false;
                }
                xr = v.zr;
                xi = v.zi;
            }
        }
        if (mine && !left) put(A, B, k, u);
        if (!is_stuck && __ballot(left)) {   // the block's first row with an open root
            is_stuck = true;
            stuck_row = B.row;
            if (valid) {
                const int64_t i = base_f + k;
                A.flagrow[i] = left ? -1 : 4 * B.row;
                if (polish) A.errbuf[i] = err;
            }
            if (polish) break;
        }
        if (left) goes_on = false;
        if (mine && !left) {
            root_row += B.dir;
            z3 = z2;
            z2 = z1;
            z1 = make_double2(u.zr, u.zi);
        }
    }
    if (valid && !polish) A.root_row[base_f + k] = root_row;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        t_steps += __shfl_xor(t_steps, off, 64);
        t_exp += __shfl_xor(t_exp, off, 64);
        t_near += __shfl_xor(t_near, off, 64);
    }
    if (B.lane == 0) {
        A.next_row[B.vslot] = is_stuck ? stuck_row : polish ? B.row : B.end_row + B.dir;
        A.stuck[B.vslot] = is_stuck;
        unsigned long long *s = A.fmm_tally + (blockIdx.x % FMM_STRIPES) * FMM_STRIPE_U64 + FMM_T_EXP;
        if (t_steps) atomicAdd(&s[EXP_STEPS_DONE], t_steps);
        if (t_exp) {
            atomicAdd(&s[EXP_FORMED], t_exp);
            atomicAdd(&s[EXP_STARS], t_exp * (unsigned long long)B.n_stars);
        }
        if (t_near) atomicAdd(&s[EXP_NEAR], t_near);
    }
}

// One FP64 Aberth pass of a block (the block context is set by enter()).
// `tiles` holds two tiles of up to 32-byte records.
template <bool EQUAL, bool FMM>
__device__ __forceinline__ void sweep_f64_pass(const RoundArgs<typename StarRec<EQUAL>::T> &A,
                                               const BlockCtx<typename StarRec<EQUAL>::T> &B,
                                               double4 *tiles)
{
    using T = typename StarRec<EQUAL>::T;
    if (B.reseed) {
        // restart the row from its start values: the seeds z_i +- 1 for a
        // cold start, the previous row of the subchain otherwise.  The second
        // set for a stalled cold start: z_i +- i, and the extra roots of a
        // rectangular sheet turned by half their spacing.
        const bool second = B.second;
        if (B.valid) {
            double2 z;
            if (B.dir == 0 && B.k >= 2 * B.n_stars) {   // a rectangular sheet's extra root
                const int x = B.k - 2 * B.n_stars;
                z = make_double2(B.sheet[2 * B.n_poly + 2 * x], B.sheet[2 * B.n_poly + 2 * x + 1]);
                if (second) {
                    double sn, cs;
                    sincos(M_PI / (double)B.n_extra, &sn, &cs);
                    z = make_double2(z.x * cs - z.y * sn, z.x * sn + z.y * cs);
                }
            } else if (B.dir == 0) {
                const T st = B.stars[B.k >> 1];
                const double o = (B.k & 1) ? -1.0 : 1.0;
                z = second ? make_double2(st.x, st.y + o) : make_double2(st.x + o, st.y);
            } else {
                const int64_t o = B.out_off + (int64_t)(B.row - B.dir) * B.n_r + B.k;
                z = make_double2(A.out_re[o], A.out_im[o]);
            }
            B.nxt[B.base_f + B.k] = z;
        }
        const int n_valid = __popcll(__ballot(B.valid));
        if (B.lane == 0) atomicAdd(B.count, n_valid);
        return;
    }
    const int lane = B.lane, k0 = B.k0, k = B.k, n_r = B.n_r, n_stars = B.n_stars;
    const bool valid = B.valid;
    const int64_t base_f = B.base_f;
    const double2 *__restrict__ zsrc = B.zsrc;
    const T *__restrict__ stars = B.stars;
    double2 *__restrict__ nxt = B.nxt;
    int32_t *__restrict__ flagrow = A.flagrow;
    const double m0 = B.m0, gamma = B.gamma, a = B.a, a1 = B.a1;
    const double tol_step2 = A.tol_step2, tol_mu = A.tol_mu;
    double zr = 0.0, zi = 0.0;
    bool act = false;
    if (valid) {
        const double2 z = zsrc[k];
        zr = z.x;
        zi = z.y;
        act = flagrow[base_f + k] != B.stamp;
        if (!act && B.fresh) {   // accepted by the expansions
            const double2 w = accepted_root(A, B, k);
            zr = w.x;
            zi = w.y;
        } else if (B.pred) {
            predict(A, B, k, zr, zi);
        }
        if (!act) nxt[base_f + k] = make_double2(zr, zi);   // carried forward
    }
    const unsigned long long amask = __ballot(act);
    const int n_act = __popcll(amask);
    if (n_act == 0) return;

    const double2 e = B.e;
    auto store = [&](int kk, const Update &u) {
        nxt[base_f + kk] = make_double2(u.zr, u.zi);
        if (!u.flag) return;
        flagrow[base_f + kk] = B.stamp;
        put(A, B, kk, u);
    };

    int n_after = 0;
    if (n_act <= SPARSE_MAX) {
        // Few roots left (a straggler sweep): the wave takes them one at a
        // time, lanes splitting the star and root sums, then a butterfly
        // reduction.  Latency per root drops ~64x against one lane doing it.
        unsigned long long mm = amask;
        while (mm) {
            const int l = __ffsll((long long)mm) - 1;
            mm &= mm - 1;
            const double xk = __shfl(zr, l, 64), yk = __shfl(zi, l, 64);
            Sums S;
            zero(S);
            each_strided(stars, n_stars, lane,
                         [&](int, const T &st) { add_star<EQUAL>(S, xk, yk, st); });
            const int kk = k0 + l;
            each_strided(zsrc, n_r, lane, [&](int j, const double2 &o) {
                if (j != kk) add_root(S, xk, yk, o);
            });
            wave_sum(S.s1r); wave_sum(S.s1i);
            if (!EQUAL) { wave_sum(S.s0r); wave_sum(S.s0i); }
            wave_sum(S.s2r); wave_sum(S.s2i);
            wave_sum(S.s3r); wave_sum(S.s3i);
            wave_sum(S.Rr); wave_sum(S.Ri);
            const Update u = finish<EQUAL>(S, xk, yk, m0, e, gamma, a, a1, tol_step2, tol_mu, kk,
                                           B.sheet, B.n_poly);
            if (lane == l) store(kk, u);
            n_after += u.flag ? 0 : 1;
        }
    } else {
        Sums S;
        zero(S);
        if constexpr (FMM) {
            int cell;
            double2 f, f1, f2, g;
            double q;
            fmm_far(A.fmm[B.r], zr, zi, cell, f, f1, f2, g, q, true);
            const int n_near = fmm_near(A.fmm[B.r], cell, [&](const double4 &s4) {
                if constexpr (EQUAL) add_star<EQUAL>(S, zr, zi, make_double2(s4.x, s4.y));
                else add_star<EQUAL>(S, zr, zi, s4);
            });
            FmmTally tl;
            fmm_count(tl, act, n_near, n_stars);
            fmm_flush(A.fmm_tally, FMM_T_F64, tl);
            // far terms in the accumulators' conventions (s2i holds -Im/2)
            S.s1r += g.x; S.s1i += g.y;
            if (!EQUAL) { S.s0r += f.x; S.s0i += f.y; }
            S.s2r -= f1.x; S.s2i += 0.5 * f1.y;
            S.s3r += 0.5 * f2.x; S.s3i += 0.5 * f2.y;
        } else {
            stream_tiles_grouped(stars, n_stars, reinterpret_cast<T *>(tiles),
                                 [&](auto g, const T *r) {
                                     add_star_group<EQUAL, decltype(g)::value>(S, zr, zi, r);
                                 });
        }
        if (!B.fast) {
            // the other roots in FP64, in groups outside the own block;
            // within it one at a time, skipping the root itself
            double2 *rtiles = reinterpret_cast<double2 *>(tiles);
            auto group = [&](auto g, const double2 *r) {
                add_root_group<decltype(g)::value>(S, zr, zi, r);
            };
            const int own_hi = min(k0 + 64, n_r);
            stream_tiles_grouped(zsrc, k0, rtiles, group);
            stream_tiles(zsrc + k0, own_hi - k0, rtiles, [&](int j, const double2 &o) {
                Sums T2 = S;
                add_root(T2, zr, zi, o);
                const bool self = j == lane;
                S.Rr = self ? S.Rr : T2.Rr;
                S.Ri = self ? S.Ri : T2.Ri;
            });
            stream_tiles_grouped(zsrc + own_hi, n_r - own_hi, rtiles, group);
        } else {
            // root-root sum in FP32 (add_root_hl), summed per tile and carried
            // across tiles in FP64
            float4 *rtiles = reinterpret_cast<float4 *>(tiles);
            const float4 zs = SplitRoot{}(make_double2(zr, zi));
            float pr = 0.f, pi = 0.f;
            auto other = [&](int, const float4 &o) { add_root_hl(pr, pi, zs, o); };
            auto carry = [&]() {
                S.Rr += (double)pr;
                S.Ri += (double)pi;
                pr = pi = 0.f;
            };
            const int own_hi = min(k0 + 64, n_r);
            stream_tiles_ex(zsrc, k0, rtiles, SplitRoot{}, other, carry);
            stream_tiles_ex(zsrc + k0, own_hi - k0, rtiles, SplitRoot{},
                            [&](int j, const float4 &o) {
                                float tr = pr, ti = pi;
                                add_root_hl(tr, ti, zs, o);
                                const bool self = j == lane;
                                pr = self ? pr : tr;
                                pi = self ? pi : ti;
                            }, carry);
            stream_tiles_ex(zsrc + own_hi, n_r - own_hi, rtiles, SplitRoot{}, other, carry);
        }
        const Update u = finish<EQUAL>(S, zr, zi, m0, e, gamma, a, a1, tol_step2, tol_mu, k,
                                       B.sheet, B.n_poly);
        if (act) store(k, u);
        n_after = __popcll(__ballot(act && !u.flag));
    }
    if (lane == 0) {
        if (n_after) atomicAdd(B.count, n_after);
        atomicAdd(B.upd, n_act);
    }
}

template <bool EQUAL, bool FMM>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MLCC_SWEEP_WAVES, 8)))
aberth_sweep_f64(RoundArgs<typename StarRec<EQUAL>::T> A)
{
    __shared__ double4 tiles[128];
    BlockCtx<typename StarRec<EQUAL>::T> B;
    if (!enter(A, PH_F64, B)) return;
    sweep_f64_pass<EQUAL, FMM>(A, B, tiles);
}

// ---------------------------------------------------------------------------
// FP32 Aberth sweep (mixed mode: cold starts, rows without a prediction, and
// rows the polish did not settle)
// ---------------------------------------------------------------------------

// Steps shorter than this (theta_E units) are below what the FP32 sums
// resolve reliably; the FP64 polish takes over from there.
constexpr double TOL_F32 = 1e-6;

// One Aberth step for every root of the row with the sums in FP32.  The
// distance to each star is formed in FP64 and rounded, so no precision is
// lost to the size of the coordinates; each 64-star tile is summed in FP32
// and the tile sums are carried in FP64, which keeps the large near-star
// terms from swamping the accumulation.  The other roots enter in FP32
// coordinates (they only steer the step).  The step itself and the new
// iterate are FP64.
template <bool EQUAL, bool FMM>
__device__ __forceinline__ void sweep_f32_pass(const RoundArgs<typename StarRec<EQUAL>::T> &A,
                                               const BlockCtx<typename StarRec<EQUAL>::T> &B,
                                               double4 *tiles)
{
    using T = typename StarRec<EQUAL>::T;
    const int lane = B.lane, k0 = B.k0, k = B.k, n_r = B.n_r, n_stars = B.n_stars;
    const bool valid = B.valid;
    const int64_t base_f = B.base_f;
    const double2 *__restrict__ zsrc = B.zsrc;
    const T *__restrict__ stars = B.stars;
    const double m0 = B.m0, gamma = B.gamma;
    double zr = 0.0, zi = 0.0;
    if (valid) {
        const double2 z = zsrc[k];
        zr = z.x;
        zi = z.y;
        if (B.pred) predict(A, B, k, zr, zi);
    }
    // star sums: FP32 within a tile, FP64 across tiles (with multipole
    // sums: the near stars' terms and the cell's series, in FP64)
    double S1r = 0, S1i = 0, S2r = 0, S2i = 0, S3r = 0, S3i = 0;
    float p1r = 0, p1i = 0, p2r = 0, p2i = 0, p3r = 0, p3i = 0;
    if constexpr (FMM) {
        Sums S;
        zero(S);
        int cell;
        double2 f, f1, f2, g;
        double q;
        fmm_far(A.fmm[B.r], zr, zi, cell, f, f1, f2, g, q, true);
        const int n_near = fmm_near(A.fmm[B.r], cell, [&](const double4 &s4) {
            if constexpr (EQUAL) add_star<EQUAL>(S, zr, zi, make_double2(s4.x, s4.y));
            else add_star<EQUAL>(S, zr, zi, s4);
        });
        FmmTally tl;
        fmm_count(tl, valid, n_near, n_stars);
        fmm_flush(A.fmm_tally, FMM_T_F32, tl);
        S1r = S.s1r + g.x; S1i = S.s1i + g.y;
        S2r = S.s2r - f1.x; S2i = S.s2i + 0.5 * f1.y;
        S3r = S.s3r + 0.5 * f2.x; S3i = S.s3i + 0.5 * f2.y;
    } else {
        stream_tiles_ex(
            stars, n_stars, reinterpret_cast<T *>(tiles), Same{},
            [&](int, const T &s) {
                const float dx = (float)(zr - s.x), dy = (float)(zi - s.y);
                const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, dy * dy));
                // a = ux^2, b = uy^2: p2i accumulates sum m ux uy (Im u^2 =
                // -2 ux uy), and since a + b = inv, a - 3b = inv - 4b and
                // b - 3a = inv - 4a
                const float ux = dx * inv, uy = dy * inv;
                const float a = ux * ux, b = uy * uy;
                p1r += ux;
                p1i -= uy;
                if (EQUAL) {
                    p2r += a - b;
                    p2i = fmaf(ux, uy, p2i);
                    p3r = fmaf(ux, fmaf(-4.0f, b, inv), p3r);
                    p3i = fmaf(uy, fmaf(-4.0f, a, inv), p3i);
                } else {
                    const float mi = (float)StarRec<EQUAL>::mass(s);
                    const float mux = mi * ux, muy = mi * uy;
                    p2r = fmaf(mi, a - b, p2r);
                    p2i = fmaf(mux, uy, p2i);
                    p3r = fmaf(mux, fmaf(-4.0f, b, inv), p3r);
                    p3i = fmaf(muy, fmaf(-4.0f, a, inv), p3i);
                }
            },
            [&]() {
                S1r += p1r; S1i += p1i; S2r += p2r; S2i += p2i; S3r += p3r; S3i += p3i;
                p1r = p1i = p2r = p2i = p3r = p3i = 0.f;
            });
    }
    // root-root sum in FP32 coordinates
    const float zr32 = (float)zr, zi32 = (float)zi;
    double Rr = 0, Ri = 0;
    float qr = 0, qi = 0;
    float2 *rt = reinterpret_cast<float2 *>(tiles);
    auto to32 = [](const double2 &o) { return make_float2((float)o.x, (float)o.y); };
    auto flush = [&]() { Rr += qr; Ri += qi; qr = qi = 0.f; };
    auto other = [&](int, const float2 &o) {
        const float dx = zr32 - o.x, dy = zi32 - o.y;
        const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, dy * dy));
        qr = fmaf(dx, inv, qr);
        qi = fmaf(-dy, inv, qi);
    };
    const int own_hi = min(k0 + 64, n_r);
    stream_tiles_ex(zsrc, k0, rt, to32, other, flush);
    stream_tiles_ex(zsrc + k0, own_hi - k0, rt, to32,
                    [&](int j, const float2 &o) {
                        const float dx = zr32 - o.x, dy = zi32 - o.y;
                        const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, dy * dy));
                        const bool self = j == lane;
                        qr = self ? qr : fmaf(dx, inv, qr);
                        qi = self ? qi : fmaf(-dy, inv, qi);
                    },
                    flush);
    stream_tiles_ex(zsrc + own_hi, n_r - own_hi, rt, to32, other, flush);

    S2i *= -2.0;
    if (EQUAL) {
        S2r *= m0; S2i *= m0; S3r *= m0; S3i *= m0;
    }
    const double2 e = B.e;
    const double Fr = gamma + S2r - e.x, Fi = S2i - e.y;
    const double Fpr = -2.0 * S3r, Fpi = -2.0 * S3i;
    const double Gr = 2.0 * S1r - Rr, Gi = 2.0 * S1i - Ri;
    const double Dr = Fpr + (Fr * Gr - Fi * Gi);
    const double Di = Fpi + (Fr * Gi + Fi * Gr);
    const double den = Dr * Dr + Di * Di;
    Update u;
    u.zr = zr - (Fr * Dr + Fi * Di) / den;
    u.zi = zi - (Fi * Dr - Fr * Di) / den;
    if (!isfinite(u.zr) || !isfinite(u.zi)) nudge(u, zr, zi, k);
    if (valid) B.nxt[base_f + k] = make_double2(u.zr, u.zi);
    const int n_valid = __popcll(__ballot(valid));
    // roots that moved by more than the FP32 sweep can resolve are still
    // on their way (the control kernel uses this for cold starts)
    const double mr = u.zr - zr, mi = u.zi - zi;
    const int n_moving = __popcll(__ballot(valid && !(mr * mr + mi * mi <= TOL_F32 * TOL_F32)));
    if (lane == 0) {
        if (n_moving) atomicAdd(B.count, n_moving);
        atomicAdd(B.upd, n_valid);
    }
}

template <bool EQUAL, bool FMM>
__global__ void __launch_bounds__(64)
aberth_sweep_f32(RoundArgs<typename StarRec<EQUAL>::T> A)
{
    __shared__ double4 tiles[128];
    BlockCtx<typename StarRec<EQUAL>::T> B;
    if (!enter(A, PH_F32, B)) return;
    sweep_f32_pass<EQUAL, FMM>(A, B, tiles);
}

// ---------------------------------------------------------------------------
// FP64 Newton polish (mixed mode)
// ---------------------------------------------------------------------------

// Newton step z' = z - D, D = F/F', accepted on the paper's cutoffs for the
// step just taken (|D| < tol_step, or the App. C bound on |1/mu| at z), or
// when the error it leaves, at most ~|F''| |D|^2 / (2 |F'|) by quadratic
// convergence, is below POLISH_ERR_FRACTION * tol_step -- always while
// |D| |F''/F'| < 0.1 on the bound |F''| <= 6 q, so that z' lies well inside
// the region where Newton's method converges to one root.  The error bound
// is recorded for the row identities.  The caustic of z' reuses
// the sums: sum m/(z' - z_i) = s0 + D s2 + D^2 s3 + O(D^3 sum m |u|^4).
constexpr double POLISH_ERR_FRACTION = 1e-3;

template <bool EQUAL>
__device__ __forceinline__ Update polish_finish(PSums S, double zr, double zi, double m0,
                                                double2 e, double gamma, double a, double a1,
                                                double tol_step2, double tol_mu, int k)
{
    S.s2i *= -2.0;
    if (EQUAL) {
        S.s0r *= m0; S.s0i *= m0; S.s2r *= m0; S.s2i *= m0;
        S.s3r *= m0; S.s3i *= m0; S.q *= m0;
    }
    const double Fr = gamma + S.s2r - e.x, Fi = S.s2i - e.y;
    const double Fpr = -2.0 * S.s3r, Fpi = -2.0 * S.s3i;
    const double den = Fpr * Fpr + Fpi * Fpi;
    const double Dr = (Fr * Fpr + Fi * Fpi) / den;
    const double Di = (Fi * Fpr - Fr * Fpi) / den;
    Update u;
    u.zr = zr - Dr;
    u.zi = zi - Di;
    const double aD2 = Dr * Dr + Di * Di, aD = sqrt(aD2);
    const double ratio = 6.0 * S.q / sqrt(den);   // bound on |F''/F'|
    const double aF = sqrt(Fr * Fr + Fi * Fi);
    u.err = 0.5 * ratio * aD2;
    u.flag = (aD2 < tol_step2 || aF * (aF + 2.0 * a1) < tol_mu ||
              u.err * u.err < POLISH_ERR_FRACTION * POLISH_ERR_FRACTION * tol_step2) &&
             aD * ratio < 0.1;
    if (!isfinite(u.zr) || !isfinite(u.zi)) nudge(u, zr, zi, k);
    const double d2r = Dr * Dr - Di * Di, d2i = 2.0 * Dr * Di;
    const double Tr = S.s0r + (Dr * S.s2r - Di * S.s2i) + (d2r * S.s3r - d2i * S.s3i);
    const double Ti = S.s0i + (Dr * S.s2i + Di * S.s2r) + (d2r * S.s3i + d2i * S.s3r);
    u.wr = fma(a, u.zr, gamma * u.zr) - Tr;
    u.wi = fma(a, u.zi, -gamma * u.zi) + Ti;
    return u;
}

// A Newton step needs only its own root's sums, so a root the acceptance test
// turns down takes its next step in the same pass (up to POLISH_STEPS),
// instead of waiting for the whole front's next pass.
template <bool EQUAL, bool FMM>
__device__ __forceinline__ void polish_pass(const RoundArgs<typename StarRec<EQUAL>::T> &A,
                                            const BlockCtx<typename StarRec<EQUAL>::T> &B,
                                            double4 *tiles)
{
    const int lane = B.lane, k = B.k;
    const bool valid = B.valid;
    const int64_t base_f = B.base_f;
    double zr = 0.0, zi = 0.0;   // the root's value: start of the row, then its end
    bool act = false;
    double er = 0.0;   // estimated error of that value
    if (valid) {
        const double2 z = B.zsrc[k];
        zr = z.x;
        zi = z.y;
        act = A.flagrow[base_f + k] != B.stamp;
        if (!act && B.fresh) {   // accepted by the expansions
            const double2 w = accepted_root(A, B, k);
            zr = w.x;
            zi = w.y;
        } else if (B.pred) {
            predict(A, B, k, zr, zi);
        }
        if (!act) er = A.errbuf[base_f + k];   // accepted earlier in this row
    }
    bool open = act;
    Update u{};
    int n_steps = 0, n_near = 0;
    double xr = zr, xi = zi;
    for (int it = 0; it < POLISH_STEPS; ++it) {
        const unsigned long long mask = __ballot(open);
        if (!mask) break;
        PSums S;
        int near;
        newton_sums<EQUAL, FMM>(A, B, mask, xr, xi, tiles, S, near);
        const Update v = polish_finish<EQUAL>(S, xr, xi, B.m0, B.e, B.gamma, B.a, B.a1, A.tol_step2,
                                              A.tol_mu, k);
        if (open) {
            u = v;
            n_steps += 1;
            n_near += near;
            open = !v.flag;
            xr = v.zr;
            xi = v.zi;
        }
    }
    const int n_open = __popcll(__ballot(open));
    const int n_upd = wave_count(n_steps);
    if (act) {
        zr = u.zr;
        zi = u.zi;
        if (u.flag) {
            er = u.err;
            A.errbuf[base_f + k] = u.err;
            A.flagrow[base_f + k] = B.stamp;
            put(A, B, k, u);
        }
    }
    if (valid) B.nxt[base_f + k] = make_double2(zr, zi);
    if (lane == 0) {
        if (n_open) atomicAdd(B.count, n_open);
        if (n_upd) atomicAdd(B.upd, n_upd);
    }
    if constexpr (FMM) {
        FmmTally tl;
        tl.near = (unsigned long long)wave_count(n_near);
        tl.far = (unsigned long long)n_upd;
        tl.far_n = (unsigned long long)n_upd * (unsigned long long)B.n_stars;
        fmm_flush(A.fmm_tally, FMM_T_POLISH, tl);
    }
    put_row_sums(A, B, zr, zi, er);
}

template <bool EQUAL, bool FMM>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MLCC_POLISH_WAVES, 8)))
newton_polish_f64(RoundArgs<typename StarRec<EQUAL>::T> A)
{
    __shared__ double4 tiles[128];
    BlockCtx<typename StarRec<EQUAL>::T> B;
    if (!enter(A, PH_POLISH, B)) return;
    polish_pass<EQUAL, FMM>(A, B, tiles);
}

// ---------------------------------------------------------------------------
// Seeds and front control
// ---------------------------------------------------------------------------

// Cold-start seeds at the centre row of each subchain: root 2i <- z_i + 1,
// root 2i+1 <- z_i - 1 (Sec. 3.2).  One thread per root of every front that
// starts cold (the downward front of each subchain).  The columns take their
// numbers from the first subchain's start alone; with `near_seeds` the others
// start where the star would have its two roots if it stood alone,
// z_i +- sqrt(m_i / (1 - kappa_s)) e^{i phi / 2} (1e-4 to 2 away), which
// settles in fewer sweeps.
template <class T> struct StarMass;
template <> struct StarMass<double2> {
    static __device__ __forceinline__ double get(const double2 &, double m0) { return m0; }
};
template <> struct StarMass<double4> {
    static __device__ __forceinline__ double get(const double4 &z, double) { return z.z; }
};

template <class T>
__global__ void seed_centres(const T *__restrict__ stars, const Real *__restrict__ reals,
                             const Front *__restrict__ fronts, const int2 *__restrict__ bmap,
                             const double *__restrict__ sheet, double2 *__restrict__ iter,
                             int32_t near_seeds, int64_t m_steps)
{
    const int2 fq = bmap[blockIdx.x];
    const Front *F = fronts + fq.x;
    if (F->dir != 0) return;
    const Real *R = reals + F->real;
    const int k = fq.y * 64 + threadIdx.x;
    if (k >= R->n_r) return;
    if (k >= 2 * R->n_stars) {   // a rectangular sheet's extra root (Sec. 3.2: on a circle)
        const double *sx = sheet + R->sheet_off + 2 * R->n_poly + 2 * (k - 2 * R->n_stars);
        iter[F->it_off + k] = make_double2(sx[0], sx[1]);
        return;
    }
    const T z = stars[R->star_off + (k >> 1)];
    const double o = (k & 1) ? -1.0 : 1.0;
    if (F->lo == 0 || !near_seeds) {
        iter[F->it_off + k] = make_double2(z.x + o, z.y);
        return;
    }
    // (z - z_i)^2 = m_i / (a e^{-i phi}): half the angle of a e^{i phi}
    const double m = StarMass<T>::get(z, R->m0);
    const double rad = fmax(fmin(sqrt(m / R->a1), 2.0), 1e-4);
    const double phi = M_PI * (double)F->row / (double)m_steps + (R->a < 0.0 ? 0.5 * M_PI : 0.0);
    double sn, cs;
    sincos(phi, &sn, &cs);
    iter[F->it_off + k] = make_double2(fma(o * rad, cs, z.x), fma(o * rad, sn, z.y));
}

// Row sums of every front in the polish phase: one wave per front adds its
// blocks' partial sums in a fixed order (lanes stride over the blocks, then
// a butterfly), so the control kernel reads eight numbers per front.
__global__ void __launch_bounds__(64)
row_sums(const Front *__restrict__ fronts, const Real *__restrict__ reals,
         const double4 *__restrict__ vieta, double4 *__restrict__ vsum)
{
    const int f = blockIdx.x;
    const Front *F = fronts + f;
    if (F->state != FRONT_ACTIVE || F->phase != PH_POLISH) return;
    const int bpf = (reals[F->real].n_r + 63) / 64;
    double v0 = 0, v1 = 0, v2 = 0, v3 = 0, v4 = 0, v5 = 0, v6 = 0, v7 = 0;
    for (int b = threadIdx.x; b < bpf; b += 64) {
        const double4 t = vieta[2 * (F->blk0 + b)], q = vieta[2 * (F->blk0 + b) + 1];
        v0 += t.x; v1 += t.y; v2 += t.z; v3 += t.w;
        v4 += q.x; v5 += q.y; v6 += q.z; v7 += q.w;
    }
    wave_sum(v0); wave_sum(v1); wave_sum(v2); wave_sum(v3);
    wave_sum(v4); wave_sum(v5); wave_sum(v6); wave_sum(v7);
    if (threadIdx.x == 0) {
        vsum[2 * f] = make_double4(v0, v1, v2, v3);
        vsum[2 * f + 1] = make_double4(v4, v5, v6, v7);
    }
}

constexpr int CONTROL_THREADS = 256;

// Adds a pass's updates to the call's totals, plain and weighted by the
// field's star count.
__device__ __forceinline__ void tally_updates(unsigned long long *upd, unsigned long long *star,
                                              int ph, bool fast, unsigned long long u,
                                              unsigned long long ns)
{
    upd[ph] += u;
    star[ph] += u * ns;
    if (ph == PH_F64 && fast) {
        upd[TALLY_FAST] += u;
        star[TALLY_FAST] += u * ns;
    }
}

constexpr int MAX_FRONTS = 1 << 16;
// Polish passes a row may take before it is retried another way: a root with
// direct sums is given POLISH_STEPS Newton steps in all, one with multipole
// sums as many in each of three passes.
constexpr int MAX_POLISH = 3;
__host__ __device__ constexpr int max_polish_passes(bool fmm) { return fmm ? MAX_POLISH : 1; }
constexpr int F32_STALL = 4;

// Puts a front at the start of its (new) row.  Mixed mode: a row with a
// chain prediction goes straight to the FP64 polish; one without (the two
// rows next to a subchain centre, or predictor 0) starts with an FP32 sweep.
__device__ __forceinline__ void start_row(Front &fr, int predictor, int xfrom)
{
    fr.sweeps = 0;
    fr.passes = 0;
    fr.tried = 0;
    fr.f32 = 0;
    fr.best = 0x7fffffff;
    fr.stall = 0;
    fr.passes_row = 0;
    fr.reseed = 0;
    fr.stamp = 4 * fr.row;
    fr.fresh = 1;
    fr.shared = 0;
    fr.settled = 0;
    if (fr.mode == PH_F64)
        fr.phase = PH_F64;
    else
        fr.phase = (predictor > 0 && fr.hist >= 2) ? PH_POLISH : PH_F32;
    // rows with enough rows behind them wait for the expansion kernel
    if (xfrom > 0 && fr.dir != 0 && fr.hist >= xfrom && fr.phase != PH_F32)
        fr.state = FRONT_PARKED;
}

__device__ __forceinline__ void row_done(Front &fr, int32_t *st, int f, int predictor, int xfrom)
{
    if (fr.row == fr.end_row) {
        fr.state = FRONT_DONE;
        if (st) st[f] = FRONT_DONE;
    } else {
        fr.row += fr.dir;
        fr.hist = min(fr.hist + 1, 3);
        start_row(fr, predictor, xfrom);
        if (st) st[f] = fr.state;
    }
}

// Every root of the current row converged.  A cold start hands the upward
// half of its subchain to its partner front and turns downward itself; a
// warm row moves one row on or finishes at its end row.
__device__ __forceinline__ int row_converged(Front &fr, int f, Front *fronts, int32_t *st,
                                             int f0, int predictor, int xfrom)
{
    if (fr.dir == 0) {
        fr.cold = fr.passes_row;
        const int p = fr.partner;
        const int centre = fr.row;
        Front pr = fronts[p];
        pr.state = FRONT_ACTIVE;
        pr.row = centre + 1;
        pr.dir = 1;
        pr.src = f;    // first pass reads the converged centre row
        pr.hist = 1;   // the centre row
        start_row(pr, predictor, xfrom);
        fronts[p] = pr;
        if (st) st[p - f0] = pr.state;
        fr.dir = -1;
        fr.row = centre - 1;
        fr.hist = 1;
        start_row(fr, predictor, xfrom);
        if (st) st[f - f0] = fr.state;
        return p;
    }
    fr.max_warm = max(fr.max_warm, fr.passes_row);
    if (fr.shared && fr.mode == PH_F64) {   // its identities are checked first (expand_check)
        fr.settled = 1;
        fr.state = FRONT_PARKED;
        if (st) st[f - f0] = fr.state;
    } else {
        row_done(fr, st, f - f0, predictor, xfrom);
    }
    return -1;
}

// The two row identities of a row (see aberth_control) from its row sums rs:
// sum r and sum r^2, then the error terms.
// A sheet -P(z), P = sum_{k=1..n} d_2k z^2k, makes the polynomial
// (c - P) prod (z - z_i)^2 + ..., where the dots stay 2 n + 2 degrees below the
// leading term: sum r stays 2 sum z_i, and sum r^2 is 2 sum z_i^2 plus that of
// the roots of c - P, -2 d_2(n-1) / d_2n, or 2 c / d_2 for n = 1.
__device__ __forceinline__ bool row_identities_hold(const Real &R, double2 u, const double4 *rs)
{
    const int bpf = (R.n_r + 63) / 64;
    const double4 t = rs[0], q = rs[1];
    const double a1r = t.x, a1i = t.y, a2r = t.z, a2i = t.w;
    const double se = q.x, se2 = q.y, sa = q.z, sa2 = q.w;
    const double cr = R.gamma - R.a * u.x, ci = -R.a * u.y;   // c(phi)
    const double cc = cr * cr + ci * ci;
    // M / c, or what takes its place with a sheet
    const bool sheet = R.n_poly > 0;
    const double mcr = sheet ? fma(R.sheet_mc, cr, R.sheet_m) : R.M * cr / cc;
    const double mci = sheet ? R.sheet_mc * ci : -R.M * ci / cc;
    const double e1r = a1r - 2.0 * R.sz_r, e1i = a1i - 2.0 * R.sz_i;
    const double e2r = a2r - (2.0 * R.sz2_r - 2.0 * mcr);
    const double e2i = a2i - (2.0 * R.sz2_i - 2.0 * mci);
    const double u_ro = 1.1102230246251565e-16;
    const double tol1 = 2.0 * se + 2.0 * (12 + bpf) * u_ro * sa + R.tol1;
    const double tol2 = 2.0 * se2 + 2.0 * (13 + bpf) * u_ro * sa2 + R.tol2 +
                        16.0 * u_ro * sqrt(mcr * mcr + mci * mci);
    return sqrt(e1r * e1r + e1i * e1i) <= tol1 && sqrt(e2r * e2r + e2i * e2i) <= tol2;
}

// A row the polish did not settle: once an FP32 sweep of the whole row, then
// FP64 sweeps.  What blocks ahead of the row found is done anew.
__device__ __forceinline__ void retry_row(Front &fr, Control *ctl, bool count)
{
    fr.tried |= TRIED_POLISH;
    fr.redo = 1;
    if (!(fr.tried & TRIED_F32)) {
        fr.phase = PH_F32;
    } else {
        // plain FP64 Aberth sweeps over every root from the row's
        // start values: Newton steps may have sent two columns to
        // one root, which Aberth steps from there would not undo
        fr.stamp += 1;
        fr.reseed = 1;
        fr.phase = PH_F64;
        fr.sweeps = 0;
        if (count) atomicAdd((unsigned long long *)&ctl->rows_fallback, 1ull);
    }
}

// One front after its pass (c = its roots still unconverged, or, after an
// FP32 sweep, still moving; rs = its row sums when the pass was a polish).
// Returns the partner front a finished cold start activated, else -1.
// `st` (the control kernel's LDS copy of the states) may be null.
// (Inlined, so that the record stays in registers: through a call it would be
// reached by flat accesses, in LDS or scratch memory.)
__device__ __forceinline__ int advance_front(Front &fr, int f, int32_t c, const double4 *rs, Front *fronts,
                             int32_t *st, int f0, Control *ctl, const Real *reals,
                             const double2 *unit, int max_cold, int max_warm, int predictor,
                             int max_polish, int xfrom)
{
    int partner = -1;
    fr.npass += 1;
    fr.src = f;
    fr.fresh = 0;
    fr.passes_row += 1;
    if (fr.phase == PH_F32) {
        fr.f32 += 1;
        bool polish = true;
        if (fr.dir == 0) {
            if (c < fr.best) {
                fr.best = c;
                fr.stall = 0;
            } else {
                fr.stall += 1;
            }
            polish = c == 0 || fr.stall >= F32_STALL || fr.f32 >= max_cold;
        }
        if (polish) {
            if (fr.tried & TRIED_POLISH) fr.stamp += 1;   // polish every root again
            fr.tried |= TRIED_F32;
            fr.phase = PH_POLISH;
            fr.passes = 0;
        }
    } else if (fr.phase == PH_POLISH) {
        fr.tried |= TRIED_POLISH;
        bool retry = false;
        if (c == 0) {
            if (row_identities_hold(reals[fr.real], unit[fr.row], rs))
                partner = row_converged(fr, f, fronts, st, f0, predictor, xfrom);
            else
                retry = true;
        } else if (++fr.passes >= max_polish) {
            retry = true;
        }
        if (retry) retry_row(fr, ctl, true);
    } else if (fr.reseed) {
        fr.reseed = 0;   // the restart pass only reloaded the start values
    } else if (c == 0) {
        partner = row_converged(fr, f, fronts, st, f0, predictor, xfrom);
    } else {
        fr.sweeps += 1;
        if (fr.dir == 0 && fr.phase == PH_F64 && fr.seedvar == 0 &&
            fr.sweeps >= reals[fr.real].restart && fr.sweeps < max_cold) {
            // a stalled cold start: once, all over again from other seeds
            fr.seedvar = 1;
            fr.reseed = 1;
            fr.stamp += 1;
            fr.sweeps = 0;
            atomicAdd((unsigned long long *)&ctl->cold_restarts, 1ull);
        } else if (fr.sweeps >= (fr.dir == 0 ? max_cold : max_warm)) {
            fr.state = FRONT_FAILED;
            if (st) st[f - f0] = FRONT_FAILED;
            atomicAdd(&ctl->failed_rows, 1);
            atomicAdd((unsigned long long *)&ctl->unconverged, (unsigned long long)c);
            if (fr.dir == 0) {
                fronts[fr.partner].state = FRONT_FAILED;
                if (st) st[fr.partner - f0] = FRONT_FAILED;
            }
        }
    }
    return partner;
}

// Advances every front after a round (counts[f] = roots of front f still
// unconverged after its pass, or, after an FP32 sweep, still moving).
//   FP64 phase: a converged row moves on (row_converged); a front that
//     reaches its sweep cap stops and is counted as failed (with a partner
//     it can no longer start).
//   FP32 phase (mixed): warm rows take one sweep; a cold start sweeps until
//     no root moves by more than TOL_F32, or that count has not fallen for
//     F32_STALL sweeps, or max_cold; then the polish.
//   Polish phase (mixed): a row whose roots were all accepted and whose sums
//     satisfy the row identities has converged.  Otherwise more polish
//     passes (up to MAX_POLISH); then, once per row, an FP32 sweep of the
//     whole row and the polish again; then the row restarts from its start
//     values (seeds, or the previous row) with plain FP64 Aberth sweeps.
//
// Row identities: the rationalised polynomial has leading coefficient
// c = gamma - (1 - kappa_s) e^{-i phi} and next coefficient -2 c sum z_i, so
// sum r = 2 sum z_i and sum r^2 = 2 sum z_i^2 - 2 M / c (M = sum m_i).  A
// root found twice and one missed shifts them by the distance of the two.
// The test allows the roots' own estimated errors (twice over) plus a
// bound on the rounding of the sums: partial sums of 64 values by a
// butterfly, then (row_sums) lanes striding over the blocks and another
// butterfly, gives at most (12 + blocks) unit roundoffs of sum |r| (one
// more for sum |r|^2, whose terms round too).
//
// `st` keeps the states in LDS: the two fronts of a subchain sit in adjacent
// lanes of one wave, which read their states before either is written, so
// a partner activated in this pass is not also advanced in it.  With more
// fronts than fit, the kernel runs as several work groups over disjoint
// ranges that keep each subchain's two fronts together.
__global__ void __launch_bounds__(CONTROL_THREADS)
aberth_control(Front *__restrict__ fronts, int32_t *__restrict__ counts, int32_t n_fronts,
               Control *__restrict__ ctl, int32_t max_cold, int32_t max_warm,
               int32_t *__restrict__ workflag, const double4 *__restrict__ vsum,
               const Real *__restrict__ reals, const double2 *__restrict__ unit,
               int32_t fronts_per_group, int32_t predictor, int32_t *__restrict__ passupd,
               int32_t max_polish, int32_t xfrom)
{
    __shared__ int32_t st[4096];
    __shared__ int32_t s_active, s_live;
    __shared__ unsigned long long s_upd[TALLIES], s_star[TALLIES];
    const int tid = threadIdx.x;
    const int f0 = blockIdx.x * fronts_per_group;
    const int f1 = min(n_fronts, f0 + fronts_per_group);
    if (tid == 0) {
        s_active = 0;
        s_live = 0;
    }
    if (tid < TALLIES) s_upd[tid] = s_star[tid] = 0ull;
    unsigned long long my_upd[TALLIES] = {}, my_star[TALLIES] = {};
    for (int f = f0 + tid; f < f1; f += CONTROL_THREADS) st[f - f0] = fronts[f].state;
    __syncthreads();
    for (int f = f0 + tid; f < f1; f += CONTROL_THREADS) {
        if (st[f - f0] != FRONT_ACTIVE) continue;
        Front fr = fronts[f];
        atomicOr(&s_live, 1 << fr.phase);
        const Real &R = reals[fr.real];
        const int ph = fr.phase;
        const bool fast = fast_roots_pass(fr, R);
        const unsigned long long u = (unsigned)passupd[f];   // this round's updates of the front
        passupd[f] = 0;
        const int32_t c = counts[f];
        counts[f] = 0;
        advance_front(fr, f, c, vsum + 2 * f, fronts, st, f0, ctl, reals, unit, max_cold,
                      max_warm, predictor, max_polish, xfrom);
        tally_updates(my_upd, my_star, ph, fast, u, (unsigned)R.n_stars);
        fronts[f] = fr;
    }
    for (int q = 0; q < TALLIES; ++q) {
        if (my_upd[q]) {
            atomicAdd(&s_upd[q], my_upd[q]);
            atomicAdd(&s_star[q], my_star[q]);
        }
    }
    __syncthreads();
    if (tid < TALLIES && s_upd[tid]) {
        atomicAdd(&ctl->upd[tid], s_upd[tid]);
        atomicAdd(&ctl->star[tid], s_star[tid]);
    }
    int mine = 0;
    for (int f = f0 + tid; f < f1; f += CONTROL_THREADS)
        mine += (st[f - f0] == FRONT_ACTIVE || st[f - f0] == FRONT_IDLE);
    if (mine) atomicAdd(&s_active, mine);
    __syncthreads();
    if (tid == 0) {
        // several groups: each adds its share; the first round of counting is
        // reset by the host-side clear kernel below
        atomicAdd(&ctl->active_fronts, s_active);
        if (s_live) atomicOr(workflag, s_live);
    }
}

// Clears the per-round totals the control groups add into, and counts the
// round as live if any group saw an active front (runs after them).
__global__ void control_begin(Control *__restrict__ ctl, int32_t *__restrict__ workflag)
{
    if (threadIdx.x == 0) {
        ctl->active_fronts = 0;
        *workflag = 0;
    }
}

__global__ void control_end(Control *__restrict__ ctl, const int32_t *__restrict__ workflag)
{
    if (threadIdx.x == 0 && *workflag) ctl->live_sweeps += 1;
}

// ---------------------------------------------------------------------------
// Persistent scheduler
// ---------------------------------------------------------------------------
//
// One launch of as many work groups as fit on the chip.  Work items are
// (front, task) passes in a device-side ring, a task being a run of the
// front's blocks: a worker claims the next slot, waits until it is filled,
// runs the pass the front's phase asks for, and the worker that completes the
// last task of a front's pass advances that front (advance_front) and queues
// its next pass, or runs it itself when the front makes one task, so fronts
// move on independently instead of in global rounds.  Each front keeps its
// own ping-pong parity; a cold start hands its converged centre row to its
// partner by copying it into the partner's buffer.  No worker ever waits
// for another one's pass: it waits only for its claimed slot, which the
// worker that queued the work fills, and leaves when every front is done,
// or, failing that, after a wall-clock interval without any pass finishing
// anywhere (the call then reports an error).

// Queue header; every counter sits on a cache line of its own, so workers
// polling one of them do not slow the atomics on another.
struct PQueue {
    unsigned long long head;      // next slot to claim
    unsigned long long pad0[31];
    unsigned long long tail;      // next slot to fill
    unsigned long long pad1[31];
    unsigned long long progress;  // passes completed
    unsigned long long pad2[31];
    int32_t done;                 // fronts finished (DONE, FAILED or PARKED)
    int32_t pad3[63];
    int32_t abort;                // a worker saw no progress for too long
    int32_t target;               // fronts the launch has to finish
    int32_t pad4[62];
};
// Slot sequence numbers are spread one per 64-byte line.
constexpr int SEQ_STRIDE = 8;
// Most waves of a work group of the persistent launch.
constexpr int MAX_WORK_WAVES = 8;

// Tasks of a pass over a front of field r.
__device__ __forceinline__ int task_count(const Real &r)
{
    return (((r.n_r + 63) >> 6) + r.chunk - 1) / r.chunk;
}

// Queues the n tasks of a pass of front f (whole wave).
__device__ __forceinline__ void push_front(PQueue *q, int2 *tasks, unsigned long long *seq,
                                           unsigned long long mask, int f, int n)
{
    const int lane = threadIdx.x & 63;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&q->tail, (unsigned long long)n);
    base = __shfl(base, 0, 64);
    for (int i = lane; i < n; i += 64) tasks[(base + i) & mask] = make_int2(f, i);
    // publishes the tasks and everything the work group wrote before them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    for (int i = lane; i < n; i += 64)
        __hip_atomic_store(&seq[((base + i) & mask) * SEQ_STRIDE], base + i + 1,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until the wave's stores have reached L2, where a release fence of
// another wave of the work group publishes them.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Row sums of a polished row from its blocks' partial sums (slots of one
// row), in row_sums' order (whole wave; every lane holds the result).
__device__ __forceinline__ void sum_row(const double4 *__restrict__ v, int bpf, double4 *rs)
{
    double v0 = 0, v1 = 0, v2 = 0, v3 = 0, v4 = 0, v5 = 0, v6 = 0, v7 = 0;
    for (int b = threadIdx.x & 63; b < bpf; b += 64) {
        const double4 t = v[2 * b], u = v[2 * b + 1];
        v0 += t.x; v1 += t.y; v2 += t.z; v3 += t.w;
        v4 += u.x; v5 += u.y; v6 += u.z; v7 += u.w;
    }
    wave_sum(v0); wave_sum(v1); wave_sum(v2); wave_sum(v3);
    wave_sum(v4); wave_sum(v5); wave_sum(v6); wave_sum(v7);
    rs[0] = make_double4(v0, v1, v2, v3);
    rs[1] = make_double4(v4, v5, v6, v7);
}

// ---------------------------------------------------------------------------
// Fronts between the expansions and the passes
// ---------------------------------------------------------------------------

// Before the expansions: no front counted, and an empty queue, whose slots go
// on being numbered (workers of the last launch claimed beyond its tail).
__global__ void expand_begin(Control *__restrict__ ctl, PQueue *q)
{
    ctl->active_fronts = 0;
    ctl->parked_fronts = 0;
    if (q) {
        q->head = q->tail;
        q->done = 0;
        q->target = 0;
    }
}

// Rows with roots from expansions, each accepted by itself: nothing kept two
// chains from ending at one root, as the root-root sum of an Aberth step does, so
// a row counts once its identities hold.  For every parked front, the work groups of grid row blockIdx.x take in turn the rows which all
// its blocks have settled, read their roots back and leave in bad[f] the first
// row, counted from the front's own, whose identities fail.  The error of a root
// is allowed EXP_ERR, which acceptance bounds, and what the rounding of F leaves,
// 4 u (|gamma| + |1 - kappa_s|) / |F'| with F' = -2 M / d^3 of all stars at their
// centre, d away: roots far outside the stars are moved most by it.  The sums of
// those errors, and sum |r|, are bounded through sums of even powers (Cauchy's
// inequality), so that no root takes a square root.
// Bound by the latency of a row: a few reads a lane, then the reduction.  One
// work group of four waves a row and eight separate reductions took 163 us a
// launch for 86 fields of 1,088 steps; a wave a row and one reduction in halves
// take 70, and 48 with a work group for every eight rows of a front (2.8, 1.2 and
// 0.8 ms a call; N = 6,000, 1.9 GB of roots: 0.9 ms).  In the mixed
// form it takes the place of row sums formed in the expansion kernel, which held
// a block to 1,024 rows ahead of its front and took up to 512 MiB, and of their
// check one row at a time: N = 10,000 with multipole sums 52.0 -> 44.9 ms, of which
// 1.4 here for 6.4 GB.
__global__ void __launch_bounds__(CONTROL_THREADS)
expand_check(const Front *__restrict__ fronts, const Real *__restrict__ reals,
             const double2 *__restrict__ unit, const int32_t *__restrict__ next_row,
             const double *__restrict__ out_re, const double *__restrict__ out_im,
             const double2 *__restrict__ bnd, int32_t *__restrict__ bad)
{
    constexpr int NV = 8;
    __shared__ double part[CONTROL_THREADS / 64][NV];
    const Front *F = fronts + blockIdx.x;
    if (F->state != FRONT_PARKED) return;
    const Real &R = reals[F->real];
    const int n_r = R.n_r, bpf = (n_r + 63) >> 6, dir = F->dir, row0 = F->row;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    int h = 0x7fffffff;   // rows settled by every block
    for (int b = lane; b < bpf; b += 64) h = min(h, (next_row[F->blk0 + b] - row0) * dir);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) h = min(h, __shfl_xor(h, off, 64));
    const double cx = R.sz_r / R.n_stars, cy = R.sz_i / R.n_stars;
    const double far = 2.0 * 1.1102230246251565e-16 * (fabs(R.gamma) + R.a1) / R.M;
    for (int i = blockIdx.y; i < h; i += gridDim.y) {
        const int row = row0 + i * dir;
        const bool boundary = F->bnd_slot >= 0 && row == F->end_row;
        const int64_t o = R.out_off + (int64_t)row * n_r;
        const double2 *br = bnd + R.bnd_off + (int64_t)max(F->bnd_slot, 0) * n_r;
        // sum r, sum r^2, sum |r|^2, and sum d^2, d^4, d^6
        double v[NV] = {};
#pragma unroll 4
        for (int k = threadIdx.x; k < n_r; k += blockDim.x) {
            const double2 z = boundary ? br[k] : make_double2(out_re[o + k], out_im[o + k]);
            const double dx = z.x - cx, dy = z.y - cy, d2 = fma(dx, dx, dy * dy);
            v[0] += z.x;
            v[1] += z.y;
            v[2] += z.x * z.x - z.y * z.y;
            v[3] += 2.0 * z.x * z.y;
            v[4] += fma(z.x, z.x, z.y * z.y);
            v[5] += d2;
            v[6] += d2 * d2;
            v[7] += d2 * d2 * d2;
        }
        // a lane hands half of its values over at each of three levels, so that
        // the lanes of an eighth of the wave come to hold one of them
#pragma unroll
        for (int half = NV / 2; half >= 1; half >>= 1) {
            const bool up = lane & (8 * half);
#pragma unroll
            for (int j = 0; j < half; ++j) {
                const double give = up ? v[j] : v[j + half], keep = up ? v[j + half] : v[j];
                v[j] = keep + __shfl_xor(give, 8 * half, 64);
            }
        }
        double w = v[0];   // value lane / 8
#pragma unroll
        for (int off = 4; off >= 1; off >>= 1) w += __shfl_xor(w, off, 64);
        if ((lane & 7) == 0) part[wave][lane >> 3] = w;
        if (waves > 1) __syncthreads();
        else wave_sync();
        if (threadIdx.x == 0) {
            double s[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                s[q] = part[0][q];
                for (int x = 1; x < waves; ++x) s[q] += part[x][q];
            }
            const double e2 = 2.0 * (n_r * EXP_ERR * EXP_ERR + far * far * s[7]);   // sum err^2
            const double4 rs[2] = {
                make_double4(s[0], s[1], s[2], s[3]),
                make_double4(n_r * EXP_ERR + far * sqrt(s[5] * s[6]), 2.0 * sqrt(e2 * s[4]) + e2,
                             sqrt(n_r * s[4]), s[4])};
            if (!row_identities_hold(R, unit[row], rs)) atomicMin(&bad[blockIdx.x], i);
        }
        if (waves > 1) __syncthreads();
        else wave_sync();
    }
}

// After the expansions, one work group per parked front: the front moves past the
// rows all its blocks have settled, while their row identities hold.  If a
// block is stuck at the row it comes to, the front is active again: the row's
// first pass steps the roots left open, from their extrapolation, the others
// entering at the previous row's roots.  If a row's identities fail, the mixed
// form goes the way of a polish that does; in FP64 every root of the row takes
// Aberth steps from its extrapolation, as without expansions, which keep the
// roots apart.  Either way, what blocks ahead of it found is done anew.
// Otherwise the front stays parked, or is done.
__global__ void __launch_bounds__(64)
expand_control(Front *__restrict__ fronts, const Real *__restrict__ reals,
               const int32_t *__restrict__ next_row, const int32_t *__restrict__ stuck,
               int32_t predictor, int32_t xfrom, int32_t *__restrict__ bad,
               Control *__restrict__ ctl, PQueue *q, int2 *tasks, unsigned long long *seq,
               unsigned long long mask)
{
    const int f = blockIdx.x, lane = threadIdx.x;
    Front fr = fronts[f];   // every lane advances a copy of its own
    if (fr.state != FRONT_PARKED) return;
    const Real &R = reals[fr.real];
    const int bpf = (R.n_r + 63) >> 6;
    const bool polish = fr.phase == PH_POLISH;
    int h = 0x7fffffff;   // rows settled by every block
    for (int b = lane; b < bpf; b += 64) h = min(h, (next_row[fr.blk0 + b] - fr.row) * fr.dir);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) h = min(h, __shfl_xor(h, off, 64));
    const int row0 = fr.row, dir = fr.dir;
    const int counted = fr.settled;   // its roots are in the tallies
    const int moved = min(h, bad[f]);
    const bool failed = moved < h;
    fr.redo = 0;
    fr.npass += 1;
    if (moved > 0) {   // the last of them is done
        fr.max_warm = max(fr.max_warm, 1);
        fr.row += (moved - 1) * dir;
        fr.hist = min(fr.hist + moved - 1, 3);
        row_done(fr, nullptr, f, predictor, xfrom);
    }
    bool any = false;
    if (fr.state == FRONT_PARKED && !failed)
        for (int b = lane; b < bpf; b += 64)
            any |= stuck[fr.blk0 + b] && next_row[fr.blk0 + b] == row0 + moved * dir;
    const bool held = __ballot(any) != 0;
    if (fr.state == FRONT_PARKED && (failed || held)) {
        fr.state = FRONT_ACTIVE;
        fr.src = f;
        if (!failed) {
            fr.shared = 1;
        } else if (polish) {
            fr.fresh = 0;
            retry_row(fr, ctl, lane == 0);
        } else {
            start_row(fr, predictor, 0);
            fr.stamp += 1;
            fr.redo = 1;
            if (lane == 0) atomicAdd((unsigned long long *)&ctl->rows_fallback, 1ull);
        }
        fr.passes_row = 1;
    }
    if (lane == 0) {   // every lane has read them
        fronts[f] = fr;
        bad[f] = 0x7fffffff;   // for the next time
        const unsigned long long up = (unsigned long long)max(moved - counted, 0) * (unsigned)R.n_r;
        if (up) atomicAdd(&ctl->upd[polish ? TALLY_ROOTS + 1 : TALLY_ROOTS], up);
        if (fr.state == FRONT_ACTIVE) atomicAdd(&ctl->active_fronts, 1);
        if (fr.state == FRONT_PARKED) atomicAdd(&ctl->parked_fronts, 1);
    }
    if (q && fr.state == FRONT_ACTIVE) {   // persistent schedule: the next launch's work
        push_front(q, tasks, seq, mask, f, task_count(R));
        if (lane == 0) atomicAdd(&q->target, 1);
    }
}

// Iterates of the fronts expand_control made active: the previous row's roots
// for a row's first pass, the row's own for one that is retried; where the row
// keeps the roots its blocks found, those of blocks that had settled it are
// flagged (the stuck ones' flags are in place).  Counts the accepted roots.
__global__ void __launch_bounds__(64)
expand_gather(const Front *__restrict__ fronts, const Real *__restrict__ reals,
              const int2 *__restrict__ bmap, const int32_t *__restrict__ next_row,
              const double *__restrict__ out_re, const double *__restrict__ out_im,
              const double2 *__restrict__ bnd, double2 *__restrict__ iter0,
              double2 *__restrict__ iter1, int32_t *__restrict__ flagrow,
              double *__restrict__ errbuf, Control *__restrict__ ctl)
{
    const int2 fq = bmap[blockIdx.x];
    const Front *F = fronts + fq.x;
    if (F->state != FRONT_ACTIVE) return;
    const Real *R = reals + F->real;
    const int k = fq.y * 64 + threadIdx.x;
    const bool valid = k < R->n_r;
    const int64_t i = F->it_off + k;
    bool flagged = false;
    if (valid) {
        const int row = F->fresh ? F->row - F->dir : F->row;
        const int64_t o = R->out_off + (int64_t)row * R->n_r + k;
        const bool b = F->bnd_slot >= 0 && row == F->end_row;
        (F->par ? iter1 : iter0)[i] =
            b ? bnd[R->bnd_off + (int64_t)F->bnd_slot * R->n_r + k] : make_double2(out_re[o], out_im[o]);
        if (!F->shared) {
            flagged = false;
        } else if (next_row[F->blk0 + fq.y] != F->row) {
            flagrow[i] = F->stamp;
            if (errbuf) errbuf[i] = 0.0;
            flagged = true;
        } else {
            flagged = flagrow[i] == F->stamp;
        }
    }
    const unsigned long long n = __popcll(__ballot(flagged));
    if (threadIdx.x == 0 && n)
        atomicAdd(&ctl->upd[F->phase == PH_F64 ? TALLY_ROOTS : TALLY_ROOTS + 1], n);
}

// What the waves of a work group share: the front it works on, the pass's
// block cursor and totals, and what its first wave decided after the pass.
struct WorkShare {
    Front fr;
    int32_t task_f, task_c;   // claimed task (task_f < 0: leave)
    int32_t begin, end;       // blocks of the task
    int32_t count, upd;       // the pass's totals over this task
    int32_t go;               // the work group owns the front and runs its next pass
    int32_t partner;          // front whose cold start just ended here (else -1)
    int64_t src_off, dst_off;
    int32_t src_par, dst_par;
    unsigned long long upd_tot[TALLIES], star_tot[TALLIES];   // the work group's (tally_work)
};

// What bounds short passes is not their sums but what surrounds them: a
// device saturates at ~12.6 M agent-scope release fences plus queue claims per
// second, so with one 64-root block per claim the 1,000-star workload (32
// blocks per front, ~700 k block passes) ran at that rate whatever its
// kernels did.  A work group therefore has several waves and takes a task of
// several blocks, dealt to its waves in turn: one claim, one fence and one
// count per task.  A front that makes a single task is owned
// by the work group that took it: its passes follow each other behind work
// group barriers alone, the front record stays in LDS, and nothing crosses
// XCDs until it is done or hands a cold start to its partner.
template <bool EQUAL, bool FMM>
__global__ void __launch_bounds__(64 * MAX_WORK_WAVES)
__attribute__((amdgpu_waves_per_eu(FMM ? MLCC_FMM_WAVES : MLCC_SWEEP_WAVES, 8)))
aberth_persistent(RoundArgs<typename StarRec<EQUAL>::T> A, Front *__restrict__ fronts_w,
                  PQueue *__restrict__ q, int2 *__restrict__ tasks,
                  unsigned long long *__restrict__ seq, unsigned long long mask,
                  int32_t *__restrict__ fdone, int32_t max_cold, int32_t max_warm,
                  unsigned long long stall_ticks)
{
    using T = typename StarRec<EQUAL>::T;
    extern __shared__ double4 tiles_all[];   // two tiles of 64 records per wave
    __shared__ WorkShare W;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    double4 *tiles = reinterpret_cast<double4 *>(reinterpret_cast<T *>(tiles_all) + wave * 128);
    if (threadIdx.x < TALLIES) W.upd_tot[threadIdx.x] = W.star_tot[threadIdx.x] = 0ull;
    for (;;) {
        if (threadIdx.x == 0) {
            int tf = -1, tq = 0;
            const unsigned long long t = atomicAdd(&q->head, 1ull);
            const unsigned long long *my = &seq[(t & mask) * SEQ_STRIDE];
            unsigned long long seen = load_relaxed(&q->progress);
            unsigned long long t0 = wall_clock64();
            for (unsigned it = 1;; ++it) {
                if (load_relaxed(my) == t + 1) {
                    (void)load_acquire(my);
                    const int2 w = tasks[t & mask];
                    tf = w.x;
                    tq = w.y;
                    break;
                }
                if ((it & 31) == 0) {   // the shared counters, now and then
                    if (load_relaxed(&q->abort)) break;
                    if (load_relaxed(&q->done) >= load_relaxed(&q->target)) break;
                    const unsigned long long pnow = load_relaxed(&q->progress);
                    const unsigned long long now = wall_clock64();
                    if (pnow != seen) {
                        seen = pnow;
                        t0 = now;
                    } else if (now - t0 > stall_ticks) {
                        atomicExch(&q->abort, 1);
                        break;
                    }
                }
                __builtin_amdgcn_s_sleep(2);
            }
            W.task_f = tf;
            W.task_c = tq;
        }
        __syncthreads();
        const int tf = __builtin_amdgcn_readfirstlane(W.task_f);
        if (tf < 0) break;
        int tc = __builtin_amdgcn_readfirstlane(W.task_c);
        constexpr int FRONT_WORDS = sizeof(Front) / 4;
        static_assert(FRONT_WORDS <= 64 && sizeof(Front) % 4 == 0, "front copied by one wave");
        if (wave == 0 && lane < FRONT_WORDS)
            reinterpret_cast<int32_t *>(&W.fr)[lane] =
                reinterpret_cast<const int32_t *>(fronts_w + tf)[lane];
        for (;;) {   // passes over the front: one, or all of them while it is owned
            if (wave == 0) {
                wave_sync();
                if (lane == 0) {
                    const int c = A.reals[W.fr.real].chunk;
                    const int bpf = (A.reals[W.fr.real].n_r + 63) >> 6;
                    W.begin = tc * c;
                    W.end = min((tc + 1) * c, bpf);
                    W.count = 0;
                    W.upd = 0;
                }
            }
            __syncthreads();
            const int end = __builtin_amdgcn_readfirstlane(W.end);
            const int ph = __builtin_amdgcn_readfirstlane(W.fr.phase);
            for (int blk = __builtin_amdgcn_readfirstlane(W.begin) + wave; blk < end; blk += waves) {
                BlockCtx<T> B;
                enter_fq(A, &W.fr, tf, blk, &W.count, &W.upd, B);
                if (ph == PH_F64)
                    sweep_f64_pass<EQUAL, FMM>(A, B, tiles);
                else if (ph == PH_F32)
                    sweep_f32_pass<EQUAL, FMM>(A, B, tiles);
                else
                    polish_pass<EQUAL, FMM>(A, B, tiles);
            }
            // every wave's stores have reached L2 before the first wave, which
            // publishes them, leaves the barrier
            wait_stores();
            __syncthreads();
            if (wave == 0) {
                Front fr = W.fr;   // lane 0's copy is the one that is advanced
                const Real *R = A.reals + fr.real;
                const int bpf = (R->n_r + 63) >> 6;
                const int nt = task_count(*R);
                int last = 1;
                if (nt > 1) {
                    // the last task of the front's pass advances the front;
                    // every task publishes its writes before counting itself
                    if (lane == 0) {
                        if (W.count) atomicAdd(&A.counts[tf], W.count);
                        if (W.upd) atomicAdd(&A.passupd[tf], W.upd);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    if (lane == 0) last = atomicAdd(&fdone[tf], 1) + 1 == nt;
                    last = __shfl(last, 0, 64);
                    if (last) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                        if (lane == 0) {
                            fdone[tf] = 0;
                            W.count = load_relaxed(&A.counts[tf]);
                            A.counts[tf] = 0;
                            W.upd = load_relaxed(&A.passupd[tf]);
                            A.passupd[tf] = 0;
                        }
                    }
                }
                int go = 0, partner = -1;
                if (last) {
                    double4 rs[2] = {make_double4(0, 0, 0, 0), make_double4(0, 0, 0, 0)};
                    if (ph == PH_POLISH)
                        sum_row(A.vieta + 2 * fr.blk0, bpf, rs);
                    int finished = 0;
                    if (lane == 0) {
                        const int dir0 = fr.dir;
                        tally_updates(W.upd_tot, W.star_tot, ph, fast_roots_pass(fr, *R),
                                      (unsigned)W.upd, (unsigned)R->n_stars);
                        partner = advance_front(fr, tf, W.count, rs, fronts_w, nullptr, 0, A.ctl,
                                                A.reals, A.unit, max_cold, max_warm, A.predictor,
                                                max_polish_passes(FMM), A.xfrom);
                        fr.par ^= 1;   // the pass wrote the other buffer
                        const int state = fr.state;   // finished: done, failed or parked
                        if (state != FRONT_ACTIVE)
                            finished = (state == FRONT_FAILED && dir0 == 0) ? 2 : 1;
                        else
                            go = task_count(*R) == 1 ? 1 : 2;
                        // a partner that waits for the expansions from its first row on
                        if (partner >= 0 && fronts_w[partner].state != FRONT_ACTIVE) {
                            finished += 1;
                            partner = -1;
                        }
                        W.fr = fr;
                        if (partner >= 0) {
                            W.src_par = fr.par;
                            W.src_off = fr.it_off;
                            W.dst_par = fronts_w[partner].par;
                            W.dst_off = fronts_w[partner].it_off;
                        }
                    }
                    wave_sync();
                    go = __shfl(go, 0, 64);
                    if (go != 1 && lane < FRONT_WORDS)   // it leaves this work group
                        reinterpret_cast<int32_t *>(fronts_w + tf)[lane] =
                            reinterpret_cast<const int32_t *>(&W.fr)[lane];
                    if (lane == 0) {
                        if (finished) atomicAdd(&q->done, finished);
                        atomicAdd(&q->progress, 1ull);
                    }
                }
                if (lane == 0) {
                    W.go = go;
                    W.partner = partner;
                }
            }
            __syncthreads();
            const int partner = W.partner, go = W.go;
            if (partner >= 0) {
                // the partner starts from the converged centre row (copied before
                // the front's own next pass is queued: the one after it
                // overwrites this buffer)
                const Real *R = A.reals + W.fr.real;
                const double2 *src = (W.src_par ? A.iter1 : A.iter0) + W.src_off;
                double2 *dst = (W.dst_par ? A.iter1 : A.iter0) + W.dst_off;
                for (int i = threadIdx.x; i < R->n_r; i += blockDim.x) dst[i] = src[i];
                wait_stores();
                __syncthreads();
                if (wave == 0) push_front(q, tasks, seq, mask, partner, task_count(*R));
            }
            if (go == 2 && wave == 0)
                push_front(q, tasks, seq, mask, tf, task_count(A.reals[W.fr.real]));
            if (go != 1) break;
            tc = 0;
        }
        __syncthreads();   // the claim below overwrites what the waves just read
    }
    // the work group's share of the totals
    if (threadIdx.x < TALLIES && W.upd_tot[threadIdx.x]) {
        atomicAdd(&A.ctl->upd[threadIdx.x], W.upd_tot[threadIdx.x]);
        atomicAdd(&A.ctl->star[threadIdx.x], W.star_tot[threadIdx.x]);
    }
}

// ---------------------------------------------------------------------------
// Subchains and the autotuner
// ---------------------------------------------------------------------------

// Subchain counts S must divide m/2 (integer centre rows).  The autotuner
// prices a run with S subchains from measured costs of the kernels on
// gfx950 and picks the cheapest S.
//
// Cost of one wave's pass over a field of N stars and n_r = 2N roots, in
// SIMD cycles (issue costs measured per wave64 instruction with eight
// independent chains per lane: FP64 add/mul ~4.8, FMA ~5.3, v_rcp_f64
// ~16.6; FP32 add/mul ~2.7, FMA ~4.1, v_rcp_f32 ~8.6), fitted when the
// kernels spent ~21 instructions per star term and ~9 per root term in a
// sweep and ~22 per star term in the polish (now ~19, ~9 and ~20 with the
// eight-term reciprocal groups; S depends on the ratios of these costs,
// which moved by a few per cent):
//   FP64 Aberth sweep   114 N + 47 n_r
//   FP32 Aberth sweep    56 N + 22 n_r
//   FP64 Newton polish  120 N
// (Warm rows of MLCC_FP64_R32 take their root terms in FP32, ~40 instead of
// ~47 cycles per root; the model keeps 47, and S sweeps of measured run
// times put its choice within 1% of the best S on the workloads tried.)
// A run does, per field, u (m + S) row passes of every block (u ~ 1.03
// with the chain predictor, ~2 without; in the mixed form a row without a
// prediction takes an FP32 sweep and a polish) plus S cold starts of ~27
// sweeps.  Its time is that work over the 1024 SIMDs (fewer when fewer than
// two waves per SIMD are in flight), plus, for every round, the tail of a
// round: ~0.8 of the longest wave pass, plus ~40 us of launches and control.
// The number of rounds is ~2.1 per row of a front's m / 2S rows, plus the
// cold start.
// With multipole star sums (one field) a wave's star part is a few near
// stars and one series of order ~48: ~3,400 instructions, but bound by the
// latency of its chain of dependent loads (cell, coefficients chunk by
// chunk, near-cell ranges): measured on n10k at 4 waves per SIMD, a polish
// pass occupies ~94k SIMD cycles whatever N, and the star part of a sweep
// is priced the same; the root terms keep their cost.
// All of this prices warm rows that sum over every star in passes, among them
// multipole polish passes of the persistent mixed form that went on through
// further rows (fmm_rows_per_pass), as they no longer do: rows come from
// expansions, priced by nothing here.  The choice stays what it was because the
// centre row of the first of the S subchains is where the columns get their
// numbers.  For one field it decides nothing else (plan_pieces), but a batch
// grows its S subchains, and what S would be best for it now is not measured.
struct TuneModel {
    double cold_sweeps = 27.0, rounds_per_row = 2.1, tail = 0.8, round_us = 40.0;
    double clock_hz = 2.4e9, simds = 1024.0;
    double fmm_star_cycles = 94000.0;
    double fmm_rows_per_pass = 6.0;
};

static double pass_cycles(int kind, double n, bool fmm)
{
    const TuneModel tm;
    const double n_r = 2.0 * n;
    if (kind == PH_F64) return (fmm ? tm.fmm_star_cycles : 114.0 * n) + 47.0 * n_r;
    if (kind == PH_F32) return (fmm ? tm.fmm_star_cycles : 56.0 * n) + 22.0 * n_r;
    return fmm ? tm.fmm_star_cycles : 120.0 * n;
}

static double predicted_seconds(const std::vector<RealHost> &reals, int64_t m, int64_t s, bool mixed,
                         int predictor, bool fmm, bool xrows)
{
    const TuneModel tm;
    double work = 0.0, blocks_all = 0.0, longest = 0.0;
    for (const RealHost &r : reals) {
        const double n = (double)r.n, blocks = std::ceil(2.0 * n / 64.0);
        double row, cold;
        if (!mixed) {
            row = (predictor > 0 ? 1.03 : 2.0) * pass_cycles(PH_F64, n, fmm);
            cold = tm.cold_sweeps * pass_cycles(PH_F64, n, fmm);
        } else {
            row = 1.02 * pass_cycles(PH_POLISH, n, fmm) +
                  (predictor > 0 ? 0.0 : pass_cycles(PH_F32, n, fmm));
            cold = tm.cold_sweeps * pass_cycles(PH_F32, n, fmm) + pass_cycles(PH_POLISH, n, fmm);
        }
        work += blocks * (row * (double)(m + s) + cold * (double)s);
        blocks_all += blocks;
        longest = std::max(longest, mixed ? pass_cycles(PH_POLISH, n, fmm)
                                          : pass_cycles(PH_F64, n, fmm));
    }
    // about half of the 2S fronts are in a full pass at any time
    const double waves = (double)s * blocks_all;
    const double simds = std::min(tm.simds, std::max(1.0, waves / 2.0));
    const double rows_per_pass = (xrows && mixed && fmm && predictor > 0) ? tm.fmm_rows_per_pass : 1.0;
    const double rounds =
        tm.rounds_per_row * (double)(m / 2) / (double)s / rows_per_pass + tm.cold_sweeps;
    return work / (simds * tm.clock_hz) +
           rounds * (tm.tail * longest / tm.clock_hz + tm.round_us * 1e-6);
}

// Picks S for every field of a call (all fields share one round clock, so a
// common S keeps their fronts in step): the divisor of m/2 with the lowest
// predicted time among those that leave every subchain at least 16 rows and
// keep the front table within MAX_FRONTS.
static int autotune_subchains(const std::vector<RealHost> &reals, int64_t m, bool mixed,
                              int predictor, bool fmm, bool persistent)
{
    const int64_t half = m / 2;
    const int64_t s_max = std::max<int64_t>(
        1, std::min<int64_t>(MAX_FRONTS / (2 * (int64_t)reals.size()), m / 16));
    double best = 1e300;
    int best_s = 1;
    for (int64_t s = 1; s <= std::min<int64_t>(half, std::min<int64_t>(s_max, 4096)); ++s) {
        if (half % s) continue;
        const double t = predicted_seconds(reals, m, s, mixed, predictor, fmm, persistent);
        if (t < best * 0.999) {
            best = t;
            best_s = (int)s;
        }
    }
    return best_s;
}

// A piece of the phase grid grown from one cold start at its centre row.
struct Piece {
    int64_t lo, hi, cen;
};

// With rows from expansions a cold start (11-30 sweeps over every star and
// root) costs as much as hundreds of rows, so it is the cold starts that make
// up a call, and no more of them are made than keep the device full: pieces
// whose fronts hold COLD_BLOCKS blocks of 64 roots between them.  The first
// one keeps the centre row of the first of S equal subchains, whose cold start
// numbers the columns.  Measured, ms a call for each of two fields, with 2048 /
// 3072 / 4096 / 6144 blocks: N = 6,000 FP64 52 47 / 44 47 / 43 43 / 46 44; N = 4,099
// mixed 23 41 / 24 37 / 26 36 / 30 34; N = 10,000 mixed with multipole sums 43 66 /
// 44 57 / 45 51 / 46 51; N = 5,000 FP64 with them 25 28 / 21 22 / 20 22 / 20 21; N = 3,000
// 11.9 9.6 / 11.4 10.4 / 10.8 10.4 / 11.8 10.7; N = 1,000 FP64 5.4 5.2 / 6.1 5.6 / 5.8 6.3 / 7.4
// 6.9; N = 300 2.1 1.7 / 2.5 1.9 / 2.6 2.3 / 2.9 2.5; rectangular N = 437 4.2 5.2 / 4.3 4.7 / 4.4
// 5.0 / 5.2 5.8.  A few long pieces wait for their stuck blocks, most in the largest
// fields, and how long differs from field to field; 4096 is near the best for all
// of them but the small ones, which 2048 serves 10 to 25% faster.  Batches keep
// their subchains: their largest fields' pieces would set the time (40 fields mixed
// 65 ms with one piece per subchain, 197 / 134 / 112 with 2048 / 4096 / 6144 blocks).
#ifndef MLCC_COLD_BLOCKS
#define MLCC_COLD_BLOCKS 4096
#endif

static std::vector<Piece> plan_pieces(const std::vector<RealHost> &reals, int64_t m, int S,
                                      bool fewer)
{
    int64_t blocks = 0;
    for (const RealHost &r : reals) blocks += ceil_div(2 * r.n + sheet_poly(r).n_extra, 64);
    const int64_t L = m / S;
    const int64_t n =
        fewer ? std::min<int64_t>(S, std::max<int64_t>(1, MLCC_COLD_BLOCKS / (2 * blocks))) : S;
    std::vector<Piece> v;
    if (n == S) {
        for (int64_t s = 0; s < S; ++s) v.push_back(Piece{s * L, (s + 1) * L, s * L + L / 2});
        return v;
    }
    // the first piece's upper half is as long as the halves of the others
    const int64_t first = n == 1 ? m : (L * (n - 1) + m) / (2 * n - 1);
    v.push_back(Piece{0, first, L / 2});
    for (int64_t s = 1; s < n; ++s) {
        const int64_t lo = v.back().hi, hi = first + (m - first) * s / (n - 1);
        v.push_back(Piece{lo, hi, lo + (hi - lo) / 2});
    }
    return v;
}

// ---------------------------------------------------------------------------
// Work groups of the persistent launch
// ---------------------------------------------------------------------------

// Workers beyond the tasks a launch can have at a time: they find nothing to
// run and watch for a stall.
constexpr int WATCHERS = 8;
// Most blocks of a front whose passes one work group may own, and waves per
// work group when the longest front has more.
constexpr int OWN_MAX_BLOCKS = 8;
#ifndef MLCC_WORK_WAVES
#define MLCC_WORK_WAVES 4
#endif

// Waves per work group, and per field the blocks of a front that make one
// task (Real::chunk).  Fronts of at most 8 blocks are owned, one wave per
// block: a pass of so few blocks is shorter than the claim and the fences
// (N = 10: 1.09 -> 0.31 ms per launch; N = 137, 5 blocks: 3.07 -> 1.08 ms, where
// four waves and two tasks take 1.43).  Longer fronts go through the queue in
// tasks of four blocks, one per wave: measured launches, ms, with 1 / 2 / 4 / 8
// / 16 waves and as many blocks: rectangular field of 15 blocks 28.0 / 22.4 /
// 16.3 / 20.1 / 17.7; N = 3,000 with multipole sums 148 / 132 / 126 / 127 / 139;
// N = 6,000 FP64 1197 / 1139 / 1035 / 1042 / 1099; N = 10,000 mixed with
// multipole sums 146 / 128 / 121 / 119 / 124.  More blocks per task than waves
// lost everywhere (N = 1,000: 51 to 64 ms against 43), as did owning fronts
// of several blocks per wave (51 ms).
static int plan_workers(std::vector<Real> &rd)
{
    int64_t longest = 0;
    for (const Real &R : rd) longest = std::max(longest, ceil_div(R.n_r, 64));
    int waves = 1;
    while (waves < longest && waves < OWN_MAX_BLOCKS) waves <<= 1;
    if (longest > OWN_MAX_BLOCKS) waves = MLCC_WORK_WAVES;
    for (Real &R : rd) R.chunk = waves;
    return waves;
}

// ---------------------------------------------------------------------------
// Host driver
// ---------------------------------------------------------------------------

// Builds the fast-multipole grids of every field of the call: each field's
// stars binned and sorted by cell (the kernels then take the stars in that
// order), its expansions about the field centre on the host, its cells'
// local expansions on the device; one FmmArgs record per field, with
// pointers into the concatenated arrays.
static mlcc_status build_fmm(Ctx *c, int order, bool equal, std::vector<FmmArgs> &recs)
{
    const std::vector<double4> &st = c->hstars;
    const int pp = order > 0 ? order : 48;
    const int stride = (pp + 8) & ~7;
    const int n_real = (int)c->reals.size();
    struct Grid { int G; double x0, y0, w, cx, cy, R, wsum; int64_t cs_off, cell_off; };
    std::vector<Grid> grids(n_real);
    int64_t n_cs = 0, n_cells = 0;
    const int64_t n_all = (int64_t)st.size();
    std::vector<double4> sorted(n_all);
    std::vector<int32_t> starts;
    std::vector<double2> mm((size_t)n_real * 2 * (pp + 1), make_double2(0.0, 0.0));
    for (int r = 0; r < n_real; ++r) {
        const int64_t o = c->reals[r].star_off, n = c->reals[r].n;
        double xmin = st[o].x, xmax = st[o].x, ymin = st[o].y, ymax = st[o].y;
        for (int64_t i = o; i < o + n; ++i) {
            xmin = std::min(xmin, st[i].x); xmax = std::max(xmax, st[i].x);
            ymin = std::min(ymin, st[i].y); ymax = std::max(ymax, st[i].y);
        }
        Grid &g = grids[r];
        g.cx = 0.5 * (xmin + xmax);
        g.cy = 0.5 * (ymin + ymax);
        g.R = 0.0;
        g.wsum = 0.0;
        for (int64_t i = o; i < o + n; ++i) {
            g.R = std::max(g.R, std::hypot(st[i].x - g.cx, st[i].y - g.cy));
            g.wsum += equal ? 1.0 : st[i].z;
        }
        if (!(g.R > 0.0)) g.R = 1.0;
        g.R *= 1.0 + 1e-12;   // every star strictly inside the radius
        g.G = (int)std::min<double>(256.0, std::max(4.0, std::round(std::sqrt(1.7 * (double)n))));
        g.w = 4.0 * g.R / g.G;
        g.x0 = g.cx - 2.0 * g.R;
        g.y0 = g.cy - 2.0 * g.R;
        g.cs_off = n_cs;
        g.cell_off = n_cells;
        const int G = g.G;
        n_cs += (int64_t)G * G + 1;
        n_cells += (int64_t)G * G;
        // counting sort by cell; indices local to the field
        std::vector<int32_t> cell_of(n), start((size_t)G * G + 1, 0);
        for (int64_t i = 0; i < n; ++i) {
            const double4 &a = st[o + i];
            const int ix = std::min(G - 1, std::max(0, (int)std::floor((a.x - g.x0) / g.w)));
            const int iy = std::min(G - 1, std::max(0, (int)std::floor((a.y - g.y0) / g.w)));
            cell_of[i] = iy * G + ix;
            start[cell_of[i] + 1] += 1;
        }
        for (int q = 0; q < G * G; ++q) start[q + 1] += start[q];
        // sorted by cell; the fourth component carries the cell index
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        for (int64_t i = 0; i < n; ++i) {
            double4 a = st[o + i];
            a.w = (double)cell_of[i];
            sorted[o + fill[cell_of[i]]++] = a;
        }
        starts.insert(starts.end(), start.begin(), start.end());
        // expansions about the centre: M_k = sum w_i (z_i - c0)^k, and unit weights
        double2 *mf = mm.data() + (size_t)r * 2 * (pp + 1), *mg = mf + (pp + 1);
        for (int64_t i = o; i < o + n; ++i) {
            const double dx = st[i].x - g.cx, dy = st[i].y - g.cy, wi = equal ? 1.0 : st[i].z;
            double pr = 1.0, pi = 0.0;
            for (int k = 0; k <= pp; ++k) {
                mf[k].x += wi * pr; mf[k].y += wi * pi;
                mg[k].x += pr; mg[k].y += pi;
                const double t = pr * dx - pi * dy;
                pi = pr * dy + pi * dx;
                pr = t;
            }
        }
    }
    MLCC_TRY(c->fmm_cs.reserve(starts.size() * sizeof(int32_t)));
    MLCC_TRY(c->fmm_st.reserve(std::max<int64_t>(n_all, 1) * sizeof(double4)));
    MLCC_TRY(c->fmm_st2.reserve(std::max<int64_t>(n_all, 1) * sizeof(double2)));
    MLCC_TRY(c->fmm_cf.reserve((size_t)n_cells * stride * sizeof(double2)));
    MLCC_TRY(c->fmm_cg.reserve((size_t)n_cells * stride * sizeof(double2)));
    MLCC_TRY(c->fmm_q.reserve((size_t)n_cells * sizeof(double)));
    MLCC_TRY(c->fmm_m.reserve(mm.size() * sizeof(double2)));
    MLCC_TRY(c->fmm_args.reserve((size_t)n_real * sizeof(FmmArgs)));
    std::vector<double2> sorted2(n_all);
    for (int64_t i = 0; i < n_all; ++i) sorted2[i] = make_double2(sorted[i].x, sorted[i].y);
    MLCC_HIP(hipMemcpyAsync(c->fmm_cs.p, starts.data(), starts.size() * sizeof(int32_t),
                            hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemcpyAsync(c->fmm_st.p, sorted.data(), n_all * sizeof(double4),
                            hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemcpyAsync(c->fmm_st2.p, sorted2.data(), n_all * sizeof(double2),
                            hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemcpyAsync(c->fmm_m.p, mm.data(), mm.size() * sizeof(double2),
                            hipMemcpyHostToDevice, c->stream));
    recs.assign(n_real, FmmArgs{});
    for (int r = 0; r < n_real; ++r) {
        const Grid &g = grids[r];
        const int64_t o = c->reals[r].star_off;
        FmmArgs &M = recs[r];
        M.on = 1;
        M.G = g.G;
        M.p = pp;
        M.equal = equal;
        M.stride = stride;
        M.x0 = g.x0; M.y0 = g.y0; M.w = g.w; M.inv_w = 1.0 / g.w;
        M.cx = g.cx; M.cy = g.cy; M.R = g.R; M.wsum = g.wsum;
        M.cell_start = c->fmm_cs.as<int32_t>() + g.cs_off;
        M.fstars = c->fmm_st.as<double4>() + o;
        M.cf = c->fmm_cf.as<double2>() + g.cell_off * stride;
        M.cg = c->fmm_cg.as<double2>() + g.cell_off * stride;
        M.qfar = c->fmm_q.as<double>() + g.cell_off;
        M.mf = c->fmm_m.as<double2>() + (size_t)r * 2 * (pp + 1);
        M.mg = M.mf + (pp + 1);
    }
    MLCC_HIP(hipMemcpyAsync(c->fmm_args.p, recs.data(), recs.size() * sizeof(FmmArgs),
                            hipMemcpyHostToDevice, c->stream));
    // the cells' expansions, by the kernel that takes less time: a work group a
    // cell costs 0.09 ns per cell and star and ~8 us a launch; a lane a cell 0.8 us
    // per star of the largest field while there is a SIMD for every wave
    const int kb = stride == 56 ? 28 : 32, parts = (int)ceil_div(stride, kb);
    std::vector<P2lJob> jobs;
    double by_group = 0.0;
    int64_t n_max = 0;
    for (int r = 0; r < n_real; ++r) {
        const int64_t n = c->reals[r].n, cells = (int64_t)grids[r].G * grids[r].G;
        by_group += 8.0 + 9e-5 * (double)cells * (double)n;
        n_max = std::max(n_max, n);
        for (int64_t b = 0; b < cells; b += 64)
            for (int h = 0; h < parts; ++h) jobs.push_back(P2lJob{r, (int32_t)b, h * kb, (int32_t)n});
    }
    const double by_lane = 8.0 + 0.8 * (double)n_max * std::max(1.0, (double)jobs.size() / 1024.0);
    if (by_lane < by_group) {
        MLCC_TRY(c->fmm_jobs.reserve(jobs.size() * sizeof(P2lJob)));
        MLCC_HIP(hipMemcpyAsync(c->fmm_jobs.p, jobs.data(), jobs.size() * sizeof(P2lJob),
                                hipMemcpyHostToDevice, c->stream));
        auto lanes = [&](auto k, auto e) {
            hipLaunchKernelGGL((fmm_p2l_lanes<decltype(k)::value, decltype(e)::value>),
                               dim3((unsigned)jobs.size()), dim3(64), 0, c->stream,
                               c->fmm_jobs.as<P2lJob>(), c->fmm_args.as<FmmArgs>());
        };
        using K28 = std::integral_constant<int, 28>;
        using K32 = std::integral_constant<int, 32>;
        if (kb == 28) equal ? lanes(K28{}, std::true_type{}) : lanes(K28{}, std::false_type{});
        else equal ? lanes(K32{}, std::true_type{}) : lanes(K32{}, std::false_type{});
    } else {
        for (int r = 0; r < n_real; ++r) {
            const Grid &g = grids[r];
            const FmmArgs &M = recs[r];
            hipLaunchKernelGGL(fmm_p2l, dim3((unsigned)((int64_t)g.G * g.G)), dim3(64), 0, c->stream,
                               g.G, pp, stride, g.x0, g.y0, g.w, (int32_t)equal,
                               (int32_t)c->reals[r].n, M.fstars, const_cast<double2 *>(M.cf),
                               const_cast<double2 *>(M.cg), const_cast<double *>(M.qfar));
        }
    }
    MLCC_HIP(hipGetLastError());
    // host vectors must outlive the copies
    MLCC_HIP(hipStreamSynchronize(c->stream));
    return MLCC_OK;
}

mlcc_status find_critical_curves_impl(Ctx *c, const mlcc_cc_params *p, double *roots_re,
                                      double *roots_im, double *caus_re, double *caus_im,
                                      int32_t *chain_next, mlcc_cc_stats *stats)
{
    const bool mixed = p->precision == MLCC_MIXED;
    const int64_t m = p->m_steps;
    const int n_real = (int)c->reals.size();
    // one field with equal masses: (x, y) records, the mass applied once
    const bool equal = !c->batched && c->equal_mass;
    int S = p->n_subchains;
    if (S <= 0)
        S = autotune_subchains(c->reals, m, mixed, p->predictor,
                               p->star_sums == MLCC_STARS_FMM,
                               p->schedule == MLCC_SCHEDULE_PERSISTENT);
    if ((m / 2) % S) return fail(MLCC_ERR_INVALID, "n_subchains=%d must divide m/2", S);
    // finished rows a warm row needs behind it to be solved by expansions: the
    // centre row in FP64; in the mixed form the two after which rows start with a
    // polish; and two in MLCC_FP64_R32, where one row a front keeps its FP32
    // root-root sums
    const int32_t xfrom =
        p->predictor > 0 && m >= (mixed ? EXP_MIN_STEPS_MIXED : EXP_MIN_STEPS)
            ? (p->precision == MLCC_FP64 ? 1 : 2)
            : 0;
    // Grown pieces of the phase grid: the S subchains, or, where S is the
    // library's choice and rows come from expansions, fewer and longer ones.
    const std::vector<Piece> pieces =
        plan_pieces(c->reals, m, S, p->n_subchains <= 0 && xfrom > 0 && n_real == 1);
    const int NP = (int)pieces.size();
    int64_t L = 0;   // rows of the longest half
    for (const Piece &x : pieces) L = std::max({L, 2 * (x.hi - x.cen), 2 * (x.cen - x.lo)});
    const int max_cold = p->max_iter_cold > 0 ? p->max_iter_cold : 500;
    const int max_warm = p->max_iter_warm > 0 ? p->max_iter_warm : 100;
    constexpr int MAX_BATCH = 256;
    constexpr int KINDS = 3;   // timed kernels per round: FP64 sweep, FP32 sweep, polish

    // fronts, blocks and offsets of every field
    std::vector<Real> rd(n_real);
    std::vector<double> sheet_host;   // rectangular fields' sheet records
    std::vector<Front> fr;
    std::vector<int2> bmap;
    int64_t it_total = 0, bnd_total = 0, max_nr = 0;
    const int32_t warm_phase = mixed ? PH_F32 : PH_F64;
    for (int r = 0; r < n_real; ++r) {
        const RealHost &h = c->reals[r];
        const SheetPoly sp = sheet_poly(h);
        const int64_t n_r = 2 * h.n + sp.n_extra;
        if (n_r > ((int64_t)1 << 30)) return fail(MLCC_ERR_INVALID, "too many roots");
        max_nr = std::max(max_nr, n_r);
        Real &R = rd[r];
        R.star_off = h.star_off;
        R.out_off = (m + 1) * 2 * h.star_off;
        R.bnd_off = bnd_total;
        bnd_total += (int64_t)(NP - 1) * n_r;
        R.n_stars = (int32_t)h.n;
        R.n_r = (int32_t)n_r;
        R.m0 = h.m0;
        R.gamma = h.gamma - sp.d0;   // a rectangular sheet's constant term joins the shear
        R.n_poly = sp.n;
        R.n_extra = sp.n_extra;
        R.sheet_c = sp.seed_r;
        R.sheet_off = (int64_t)sheet_host.size();
        if (sp.n > 0) {
            // d_2k, then the lens-map terms, then the extra roots' start values:
            // evenly spread on the circle through the corners (Sec. 3.2), at
            // angles 2 pi (k + 1/2) / (t - 1)
            sheet_host.insert(sheet_host.end(), sp.d, sp.d + sp.n);
            sheet_host.insert(sheet_host.end(), sp.dmap, sp.dmap + sp.n);
            for (int k = 0; k < sp.n_extra; ++k) {
                const double ang = 2.0 * M_PI * ((double)k + 0.5) / (double)sp.n_extra;
                sheet_host.push_back(sp.seed_r * std::cos(ang));
                sheet_host.push_back(sp.seed_r * std::sin(ang));
            }
        }
        R.a = 1.0 - h.kappa_s;
        R.a1 = std::fabs(R.a);
        R.sz_r = h.sum_z.x;
        R.sz_i = h.sum_z.y;
        R.sz2_r = h.sum_z2.x;
        R.sz2_i = h.sum_z2.y;
        R.M = h.mass_total;
        // rounding of the reference values 2 sum z_i and 2 sum z_i^2 (compensated
        // sums on the host, then the squares and the doubling)
        const double u_ro = 1.1102230246251565e-16;
        R.tol1 = 8.0 * u_ro * h.sum_abs_z;
        R.tol2 = 16.0 * u_ro * h.sum_abs_z2;
        R.root32 = p->precision == MLCC_FP64_R32 ? 1 : 0;
        R.sheet_m = R.sheet_mc = 0.0;   // sum r^2 = 2 sum z_i^2 - 2 (sheet_m + sheet_mc c)
        if (sp.n > 1) R.sheet_m = sp.d[sp.n - 2] / sp.d[sp.n - 1];
        if (sp.n == 1) R.sheet_mc = -1.0 / sp.d[0];
        R.restart = p->cold_restart_sweeps > 0 ? p->cold_restart_sweeps : STALL_START;
        const int bpf = (int)ceil_div(n_r, 64);
        for (int s = 0; s < NP; ++s) {
            const int32_t lo = (int32_t)pieces[s].lo, hi = (int32_t)pieces[s].hi,
                          cen = (int32_t)pieces[s].cen;
            const int fd = (int)fr.size();
            Front d{};
            d.row = cen; d.dir = 0; d.end_row = lo; d.state = FRONT_ACTIVE;
            d.src = fd; d.partner = fd + 1; d.bnd_slot = s >= 1 ? s - 1 : -1;
            d.lo = lo; d.hi = hi;
            d.phase = warm_phase; d.mode = warm_phase; d.stamp = 4 * cen;
            d.best = 0x7fffffff;
            d.real = r;
            d.redo = 1;
            Front u{};
            u.row = cen + 1; u.dir = 1; u.end_row = hi; u.state = FRONT_IDLE;
            u.src = fd + 1; u.partner = -1; u.bnd_slot = -1; u.lo = lo; u.hi = hi;
            u.phase = warm_phase; u.mode = warm_phase; u.stamp = 4 * (cen + 1);
            u.real = r;
            u.redo = 1;
            for (Front *x : {&d, &u}) {
                x->it_off = it_total;
                it_total += n_r;
                x->blk0 = (int32_t)bmap.size();
                const int fi = (int)fr.size();
                for (int q = 0; q < bpf; ++q) bmap.push_back(make_int2(fi, q));
                fr.push_back(*x);
            }
        }
    }
    const int work_waves = plan_workers(rd);
    const int F = (int)fr.size();
    const int64_t nblocks = (int64_t)bmap.size();   // blocks of all fronts, in front order
    if (F > MAX_FRONTS || nblocks > 0x3fffffff)
        return fail(MLCC_ERR_INVALID, "too many fronts (%d) for one call", F);
#if MLCC_XCD_MAP
    // Launch-grid order: work group g runs on XCD g mod 8, so the blocks of
    // one front are all placed at indices of one residue, and each XCD's L2
    // holds the iterates of its own fronts only (fronts go to the least
    // loaded XCD, largest first).  Unused grid slots point at a sentinel
    // front that is never active.
    {
        constexpr int XCDS = 8;
        std::vector<int> byblocks(F);
        for (int f = 0; f < F; ++f) byblocks[f] = f;
        auto nb = [&](int f) { return ceil_div(rd[fr[f].real].n_r, 64); };
        std::stable_sort(byblocks.begin(), byblocks.end(),
                         [&](int a, int b) { return nb(a) > nb(b); });
        std::vector<std::vector<int2>> lists(XCDS);
        std::vector<int64_t> load(XCDS, 0);
        for (int f : byblocks) {
            const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
            for (int64_t q = 0; q < nb(f); ++q) lists[x].push_back(make_int2(f, (int)q));
            load[x] += nb(f);
        }
        const int64_t per = *std::max_element(load.begin(), load.end());
        bmap.assign((size_t)(per * XCDS), make_int2(F, 0));
        for (int x = 0; x < XCDS; ++x)
            for (size_t i = 0; i < lists[x].size(); ++i) bmap[i * XCDS + x] = lists[x][i];
    }
#endif
    const int64_t ngrid = (int64_t)bmap.size();
    {
        Front sentinel{};
        sentinel.state = FRONT_DONE;
        sentinel.dir = 1;
        fr.push_back(sentinel);
    }
    // the control kernel's groups hold whole subchains (two fronts) in LDS
    const int fronts_per_group = 4096;
    const int control_groups = (int)ceil_div(F, fronts_per_group);

    MLCC_TRY(c->iter[0].reserve((size_t)it_total * sizeof(double2)));
    MLCC_TRY(c->iter[1].reserve((size_t)it_total * sizeof(double2)));
    MLCC_TRY(c->flagrow.reserve((size_t)it_total * sizeof(int32_t)));
    MLCC_TRY(c->root_row.reserve((size_t)it_total * sizeof(int32_t)));
    MLCC_TRY(c->fronts.reserve((size_t)(F + 1) * sizeof(Front)));
    MLCC_TRY(c->counts.reserve((size_t)F * sizeof(int32_t)));
    MLCC_TRY(c->passupd.reserve((size_t)F * sizeof(int32_t)));
    MLCC_TRY(c->control.reserve(sizeof(Control)));
    MLCC_TRY(c->fmm_tally.reserve((size_t)FMM_STRIPES * FMM_STRIPE_U64 * sizeof(uint64_t)));
    MLCC_TRY(c->etab.reserve((size_t)(m + 1) * sizeof(double2)));
    MLCC_TRY(c->bnd.reserve((size_t)std::max<int64_t>(bnd_total, 1) * sizeof(double2)));
    MLCC_TRY(c->next_row.reserve((size_t)(2 * nblocks + F) * sizeof(int32_t)));
    if (mixed) {
        MLCC_TRY(c->vieta.reserve((size_t)2 * nblocks * sizeof(double4)));
        MLCC_TRY(c->errbuf.reserve((size_t)it_total * sizeof(double)));
    }
    MLCC_TRY(c->vsum.reserve((size_t)2 * F * sizeof(double4)));
    MLCC_TRY(c->reals_d.reserve((size_t)n_real * sizeof(Real)));
    MLCC_TRY(c->sheet.reserve(std::max<size_t>(1, sheet_host.size()) * sizeof(double)));
    // With multipole sums the kernels take each field's stars in cell order,
    // so that the seeds z_i +- 1 of a work group's roots, and the roots grown
    // from them, share a few cells (and those cells' series) instead of 64.
    std::vector<FmmArgs> fmm_recs;
    const bool fmm_on = p->star_sums == MLCC_STARS_FMM;
    const double2 *stars2 = c->stars.as<double2>();
    const double4 *stars4 = c->stars4.as<double4>();
    if (fmm_on) {
        MLCC_TRY(build_fmm(c, p->fmm_order, equal, fmm_recs));
        stars2 = c->fmm_st2.as<double2>();
        stars4 = c->fmm_st.as<double4>();
    }
    const FmmArgs *fmm_dev = fmm_on ? c->fmm_args.as<FmmArgs>() : nullptr;
    MLCC_TRY(c->bmap.reserve((size_t)ngrid * sizeof(int2)));
    MLCC_TRY(c->workflags.reserve(2 * MAX_BATCH * sizeof(int32_t)));
    MLCC_TRY(ensure_pinned(c, 2 * (sizeof(Control) + MAX_BATCH * sizeof(int32_t))));

    // unit phase table (cos phi_j, -sin phi_j), phi_j = 2 pi j / m (host libm);
    // each field scales it by its own 1 - kappa_s
    std::vector<double2> unit(m + 1);
    for (int64_t j = 0; j <= m; ++j) {
        const double phi = (2.0 * M_PI * (double)j) / (double)m;
        unit[j] = make_double2(std::cos(phi), -std::sin(phi));
    }
    Control ctl0{};
    ctl0.active_fronts = F;
    MLCC_HIP(hipMemcpyAsync(c->etab.p, unit.data(), (m + 1) * sizeof(double2),
                            hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemcpyAsync(c->fronts.p, fr.data(), (F + 1) * sizeof(Front), hipMemcpyHostToDevice,
                            c->stream));
    if (!sheet_host.empty())
        MLCC_HIP(hipMemcpyAsync(c->sheet.p, sheet_host.data(), sheet_host.size() * sizeof(double),
                                hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemcpyAsync(c->reals_d.p, rd.data(), n_real * sizeof(Real), hipMemcpyHostToDevice,
                            c->stream));
    MLCC_HIP(hipMemcpyAsync(c->bmap.p, bmap.data(), ngrid * sizeof(int2), hipMemcpyHostToDevice,
                            c->stream));
    MLCC_HIP(hipMemcpyAsync(c->control.p, &ctl0, sizeof ctl0, hipMemcpyHostToDevice, c->stream));
    MLCC_HIP(hipMemsetAsync(c->flagrow.p, 0xff, (size_t)it_total * sizeof(int32_t), c->stream));
    MLCC_HIP(hipMemsetAsync(c->counts.p, 0, F * sizeof(int32_t), c->stream));
    MLCC_HIP(hipMemsetAsync(c->fmm_tally.p, 0,
                            (size_t)FMM_STRIPES * FMM_STRIPE_U64 * sizeof(uint64_t), c->stream));
    MLCC_HIP(hipMemsetAsync(c->passupd.p, 0, F * sizeof(int32_t), c->stream));
    int32_t *const bad_row = c->next_row.as<int32_t>() + 2 * nblocks;
    if (xfrom > 0) MLCC_HIP(hipMemsetAsync(bad_row, 0x7f, F * sizeof(int32_t), c->stream));
    const int32_t near_seeds = p->n_subchains <= 0 && xfrom > 0;
    if (equal)
        hipLaunchKernelGGL(seed_centres<double2>, dim3((unsigned)ngrid), dim3(64), 0, c->stream,
                           stars2, c->reals_d.as<Real>(), c->fronts.as<Front>(),
                           c->bmap.as<int2>(), c->sheet.as<double>(), c->iter[0].as<double2>(),
                           near_seeds, m);
    else
        hipLaunchKernelGGL(seed_centres<double4>, dim3((unsigned)ngrid), dim3(64), 0, c->stream,
                           stars4, c->reals_d.as<Real>(), c->fronts.as<Front>(),
                           c->bmap.as<int2>(), c->sheet.as<double>(), c->iter[0].as<double2>(),
                           near_seeds, m);
    MLCC_HIP(hipGetLastError());
    // Host copies must finish before the vectors above go out of scope.
    MLCC_HIP(hipStreamSynchronize(c->stream));
    // The rounds run on the caller's stream, or, when that is the legacy null
    // stream (which cannot be captured into a graph), on a stream of the
    // context's own; the call is synchronous either way.
    hipStream_t rs = c->stream;
    if (!rs) {
        if (!c->own_stream) MLCC_HIP(hipStreamCreateWithFlags(&c->own_stream, hipStreamNonBlocking));
        rs = c->own_stream;
    }

    RoundArgs<double2> A2{};
    RoundArgs<double4> A4{};
    auto fill = [&](auto &A, auto stars, const double2 *cur, double2 *nxt) {
        A.stars = stars;
        A.reals = c->reals_d.as<Real>();
        A.bmap = c->bmap.as<int2>();
        A.fronts = c->fronts.as<Front>();
        A.flagrow = c->flagrow.as<int32_t>();
        A.root_row = c->root_row.as<int32_t>();
        A.cur = cur;
        A.nxt = nxt;
        A.unit = c->etab.as<double2>();
        A.tol_step = p->tol_step;
        A.tol_step2 = p->tol_step * p->tol_step;
        A.tol_mu = p->tol_inv_mu;
        A.out_re = roots_re;
        A.out_im = roots_im;
        A.caus_re = caus_re;
        A.caus_im = caus_im;
        A.bnd = c->bnd.as<double2>();
        A.counts = c->counts.as<int32_t>();
        A.passupd = c->passupd.as<int32_t>();
        A.ctl = c->control.as<Control>();
        A.fmm_tally = c->fmm_tally.as<unsigned long long>();
        A.vieta = c->vieta.as<double4>();
        A.predictor = p->predictor;
        A.errbuf = mixed ? c->errbuf.as<double>() : nullptr;
        A.xfrom = xfrom;
        A.next_row = c->next_row.as<int32_t>();
        A.stuck = c->next_row.as<int32_t>() + nblocks;
        A.persistent = p->schedule == MLCC_SCHEDULE_PERSISTENT;
        A.iter0 = c->iter[0].as<double2>();
        A.iter1 = c->iter[1].as<double2>();
        A.sheet = c->sheet.as<double>();
        A.fmm = fmm_dev;
    };
    const dim3 grid((unsigned)ngrid);
    auto launch_kind = [&](int kind, const double2 *cur, double2 *nxt) {
        // each kernel comes with and without multipole sums, so that the
        // direct kernels carry none of the multipole code's registers
        auto go = [&](auto &A, auto eq, auto fm) {
            constexpr bool E = decltype(eq)::value, M = decltype(fm)::value;
            if (kind == 0) hipLaunchKernelGGL((aberth_sweep_f64<E, M>), grid, dim3(64), 0, rs, A);
            if (kind == 1) hipLaunchKernelGGL((aberth_sweep_f32<E, M>), grid, dim3(64), 0, rs, A);
            if (kind == 2) hipLaunchKernelGGL((newton_polish_f64<E, M>), grid, dim3(64), 0, rs, A);
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        if (equal) {
            fill(A2, stars2, cur, nxt);
            if (fmm_on) go(A2, T_{}, T_{}); else go(A2, T_{}, F_{});
        } else {
            fill(A4, stars4, cur, nxt);
            if (fmm_on) go(A4, F_{}, T_{}); else go(A4, F_{}, F_{});
        }
    };

    Control *dctl = c->control.as<Control>();
    char *pin = static_cast<char *>(c->pinned);
    auto pin_ctl = [&](int slot) {
        return reinterpret_cast<Control *>(pin + slot * (sizeof(Control) + MAX_BATCH * 4));
    };
    auto pin_flags = [&](int slot) {
        return reinterpret_cast<int32_t *>(pin + slot * (sizeof(Control) + MAX_BATCH * 4) +
                                           sizeof(Control));
    };

    // event pairs: [slot][round][kind][begin, end]
    std::vector<hipEvent_t> evs;
    auto ev = [&](int slot, int i, int kind, int end) -> hipEvent_t & {
        return evs[(((size_t)slot * MAX_BATCH + i) * KINDS + kind) * 2 + end];
    };
    if (p->timing) {
        evs.resize((size_t)2 * MAX_BATCH * KINDS * 2);
        for (auto &e : evs) MLCC_HIP(hipEventCreate(&e));
    }
    hipEvent_t done_ev[2];
    MLCC_HIP(hipEventCreateWithFlags(&done_ev[0], hipEventDisableTiming));
    MLCC_HIP(hipEventCreateWithFlags(&done_ev[1], hipEventDisableTiming));
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    int graph_len = 0;
    auto cleanup = [&]() {
        for (auto &e : evs) (void)hipEventDestroy(e);
        evs.clear();
        for (auto &g : gexec)
            if (g) (void)hipGraphExecDestroy(g);
        (void)hipEventDestroy(done_ev[0]);
        (void)hipEventDestroy(done_ev[1]);
    };

    const bool persistent = p->schedule == MLCC_SCHEDULE_PERSISTENT;
    const bool use_graphs = !p->timing && !persistent;
    int parity = 0;
    int batch_len[2] = {0, 0};
    int G = 4;
    double kind_ms[KINDS] = {0.0, 0.0, 0.0};
    int64_t kind_launches[KINDS] = {0, 0, 0};
    double persistent_ms = 0.0;
    int64_t persistent_launches = 0;
    int32_t polls = 0;
    // Every front finishes within max_cold + (L/2 + 1) * (max_warm + polish
    // rounds) rounds; the extra margin covers the batches enqueued ahead of
    // the last poll.
    const int64_t launch_cap =
        (int64_t)max_cold + (L / 2 + 2) * (int64_t)(max_warm + MAX_POLISH + 2) + 4 * MAX_BATCH;
    int64_t launched = 0;
    int rounds_runs = 0;   // the first run of rounds (the cold starts) is replayed from graphs
    // One round: every pass kind once over every block (blocks whose front is
    // in another phase return at once), then the control kernel.
    auto enqueue_rounds = [&](int slot, int g, bool timed) -> mlcc_status {
        for (int i = 0; i < g; ++i) {
            const double2 *cur = c->iter[parity].as<double2>();
            double2 *nxt = c->iter[parity ^ 1].as<double2>();
            for (int kind = 0; kind < (mixed ? KINDS : 1); ++kind) {
                if (timed) MLCC_HIP(hipEventRecord(ev(slot, i, kind, 0), rs));
                launch_kind(kind, cur, nxt);
                if (timed) MLCC_HIP(hipEventRecord(ev(slot, i, kind, 1), rs));
                if (kind == 2)
                    hipLaunchKernelGGL(row_sums, dim3((unsigned)F), dim3(64), 0, rs,
                                       c->fronts.as<Front>(), c->reals_d.as<Real>(),
                                       c->vieta.as<double4>(), c->vsum.as<double4>());
            }
            int32_t *wf = c->workflags.as<int32_t>() + slot * MAX_BATCH + i;
            hipLaunchKernelGGL(control_begin, dim3(1), dim3(64), 0, rs, dctl, wf);
            hipLaunchKernelGGL(aberth_control, dim3(control_groups), dim3(CONTROL_THREADS), 0,
                               rs, c->fronts.as<Front>(), c->counts.as<int32_t>(), F, dctl,
                               max_cold, max_warm, wf, c->vsum.as<double4>(),
                               c->reals_d.as<Real>(), c->etab.as<double2>(), fronts_per_group,
                               p->predictor, c->passupd.as<int32_t>(), max_polish_passes(fmm_on), xfrom);
            hipLaunchKernelGGL(control_end, dim3(1), dim3(64), 0, rs, dctl, wf);
            parity ^= 1;
        }
        MLCC_HIP(hipGetLastError());
        MLCC_HIP(hipMemcpyAsync(pin_ctl(slot), dctl, sizeof(Control), hipMemcpyDeviceToHost,
                                rs));
        MLCC_HIP(hipMemcpyAsync(pin_flags(slot), c->workflags.as<int32_t>() + slot * MAX_BATCH,
                                g * sizeof(int32_t), hipMemcpyDeviceToHost, rs));
        return MLCC_OK;
    };
    auto enqueue_batch = [&](int slot, int g) -> mlcc_status {
        if (gexec[slot] && rounds_runs == 0) {
            MLCC_HIP(hipGraphLaunch(gexec[slot], rs));
            g = graph_len;
        } else {
            MLCC_TRY(enqueue_rounds(slot, g, p->timing != 0));
        }
        MLCC_HIP(hipEventRecord(done_ev[slot], rs));
        batch_len[slot] = g;
        launched += g;
        return MLCC_OK;
    };
    // Without per-kernel timing the rounds of a batch are captured once per
    // slot into a hipGraph (an even number of rounds, so the ping-pong buffers
    // line up) and replayed until the fronts are done.
    auto build_graphs = [&](int g) -> mlcc_status {
        g = std::max(2, g & ~1);
        for (int slot = 0; slot < 2; ++slot) {
            hipGraph_t graph = nullptr;
            const int saved = parity;
            parity = 0;
            MLCC_HIP(hipStreamBeginCapture(rs, hipStreamCaptureModeThreadLocal));
            mlcc_status s = enqueue_rounds(slot, g, false);
            hipError_t e = hipStreamEndCapture(rs, &graph);
            parity = saved;
            if (s != MLCC_OK) {
                if (graph) (void)hipGraphDestroy(graph);
                return s;
            }
            MLCC_HIP(e);
            e = hipGraphInstantiate(&gexec[slot], graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            MLCC_HIP(e);
        }
        graph_len = g;
        return MLCC_OK;
    };
    auto harvest = [&](int slot) {
        // live bits per round: 1 << phase of every front that was active
        const int kind_phase[KINDS] = {PH_F64, PH_F32, PH_POLISH};
        for (int i = 0; i < batch_len[slot]; ++i) {
            const int32_t live = pin_flags(slot)[i];
            for (int kind = 0; kind < KINDS; ++kind) {
                if (!(live & (1 << kind_phase[kind]))) continue;
                kind_launches[kind] += 1;
                if (p->timing && !gexec[slot]) {
                    float ms = 0.f;
                    (void)hipEventElapsedTime(&ms, ev(slot, i, kind, 0), ev(slot, i, kind, 1));
                    kind_ms[kind] += ms;
                }
            }
        }
    };

    // The persistent scheduler: one launch at a time, fronts advance independently.
    PQueue *dq = nullptr;
    int2 *dtasks = nullptr;
    unsigned long long *dseq = nullptr;
    unsigned long long qmask = 0;
    hipGraphExec_t pgraph = nullptr;
    auto setup_persistent = [&]() -> mlcc_status {
        int cus = 0, clock_khz = 0;
        MLCC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device));
        MLCC_HIP(hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, c->device));
        if (cus < 1 || clock_khz < 1) return fail(MLCC_ERR_HIP, "cannot size the persistent launch");
        int64_t ntasks = 0;
        for (int f = 0; f < F; ++f) {
            const Real &R = rd[fr[f].real];
            ntasks += ceil_div(ceil_div(R.n_r, 64), R.chunk);
        }
        int64_t cap = 1024;
        while (cap < 2 * ntasks) cap <<= 1;
        const size_t o_tasks = (sizeof(PQueue) + 255) & ~(size_t)255;
        const size_t o_seq = o_tasks + (size_t)cap * sizeof(int2);
        const size_t o_fdone = o_seq + (size_t)cap * SEQ_STRIDE * sizeof(unsigned long long);
        const size_t pq_bytes = o_fdone + (size_t)F * sizeof(int32_t);
        MLCC_TRY(c->pq.reserve(pq_bytes));
        char *base = static_cast<char *>(c->pq.p);
        dq = reinterpret_cast<PQueue *>(base);
        dtasks = reinterpret_cast<int2 *>(base + o_tasks);
        dseq = reinterpret_cast<unsigned long long *>(base + o_seq);
        qmask = (unsigned long long)(cap - 1);
        int32_t *dfdone = reinterpret_cast<int32_t *>(base + o_fdone);
        std::vector<int2> t0;
        for (int f = 0; f < F; ++f) {
            if (fr[f].state != FRONT_ACTIVE) continue;
            const Real &R = rd[fr[f].real];
            for (int64_t qb = 0; qb < ceil_div(ceil_div(R.n_r, 64), R.chunk); ++qb)
                t0.push_back(make_int2(f, (int)qb));
        }
        std::vector<unsigned long long> s0(t0.size() * SEQ_STRIDE, 0ull);
        for (size_t i = 0; i < t0.size(); ++i) s0[i * SEQ_STRIDE] = i + 1;
        PQueue hq{};
        hq.tail = (unsigned long long)t0.size();
        hq.target = F;
        MLCC_HIP(hipMemsetAsync(base, 0, pq_bytes, rs));
        MLCC_HIP(hipMemcpyAsync(dq, &hq, sizeof hq, hipMemcpyHostToDevice, rs));
        MLCC_HIP(hipMemcpyAsync(dtasks, t0.data(), t0.size() * sizeof(int2), hipMemcpyHostToDevice,
                                rs));
        MLCC_HIP(hipMemcpyAsync(dseq, s0.data(), s0.size() * sizeof(unsigned long long),
                                hipMemcpyHostToDevice, rs));
        const void *kfn =
            equal ? (fmm_on ? reinterpret_cast<const void *>(&aberth_persistent<true, true>)
                            : reinterpret_cast<const void *>(&aberth_persistent<true, false>))
                  : (fmm_on ? reinterpret_cast<const void *>(&aberth_persistent<false, true>)
                            : reinterpret_cast<const void *>(&aberth_persistent<false, false>));
        const unsigned threads = 64u * (unsigned)work_waves;
        const size_t lds = (size_t)work_waves * 128 * (equal ? sizeof(double2) : sizeof(double4));
        if (lds + sizeof(WorkShare) > 65536)
            MLCC_HIP(hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        int per_cu = 0;
        MLCC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, (int)threads, lds));
        if (per_cu < 1) return fail(MLCC_ERR_HIP, "cannot size the persistent launch");
        // as many workers as fit, but hardly more than there are tasks at a time
        // (the few beyond them watch for a stall)
        const unsigned workers =
            (unsigned)std::min<int64_t>((int64_t)cus * per_cu, ntasks + WATCHERS);
        // a worker gives up after watchdog_ms (default 5 s) in which no pass
        // finished anywhere
        const unsigned long long stall =
            (unsigned long long)clock_khz * (unsigned long long)(p->watchdog_ms > 0 ? p->watchdog_ms : 5000);
        const double2 *cur0 = c->iter[0].as<double2>();
        // The one launch is captured into a hipGraph (a single kernel node; the
        // queue and counters above are set by copies outside it) and run from
        // the graph.
        auto launch = [&]() {
            if (equal) {
                fill(A2, stars2, cur0, c->iter[1].as<double2>());
                if (fmm_on)
                    hipLaunchKernelGGL((aberth_persistent<true, true>), dim3(workers), dim3(threads), lds,
                                       rs, A2, c->fronts.as<Front>(), dq, dtasks, dseq,
                                       (unsigned long long)(cap - 1), dfdone, max_cold, max_warm,
                                       stall);
                else
                    hipLaunchKernelGGL((aberth_persistent<true, false>), dim3(workers), dim3(threads), lds,
                                       rs, A2, c->fronts.as<Front>(), dq, dtasks, dseq,
                                       (unsigned long long)(cap - 1), dfdone, max_cold, max_warm,
                                       stall);
            } else {
                fill(A4, stars4, cur0, c->iter[1].as<double2>());
                if (fmm_on)
                    hipLaunchKernelGGL((aberth_persistent<false, true>), dim3(workers), dim3(threads), lds,
                                       rs, A4, c->fronts.as<Front>(), dq, dtasks, dseq,
                                       (unsigned long long)(cap - 1), dfdone, max_cold, max_warm,
                                       stall);
                else
                    hipLaunchKernelGGL((aberth_persistent<false, false>), dim3(workers), dim3(threads), lds,
                                       rs, A4, c->fronts.as<Front>(), dq, dtasks, dseq,
                                       (unsigned long long)(cap - 1), dfdone, max_cold, max_warm,
                                       stall);
            }
        };
        hipGraph_t graph = nullptr;
        MLCC_HIP(hipStreamBeginCapture(rs, hipStreamCaptureModeThreadLocal));
        launch();
        const hipError_t le = hipGetLastError();
        hipError_t e = hipStreamEndCapture(rs, &graph);
        if (le != hipSuccess || e != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            MLCC_HIP(le);
            MLCC_HIP(e);
        }
        e = hipGraphInstantiate(&pgraph, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        MLCC_HIP(e);
        // host vectors must outlive the copies above
        MLCC_HIP(hipStreamSynchronize(rs));
        return MLCC_OK;
    };
    auto run_persistent = [&]() -> mlcc_status {
        MLCC_HIP(hipGraphLaunch(pgraph, rs));
        PQueue *hq = static_cast<PQueue *>(c->pinned);
        MLCC_HIP(hipMemcpyAsync(hq, dq, sizeof *hq, hipMemcpyDeviceToHost, rs));
        MLCC_HIP(hipStreamSynchronize(rs));
        if (hq->abort)
            return fail(MLCC_ERR_HIP, "persistent scheduler: no pass finished for %d ms "
                                      "(%d of %d fronts done)",
                        p->watchdog_ms > 0 ? p->watchdog_ms : 5000, hq->done, hq->target);
        return MLCC_OK;
    };

    // expand_check: a wave a row while a lane then has few reads, else a work group
    // of four.  As many as are resident at once, or, as later launches find all
    // their rows in a few fronts, one for every eight rows a front may have (40
    // fields 1.9 -> 0.8 ms a call, 97 small ones 1.3 -> 0.6).
    const unsigned check_threads = max_nr > 4096 ? CONTROL_THREADS : 64;
    const int64_t resident = 8192 * 64 / check_threads, front_rows = L / 2 + 1;
    const unsigned check_groups = (unsigned)std::max<int64_t>(
        1, std::min(front_rows, std::max(resident / F, std::min(ceil_div(front_rows, 8), 8 * resident / F))));
    // The expansions over every parked front, and what comes of them: fronts
    // that passes take over, and fronts still parked.
    auto run_expansions = [&](int &active, int &parked) -> mlcc_status {
        hipLaunchKernelGGL(expand_begin, dim3(1), dim3(1), 0, rs, dctl, dq);
        auto go = [&](auto &A, auto eq, auto fm) {
            constexpr bool E = decltype(eq)::value, M = decltype(fm)::value;
            if (mixed) hipLaunchKernelGGL((expand_rows<E, M, true>), grid, dim3(64), 0, rs, A);
            else hipLaunchKernelGGL((expand_rows<E, M, false>), grid, dim3(64), 0, rs, A);
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        if (equal) {
            fill(A2, stars2, c->iter[0].as<double2>(), c->iter[1].as<double2>());
            if (fmm_on) go(A2, T_{}, T_{}); else go(A2, T_{}, F_{});
        } else {
            fill(A4, stars4, c->iter[0].as<double2>(), c->iter[1].as<double2>());
            if (fmm_on) go(A4, F_{}, T_{}); else go(A4, F_{}, F_{});
        }
        hipLaunchKernelGGL(expand_check, dim3((unsigned)F, check_groups), dim3(check_threads), 0, rs,
                           c->fronts.as<Front>(), c->reals_d.as<Real>(), c->etab.as<double2>(),
                           c->next_row.as<int32_t>(), roots_re, roots_im, c->bnd.as<double2>(),
                           bad_row);
        hipLaunchKernelGGL(expand_control, dim3((unsigned)F), dim3(64), 0, rs,
                           c->fronts.as<Front>(), c->reals_d.as<Real>(), c->next_row.as<int32_t>(),
                           c->next_row.as<int32_t>() + nblocks, p->predictor, xfrom, bad_row,
                           dctl, dq, dtasks, dseq, qmask);
        hipLaunchKernelGGL(expand_gather, grid, dim3(64), 0, rs, c->fronts.as<Front>(),
                           c->reals_d.as<Real>(), c->bmap.as<int2>(), c->next_row.as<int32_t>(),
                           roots_re, roots_im, c->bnd.as<double2>(), c->iter[0].as<double2>(),
                           c->iter[1].as<double2>(), c->flagrow.as<int32_t>(),
                           mixed ? c->errbuf.as<double>() : nullptr, dctl);
        MLCC_HIP(hipGetLastError());
        Control *h = static_cast<Control *>(c->pinned);
        MLCC_HIP(hipMemcpyAsync(h, dctl, sizeof *h, hipMemcpyDeviceToHost, rs));
        MLCC_HIP(hipStreamSynchronize(rs));
        active = h->active_fronts;
        parked = h->parked_fronts;
        return MLCC_OK;
    };

    // Rounds between two runs of the expansions: few fronts are active, and their
    // open roots settle in about as many rounds as the last time.  That many are
    // sent and waited for, then two at a time; none is queued ahead, as a round
    // that finds nothing to do costs as much as a wait (15 to 20 us).  With the
    // batches of a first run, which grow to 4 ms of rounds, most rounds here were
    // empty (400 steps, FP64: N = 700 9.3 -> 4.6 ms a call, a rectangular field of 40
    // stars 6.8 -> 3.7, 200 fields of 50 17.0 -> 10.0).
    int again = 2;
    auto run_few_rounds = [&]() -> mlcc_status {
        int live = 0;
        launched = 0;
        for (int g = again;; g = 2) {
            MLCC_TRY(enqueue_batch(0, g));
            MLCC_HIP(hipEventSynchronize(done_ev[0]));
            ++polls;
            harvest(0);
            for (int i = 0; i < g; ++i) live += pin_flags(0)[i] != 0;
            if (pin_ctl(0)->active_fronts == 0) break;
            if (launched > launch_cap)
                return fail(MLCC_ERR_HIP, "root finder exceeded %lld rounds", (long long)launch_cap);
        }
        again = std::min(16, std::max(2, (live + 1) & ~1));   // even: see below
        return MLCC_OK;
    };

    // The round schedule: rounds until no front is active.
    auto run_rounds = [&]() -> mlcc_status {
        if (rounds_runs > 0) return run_few_rounds();
        mlcc_status st = MLCC_OK;
        int slot = 0;
        launched = 0;
        G = 4;
        auto t_last = std::chrono::steady_clock::now();
        st = enqueue_batch(slot, G);
        while (st == MLCC_OK) {
            // keep one batch queued behind the one being polled
            const int next = slot ^ 1;
            if (use_graphs && !gexec[0] && polls == 1 && parity == 0) {
                // G now holds the batch length that takes ~4 ms
                st = build_graphs(std::min(G, 64));
                if (st != MLCC_OK) break;
            }
            st = enqueue_batch(next, G);
            if (st != MLCC_OK) break;
            if (hipEventSynchronize(done_ev[slot]) != hipSuccess) {
                st = fail(MLCC_ERR_HIP, "sweep batch failed: %s",
                          hipGetErrorString(hipGetLastError()));
                break;
            }
            ++polls;
            const Control h = *pin_ctl(slot);
            harvest(slot);
            if (h.active_fronts == 0) {
                // drain the batch queued ahead (it found nothing to do)
                if (hipEventSynchronize(done_ev[next]) != hipSuccess) {
                    st = fail(MLCC_ERR_HIP, "sweep batch failed");
                    break;
                }
                harvest(next);
                break;
            }
            if (launched > launch_cap) {
                st = fail(MLCC_ERR_HIP, "root finder exceeded %lld rounds", (long long)launch_cap);
                break;
            }
            // poll roughly every 4 ms of GPU work
            auto now = std::chrono::steady_clock::now();
            const double dt = std::chrono::duration<double, std::milli>(now - t_last).count();
            t_last = now;
            const double per = dt / std::max(1, batch_len[slot]);
            G = (int)std::min<double>(MAX_BATCH, std::max<double>(2.0, 4.0 / std::max(per, 1e-3)));
            G &= ~1;   // even batches keep the ping-pong parity at 0 between batches
            slot = next;
        }
        ++rounds_runs;
        return st;
    };

    // Passes (cold starts, the rows next to them, roots the expansions left
    // open) and expansions in turn until every front is done.
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (persistent && p->timing) {
        MLCC_HIP(hipEventCreate(&e0));
        MLCC_HIP(hipEventCreate(&e1));
    }
    mlcc_status st = persistent ? setup_persistent() : MLCC_OK;
    if (st == MLCC_OK && e0) (void)hipEventRecord(e0, rs);
    int active = F, parked = 0;
    while (st == MLCC_OK) {
        if (active > 0) st = persistent ? run_persistent() : run_rounds();
        if (st != MLCC_OK || xfrom == 0) break;
        st = run_expansions(active, parked);
        if (active == 0 && parked == 0) break;
    }
    if (e0) {
        float ms = 0.f;
        (void)hipEventRecord(e1, rs);
        (void)hipEventSynchronize(e1);
        (void)hipEventElapsedTime(&ms, e0, e1);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        persistent_ms = ms;
    }
    if (persistent) persistent_launches = 1;
    if (pgraph) (void)hipGraphExecDestroy(pgraph);
    (void)hipStreamSynchronize(rs);
    cleanup();
    if (st != MLCC_OK) return st;

    Control h{};
    MLCC_HIP(hipMemcpyAsync(&h, dctl, sizeof h, hipMemcpyDeviceToHost, c->stream));
    std::vector<uint64_t> tally((size_t)FMM_STRIPES * FMM_STRIPE_U64);
    MLCC_HIP(hipMemcpyAsync(tally.data(), c->fmm_tally.p, tally.size() * sizeof(uint64_t),
                            hipMemcpyDeviceToHost, c->stream));
    std::vector<Front> fin(F);
    MLCC_HIP(hipMemcpyAsync(fin.data(), c->fronts.p, F * sizeof(Front), hipMemcpyDeviceToHost,
                            c->stream));
    MLCC_HIP(hipStreamSynchronize(c->stream));
    // the multipole tallies, summed over their copies
    uint64_t ft[FMM_T_ALL] = {};
    for (int q = 0; q < FMM_STRIPES; ++q)
        for (int v = 0; v < FMM_T_ALL; ++v) ft[v] += tally[(size_t)q * FMM_STRIPE_U64 + v];
    const uint64_t fmm_near = ft[FMM_T_F64], fmm_far[2] = {ft[FMM_T_F64 + 1], ft[FMM_T_F64 + 2]};
    const uint64_t fmm_near_polish = ft[FMM_T_POLISH],
                   fmm_far_polish[2] = {ft[FMM_T_POLISH + 1], ft[FMM_T_POLISH + 2]};
    const uint64_t fmm_near_f32 = ft[FMM_T_F32],
                   fmm_far_f32[2] = {ft[FMM_T_F32 + 1], ft[FMM_T_F32 + 2]};
    const uint64_t fmm_near_exp = ft[FMM_T_EXP + EXP_NEAR];

    mlcc_status result = MLCC_OK;
    double maxdist = 0.0;
    if (h.failed_rows > 0) {
        result = fail(MLCC_ERR_NOT_CONVERGED, "%d rows hit the sweep cap (%lld roots unconverged)",
                      h.failed_rows, (long long)h.unconverged);
    } else {
        // join subchains: pair each duplicate boundary row with the stored
        // copy, compose the pairings into global labels, relabel the blocks;
        // then pair row m with row 0 for chain_next
        std::vector<PairJob> jobs;
        int64_t perm_total = 0;
        for (int r = 0; r < n_real; ++r) perm_total += (int64_t)NP * rd[r].n_r;
        MLCC_TRY(c->perm.reserve((size_t)std::max<int64_t>(perm_total, 1) * sizeof(int32_t)));
        int32_t *perm = c->perm.as<int32_t>();
        std::vector<int64_t> perm_off(n_real);
        int64_t po = 0;
        for (int r = 0; r < n_real; ++r) {
            perm_off[r] = po;
            const int64_t n_r = rd[r].n_r;
            double *ore = roots_re + rd[r].out_off, *oim = roots_im + rd[r].out_off;
            for (int s = 1; s < NP; ++s) {
                PairJob j{};
                j.a2 = c->bnd.as<double2>() + rd[r].bnd_off + (int64_t)(s - 1) * n_r;
                j.b_re = ore + pieces[s].lo * n_r;
                j.b_im = oim + pieces[s].lo * n_r;
                j.perm = perm + po + s * n_r;
                j.n = n_r;
                jobs.push_back(j);
            }
            po += (int64_t)NP * n_r;
        }
        double md = 0.0;
        MLCC_TRY(pair_all(c, jobs, 1e-6, &md));
        maxdist = std::max(maxdist, md);
        if (NP > 1) {
            std::vector<int32_t> hp((size_t)perm_total), lab((size_t)perm_total);
            MLCC_HIP(hipMemcpyAsync(hp.data(), perm, (size_t)perm_total * sizeof(int32_t),
                                    hipMemcpyDeviceToHost, c->stream));
            MLCC_HIP(hipStreamSynchronize(c->stream));
            for (int r = 0; r < n_real; ++r) {
                const int64_t n_r = rd[r].n_r, b = perm_off[r];
                for (int64_t k = 0; k < n_r; ++k) lab[b + k] = (int32_t)k;
                for (int s = 1; s < NP; ++s)
                    for (int64_t k = 0; k < n_r; ++k)
                        lab[b + s * n_r + k] = lab[b + (s - 1) * n_r + hp[b + s * n_r + k]];
            }
            MLCC_HIP(hipMemcpyAsync(perm, lab.data(), (size_t)perm_total * sizeof(int32_t),
                                    hipMemcpyHostToDevice, c->stream));
            std::vector<RelabelJob> rj;
            for (int r = 0; r < n_real; ++r) {
                const int64_t n_r = rd[r].n_r;
                for (int s = 1; s < NP; ++s) {
                    const int32_t *lb = perm + perm_off[r] + s * n_r;
                    rj.push_back(RelabelJob{roots_re + rd[r].out_off, roots_im + rd[r].out_off,
                                            n_r, pieces[s].lo + 1, pieces[s].hi + 1, lb});
                    if (caus_re)
                        rj.push_back(RelabelJob{caus_re + rd[r].out_off, caus_im + rd[r].out_off,
                                                n_r, pieces[s].lo + 1, pieces[s].hi + 1, lb});
                }
            }
            MLCC_TRY(relabel_all(c, rj));
            MLCC_HIP(hipStreamSynchronize(c->stream));
        }
        if (chain_next) {
            jobs.clear();
            for (int r = 0; r < n_real; ++r) {
                const int64_t n_r = rd[r].n_r;
                double *ore = roots_re + rd[r].out_off, *oim = roots_im + rd[r].out_off;
                PairJob j{};
                j.a_re = ore + m * n_r;
                j.a_im = oim + m * n_r;
                j.b_re = ore;
                j.b_im = oim;
                j.perm = chain_next + 2 * c->reals[r].star_off;
                j.n = n_r;
                jobs.push_back(j);
            }
            MLCC_TRY(pair_all(c, jobs, 1e-6, &md));
            maxdist = std::max(maxdist, md);
        }
        MLCC_HIP(hipStreamSynchronize(c->stream));
    }

    if (stats) {
        *stats = mlcc_cc_stats{};
        if (persistent) {   // no global rounds: the longest chain of passes of one front
            int64_t mp = 0;
            for (const Front &x : fin) mp = std::max<int64_t>(mp, x.npass);
            stats->sweeps = mp;
        } else {
            stats->sweeps = h.live_sweeps;
        }
        stats->root_updates = (int64_t)(h.upd[PH_F64] + h.upd[TALLY_ROOTS]);
        stats->root_updates_f32 = (int64_t)h.upd[PH_F32];
        stats->polish_updates = (int64_t)(h.upd[PH_POLISH] + h.upd[TALLY_ROOTS + 1]);
        stats->unconverged = h.unconverged;
        stats->rows_capped = h.failed_rows;
        stats->cold_restarts = h.cold_restarts;
        stats->rows_fallback = h.rows_fallback;
        stats->n_subchains = S;
        int32_t mw = 0, mc = 0;
        for (const Front &x : fin) {
            mw = std::max(mw, x.max_warm);
            mc = std::max(mc, x.cold);
        }
        stats->max_row_sweeps = mw;
        stats->cold_sweeps = mc;
        stats->polls = polls;
        stats->match_maxdist = maxdist;
        stats->sweep_ms = kind_ms[0];
        stats->sweep_f32_ms = kind_ms[1];
        stats->polish_ms = kind_ms[2];
        stats->sweep_launches = kind_launches[0];
        stats->sweep_f32_launches = kind_launches[1];
        stats->polish_launches = kind_launches[2];
        stats->persistent_ms = persistent_ms;
        stats->persistent_launches = persistent_launches;
        // algorithmic FLOP of one update of a root of a field of N stars
        // (FMA = 2, add/mul/reciprocal = 1): 29 per star term (difference,
        // |d|^2, reciprocal, u, u^2, u^3 and their sums) and 10 per root
        // term, 29 N + 10 (2N - 1) for an Aberth update, 29 N for a polish
        // update (star terms only); the device counts updates and
        // updates x N, which gives the sums over mixed field sizes
        // star terms in FP64; root terms in FP64 except in fast-root passes
        // With fast-multipole star sums (one field), an update that took
        // them has its near stars' terms at 29 FLOP each and one evaluation
        // of the cell's series of order p in place of the other N - near
        // terms: Horner's rule for f, f' and f'' together takes 26 FLOP per
        // order (the unit-weight series of unequal masses 8 more in the
        // sweeps), plus ~20 for the cell and the sums.  The outside-grid
        // expansion, rarely taken, is counted the same.
        // The FP32 sweeps take such sums in FP64: their star terms move from
        // the FP32 count to the FP64 one.
        double star64 = (double)h.star[PH_F64], starpol = (double)h.star[PH_POLISH];
        double far64 = 0.0, farpol = 0.0, star32_off = 0.0;
        if (fmm_on) {
            const double pf = (double)fmm_recs[0].p;
            const double unit_g = equal ? 0.0 : 8.0 * pf;
            far64 = (double)fmm_far[0] * (26.0 * pf + 20.0 + unit_g) +
                    (double)fmm_far_f32[0] * (26.0 * pf + 20.0 + unit_g) +
                    29.0 * (double)fmm_near_f32;
            farpol = (double)fmm_far_polish[0] * (26.0 * pf + 20.0);
            star64 += (double)fmm_near - (double)fmm_far[1];
            starpol += (double)fmm_near_polish - (double)fmm_far_polish[1];
            star32_off = 29.0 * (double)fmm_far_f32[1];
            stats->fmm_near_terms =
                (int64_t)(fmm_near + fmm_near_polish + fmm_near_f32 + fmm_near_exp);
            stats->fmm_far_evals = (int64_t)(fmm_far[0] + fmm_far_polish[0] + fmm_far_f32[0] +
                                             ft[FMM_T_EXP + EXP_FORMED]);
        }
        // Updates from expansions: a step is Horner's rule for f and three
        // derivatives (32 FLOP per moment) and the step itself; an expansion
        // MOMENT_FLOP per star term, or per near star and 8 M per order of the
        // cell's series.
        constexpr double STEP_FLOP = 32.0 * NMOM + 60.0;
        constexpr double MOMENT_FLOP = 6.0 + 28.0 + 9.0 * (NMOM - 3);
        static_assert(NMOM != 14 || (STEP_FLOP == 508.0 && MOMENT_FLOP == 133.0), "as in mlcc.h");
        const uint64_t *fx = ft + FMM_T_EXP;
        const double sums = fmm_on ? MOMENT_FLOP * (double)fx[EXP_NEAR] +
                                         (double)fx[EXP_FORMED] * 8.0 * NMOM * (double)fmm_recs[0].p
                                   : MOMENT_FLOP * (double)fx[EXP_STARS];
        const double exp_flop = sums + STEP_FLOP * (double)fx[EXP_STEPS_DONE];
        const double exp64 = mixed ? 0.0 : exp_flop, exppol = mixed ? exp_flop : 0.0;
        stats->algorithmic_flop = 29.0 * star64 + far64 + exp64 +
                                  20.0 * (double)(h.star[PH_F64] - h.star[TALLY_FAST]) -
                                  10.0 * (double)(h.upd[PH_F64] - h.upd[TALLY_FAST]);
        stats->algorithmic_flop_sweep_roots =
            20.0 * (double)h.star[TALLY_FAST] - 10.0 * (double)h.upd[TALLY_FAST];
        if (n_real == 1) {   // a rectangular field's extra roots: 10 FLOP per root term each
            const double ex = 10.0 * (double)sheet_poly(c->reals[0]).n_extra;
            stats->algorithmic_flop += ex * (double)(h.upd[PH_F64] - h.upd[TALLY_FAST]);
            stats->algorithmic_flop_sweep_roots += ex * (double)h.upd[TALLY_FAST];
        }
        stats->algorithmic_flop_f32 =
            49.0 * (double)h.star[PH_F32] - 10.0 * (double)h.upd[PH_F32] - star32_off;
        stats->algorithmic_flop_polish = 29.0 * starpol + farpol + exppol;
    }
    return result;
}

} // namespace mlcc
