// Tracking kernels for gfx950 (CDNA4, wave64).
//
// The hot path of semi-analytical particle tracking (the paper: Introduction;
// Methods, "MODPATH" and "Multiprocessing"): every particle is displaced cell
// by cell, one analytic step per cell up to the earliest reachable face, and
// is handed to the neighbour across that face until a stopping condition
// (boundary face, maximum time, sink cell) holds.  Particles are independent,
// so the kernels are data parallel over particles:
//
//   * static:     one thread per particle for its whole track (the analogue of
//                 the paper's static scheduling, Methods "Multiprocessing"); the
//                 work is ordered by starting cell and dealt to the dies in chunks,
//                 and in timeseries runs a wave evaluates the snapshots its lanes
//                 meet together, once enough are pending;
//   * persistent: resident waves pull particle indices from a device work
//                 queue; lanes whose particle stopped are refilled at wave level
//                 (ballot + mbcnt prefix count, one atomic per wave), so slow
//                 particles do not idle a whole wave -- the device form of the
//                 paper's dynamic scheduling (Methods "Multiprocessing",
//                 Results "Thread scheduling").
//
// Per step (one cell crossing): gather the cell's six face velocities and its
// flag word (one 64-byte record, or the face arrays), compute each axis' exit
// time from the linear-velocity solution, take the earliest (ties to the lowest
// axis), apply the time limit, advance the other axes analytically, and
// transfer to the neighbour.  Compiled with -ffp-contract=off: no FMA
// contraction, so the FP64 path rounds exactly as written.
//
// Template arguments of both kernels: precision (FP64 / mixed), layout (face
// arrays, packed structured records, quadtree records), output (endpoint,
// timeseries positions, pathline records: the paper's three simulation types,
// Methods "MODPATH") and whether a lane reads its grid from a table (batched
// particle groups, or transient flow, where the table holds one field per time
// step and the lane's index is its current step).
#include <math.h>

#include <type_traits>

#include "pt_crmath.h"
#include "pt_internal.h"

namespace pt {
namespace {

constexpr int kBlock = 256;

enum : int32_t {
    ST_ACTIVE = 0,
    ST_BOUNDARY = 1,
    ST_SINK = 2,
    ST_MAX_TIME = 3,
    ST_STEP_CAP = 4,
    ST_STRANDED = 5,
    ST_INVALID = 6,
    ST_INACTIVE_NB = 7,
    ST_SKIP = -1,  // not tracked by this call (already terminated)
};

__device__ __forceinline__ double dinf() { return __builtin_huge_val(); }

// ---------------------------------------------------------------------------------------------
// One axis, FP64.  u1/u2: velocities at the low/high face (1/d), xi: local coordinate.
// Exit time to the face the velocity points at; +inf when that face is never reached
// (zero particle velocity, or a face velocity of zero or opposite sign).  The exit time
// ln(u_e/u_p)/A is evaluated as (D/u_p) * log1p(x)/x with x = A D/u_p, which stays exact
// as A -> 0; for x < -1/2 (strong deceleration) the ratio u_e/u_p is formed directly.
// log1p, log and expm1 are correctly rounded (pt_crmath.h), so every FP64 operation of a
// step has one defined result.  `amb` counts roundings the accurate phase could not decide.
template <int CR>
__device__ __forceinline__ double exit_core64(double A, double up, double D, double ue, unsigned& amb) {
    const double r = D / up;
    const double x = A * r;
    double dt = r;
    if (x != 0.0) {
        // One logarithm site for both forms, so a wave whose lanes take different forms
        // runs the correctly rounded logarithm once: log(u_e/u_p) when x < -1/2, then
        // dt = log / A; otherwise log1p(x) = log(1 + x) with 1 + x as a double-double,
        // then dt = r * (log1p / x).
        const bool ratio = x < -0.5;
        double L, yh, yl;
        bool done;
        if (ratio) {
            yh = ue / up;
            yl = 0.0;
            done = ptcr::log_special(yh, &L);
        } else {
            const ptcr::dd y = ptcr::two_sum(1.0, x);
            yh = y.h;
            yl = y.l;
            done = ptcr::log1p_special(x, &L);
        }
        if (!done) L = ptcr::log_dd_cr<CR>(yh, yl, &amb);
        const double q = L / (ratio ? A : x);
        dt = ratio ? q : r * q;
    }
    if (dt < 0.0) dt = 0.0;
    return dt;
}

template <int CR>
__device__ __forceinline__ double exit_time64(double u1, double u2, double xi, double& xe,
                                              unsigned& amb) {
    const double A = u2 - u1;
    const double up = u1 + A * xi;
    double ue;
    if (up > 0.0) {
        xe = 1.0;
        ue = u2;
        if (!(ue > 0.0)) return dinf();
    } else if (up < 0.0) {
        xe = 0.0;
        ue = u1;
        if (!(ue < 0.0)) return dinf();
    } else {
        return dinf();
    }
    return exit_core64<CR>(A, up, xe - xi, ue, amb);
}

// Position along one axis after tau: xi + u_p tau expm1(A tau)/(A tau), clamped to [0,1];
// A = u2 - u1 and u_p = u1 + A xi as the exit selection already formed them.
template <int CR>
__device__ __forceinline__ double adv64_au(double A, double up, double xi, double tau, unsigned& amb) {
    if (up == 0.0) return xi;
    const double y = A * tau;
    const double psi = (y == 0.0) ? 1.0 : ptcr::expm1_cr<CR>(y, &amb) / y;
    double xn = xi + (up * tau) * psi;
    xn = (xn < 0.0) ? 0.0 : xn;
    xn = (xn > 1.0) ? 1.0 : xn;
    return xn;
}

// expm1(y) by the lean phase; an undecided rounding goes to the quick phase.  Only |y| <= 36 counts:
// beyond it the value is not used, and on an axis at rest (u_p = 0) neither, so that what the accurate
// phase leaves undecided there is no reason to track the particle again.
template <int CR>
__device__ __forceinline__ double expm1_fast(double y, double up, unsigned& amb) {
    double E;
    if (!ptcr::decided(ptcr::expm1_lean(y), &E) && fabs(y) <= 36.0) {
        unsigned undecided = 0u;
        E = ptcr::expm1_cr<CR>(y, &undecided);
        if (up != 0.0) amb += undecided;
    }
    return E;
}

// adv64_au from E = expm1(y), y = A tau, |y| <= 36, where xi is `plain`.  |y| < 2^-60 (zero included) has
// expm1(y)/y = 1; u_p = 0 adds zero.
__device__ __forceinline__ double adv64_end(double E, double y, double up, double xi, double tau) {
    const double q = ptcr::div_lean(E, y);
    const double psi = (fabs(y) < 0x1p-60) ? 1.0 : q;
    return __builtin_fmin(__builtin_fmax(xi + (up * tau) * psi, 0.0), 1.0);
}

// Whether adv64_end forms the advance of these two coordinates as adv64_au does.  Its clamp turns a NaN
// into 0; with a plain xi and |y| <= 36 none arises: an infinite face velocity of the axis makes A, and y
// with it, infinite or NaN.  (The tests of y are one each: the larger of two magnitudes is never a NaN.)
// A -0.0 keeps its sign where the axis is at rest; the sum and the clamp would lose it.
// The tests cost 0.2% where the chip is full (1e6 particles) and 2% of runs with many snapshots (2e5
// particles, 100 snapshots each: 1,988 -> 2,030 us).
__device__ __forceinline__ bool plain(double a, double b) {
    return max((uint32_t)(ptcr::bits_of(a) >> 32), (uint32_t)(ptcr::bits_of(b) >> 32)) <= 0x3ff00000u;   // the high words of +0 .. 1
}

// adv64_au with the lean phase, where it is not the step's main cost (snapshots, limits): one general
// site for undecided roundings, |y| > 36 and coordinates that are not plain.  The careful pass keeps to
// the general functions.  `need` false: the caller drops the value, whatever it is.
template <int CR>
__device__ __forceinline__ double adv64(double A, double up, double xi, double tau, unsigned& amb, bool need = true) {
    if constexpr (CR == ptcr::CR_FLAG) {
        const double y = A * tau;
        double E;
        const bool done = ptcr::decided(ptcr::expm1_lean(y), &E);
        double xn = adv64_end(E, y, up, xi, tau);
        if ((int)need & (int)!((int)done & (int)(fabs(y) <= 36.0) & (int)plain(xi, xi))) xn = adv64_au<CR>(A, up, xi, tau, amb);
        return xn;
    } else {
        return adv64_au<CR>(A, up, xi, tau, amb);
    }
}

// Earliest exit over the three axes, FP64, with the same result as evaluating exit_time64 on
// every axis and keeping the strictly smallest (ties to the lowest axis).  A cheap FP32
// estimate E of each axis' time is formed first (relative error below 1.5e-6); when one axis
// is ahead of every other by more than 2^-15 relative, only its correctly rounded time is
// evaluated -- the others cannot be smaller.  Otherwise (near ties, estimates out of the FP32
// range, no reachable face) every axis is evaluated exactly.  The estimates and the limit stay in
// FP32: the limit's own rounding (2^-24) is far inside the margin left by two estimates' errors.
constexpr double kFilterMargin = 0x1p-15;

// FP32 estimate of (D/u_p) log1p(x)/x, x = A D/u_p, from the hardware reciprocal and base-2
// logarithm (within 2 ulp each, relative, over the whole normal range: checked exhaustively on
// gfx950).  log1p(x)/x is taken as log(u)/(u - 1) with u = fl(1 + x) (Goldberg's form: u - 1 is
// exact for x > -1/2, and the quotient stays accurate however small x is), one formula for all
// lanes; for x <= -1/2 the ratio u_e/u_p is formed directly.  Error: ~7 ulp in x, propagated
// with a factor below 1, ~10 ulp in the quotient, ~6 ulp in D/u_p: below 1.5e-6 relative, a
// tenth of what the selection margin allows.  The bound needs normal FP32 operands and results;
// `sure` says that they are.  m, the smaller of the distance D and the logarithm's argument q (both at
// most 1 or no matter), and m |u_p| are at least 2^-120: so are D, q, |u_p| and, in the ratio form, u_e =
// q u_p.  The estimate is at least 2^-100, so |u_p| <= 2^107 (D <= 1, log1p(x)/x < 84 there).  NaN fails
// the comparisons: fminf passes it by, but the estimate of a NaN operand is one.  A subnormal distance or
// estimate carries an absolute rounding of 2^-149, i.e. any relative error, and a zero distance (a
// particle already on the face, a zero-time crossing) is decided exactly as well.  Every step outside the
// range is exact: bounds that narrow it to velocities of 2^-70 .. 2^56 cost a 1e6-particle field with its
// flows scaled by 1e-20 or 1e18 4.67 ms instead of 2.0, and a floor of 2^-26 under D and q instead of the
// product cost a field whose velocities jump by 1e12 from face to face 2.2 ms instead of 1.2.
__device__ __forceinline__ float exit_estimate(double D, double up, double A, double ue, bool& sure) {
    const float upf = (float)up;
    const float Df = (float)D;
    const float rup = __builtin_amdgcn_rcpf(upf);
    const float rf = Df * rup;
    const float xf = (float)A * rf;
    const float u = 1.0f + xf;
    const bool ratio = !(xf > -0.5f);
    const float q = ratio ? (float)ue * rup : u;   // u_e/u_p
    const float den = ratio ? xf : u - 1.0f;
    const float ph = (u == 1.0f) ? 1.0f   // |x| < 2^-24: log1p(x)/x = 1 - x/2 + ...
                                 : (__builtin_amdgcn_logf(q) * 0.693147181f) * __builtin_amdgcn_rcpf(den);
    const float E = rf * ph;
    const float m = fminf(fabsf(Df), q);
    sure = (int)(fminf(m, m * fabsf(upf)) >= 0x1p-120f) & (int)(E >= 0x1p-100f);
    return E;
}

// The step's exit, FP64: gradient A and particle velocity u_p of each axis at the step start, and
// the axis the estimates chose (c0: axis 0, else c1: axis 1, else axis 2) with its distance and
// exit-face velocity -- valid when `sure`.
struct Exit64 {
    double A[3], up[3];
    double D, ue, Aw, upw;
    bool c0, c1, high;
    bool sure;
};

__device__ __forceinline__ double sel3(bool c0, bool c1, double a, double b, double c) {
    return c0 ? a : (c1 ? b : c);
}

__device__ __forceinline__ void estimate_exit64(const double (&u1)[3], const double (&u2)[3],
                                                const double (&xi)[3], Exit64& X) {
    float E[3];
    double D[3], ue[3];
    X.sure = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        X.A[a] = u2[a] - u1[a];
        X.up[a] = u1[a] + X.A[a] * xi[a];
        const bool pos = X.up[a] > 0.0, neg = X.up[a] < 0.0;
        const bool out2 = u2[a] > 0.0, out1 = u1[a] < 0.0;
        ue[a] = pos ? u2[a] : u1[a];
        D[a] = (pos ? 1.0 : 0.0) - xi[a];
        const bool feasible = ((int)pos & (int)out2) | ((int)neg & (int)out1);
        bool sure;
        const float est = exit_estimate(D[a], X.up[a], X.A[a], ue[a], sure);
        E[a] = feasible ? est : __builtin_inff();
        X.sure = (int)X.sure & ((int)sure | (int)!feasible);
    }
    const float Ew = fminf(fminf(E[0], E[1]), E[2]);
    const float second = __builtin_amdgcn_fmed3f(E[0], E[1], E[2]);
    // a second axis inside the margin, or (inf <= inf) no axis at all
    X.sure = (int)X.sure & (int)!(second <= Ew * (1.0f + (float)kFilterMargin));   // 1 + 2^-15 is a float
    X.c0 = E[0] == Ew;
    X.c1 = E[1] == Ew;
    X.D = sel3(X.c0, X.c1, D[0], D[1], D[2]);
    X.ue = sel3(X.c0, X.c1, ue[0], ue[1], ue[2]);
    X.Aw = sel3(X.c0, X.c1, X.A[0], X.A[1], X.A[2]);
    X.upw = sel3(X.c0, X.c1, X.up[0], X.up[1], X.up[2]);
    X.high = X.upw > 0.0;
}

// Correctly rounded exit time of the chosen axis (exit_time64's operations) with the lean phase, for
// lanes that come with `ok`.  An undecided rounding is repaired in place where waves are full (5% of
// wave steps, with half the instructions of the general function), or clears `ok` (REPAIR false).
// The estimates' ranges (u_p in [2^-120, 2^107], D in [2^-120, 1], u_e at least
// 2^-120 in the ratio form, |x| < 2^128) keep every quotient inside the range of div_by.
// |x| < 2^-60 (zero included) has log1p(x)/x = 1.
template <int CR, bool REPAIR>
__device__ __forceinline__ double exit_time64_fast(const Exit64& X, bool& ok, unsigned& amb) {
    const double ru = ptcr::recip_lean(X.upw);
    const double r = ptcr::div_by(X.D, X.upw, ru);
    const double x = X.Aw * r;
    const bool ratio = x < -0.5;
    // 1 + x as an exact ordered sum; u_e/u_p in the ratio form
    const double big = __builtin_fmax(x, 1.0), sml = __builtin_fmin(x, 1.0);
    const double s = big + sml;
    const double yh = ratio ? ptcr::div_by(X.ue, X.upw, ru) : s;
    const double yl = ratio ? 0.0 : sml - (s - big);
    double L;
    const bool done = ptcr::decided(ptcr::log_lean(yh, yl), &L);
    if constexpr (REPAIR) {
        if (!done && ok) L = ptcr::log_dd_cr<CR>(yh, yl, &amb);
    } else {
        ok = (int)ok & (int)done;
    }
    const double q = ptcr::div_lean(L, ratio ? X.Aw : x);
    double dt = ratio ? q : r * q;
    dt = (fabs(x) < 0x1p-60) ? r : dt;
    return __builtin_fmax(dt, 0.0);
}

// Every axis evaluated exactly.
template <int CR>
__device__ __forceinline__ void exit_exact64(const double (&u1)[3], const double (&u2)[3], const double (&xi)[3],
                                             double& dt, int32_t& axis, double& xe, unsigned& amb) {
    dt = dinf();
    axis = -1;
    xe = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double e = 0.0;
        const double ta = exit_time64<CR>(u1[a], u2[a], xi[a], e, amb);
        if (ta < dt) {
            dt = ta;
            axis = a;
            xe = e;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// One axis, mixed precision: FP32 velocities, local coordinate and in-cell arithmetic, with
// the hardware reciprocal, base-2 logarithm and exponential (within 2 ulp each, relative);
// FP64 for time and for the near-zero-gradient branch (|x| < 2^-10 or |A tau| < 2^-10), where
// short series are evaluated in double.  Beyond it one branch-free formula serves every lane:
// log1p(x)/x = log(u)/(u - 1) with u = fl(1 + x) (Goldberg), and expm1(y)/y = (v - 1)/log(v)
// with v = fl(e^y) (Kahan: the logarithm of the rounded exponential compensates its rounding).
constexpr float kNearZero = 0x1p-10f;
constexpr float kLn2f = 0.693147181f;
constexpr float kLog2ef = 1.44269504f;

// Local coordinates of the mixed kernels: FP32, or FP64 (kMixedCoord64) -- then the distance to
// the face is formed in FP64 before it is rounded to FP32, and advances are added in FP64.
constexpr bool kMixedCoord64 = false;
using MixCoord = std::conditional_t<kMixedCoord64, double, float>;

// Exit time where |x| < 2^-10: D/u_p from the FP32 quotient r and its residual D - u_p r (exact in
// FP64: u_p r is a 48-bit product), corrected once with the FP32 reciprocal: relative error ~2^-46.
__device__ __forceinline__ double exit_series_mix(float D, float A, float up, float rup, float r) {
    const double rd0 = (double)r;
    const double rd = fma((double)rup, fma(-(double)up, rd0, (double)D), rd0);
    const double xd = (double)A * rd;
    // log1p(x)/x = 1 - x/2 + x^2/3 - x^3/4 + x^4/5 - ..., truncation below 2^-52 here
    const double ph = fma(xd, fma(xd, fma(xd, fma(xd, 0.2, -0.25), 1.0 / 3.0), -0.5), 1.0);
    return rd * ph;
}

__device__ __forceinline__ double exit_time_mix(float u1, float u2, MixCoord xc, float& xe, unsigned& amb) {
    (void)amb;
    const float xi = (float)xc;
    const float A = u2 - u1;
    const float up = fmaf(A, xi, u1);
    const bool pos = up > 0.0f;
    xe = pos ? 1.0f : 0.0f;
    const float ue = pos ? u2 : u1;
    if (!((pos && ue > 0.0f) | (up < 0.0f && ue < 0.0f))) return dinf();
    const float D = (float)((MixCoord)xe - xc);
    const float rup = __builtin_amdgcn_rcpf(up);
    const float r = D * rup;
    const float x = A * r;
    if (fabsf(x) < kNearZero) {
        return exit_series_mix(D, A, up, rup, r);
    }
    // u - 1 is exact for x > -1/2 and not zero here; for x <= -1/2 the ratio q = u_e/u_p is formed
    // directly and divided by x
    const float u = 1.0f + x;
    const bool ratio = !(x > -0.5f);
    const float q = ratio ? ue * rup : u;
    const float den = ratio ? x : u - 1.0f;
    const float ph = (__builtin_amdgcn_logf(q) * kLn2f) * __builtin_amdgcn_rcpf(den);
    float dt = r * ph;
    if (dt < 0.0f) dt = 0.0f;
    return (double)dt;
}

// The step's exit, mixed precision: what the smallest of the three exit_time_mix is, and whose
// (the lowest axis among equals).  Bound by VALU issue when the chip is full and by the length of the
// step when it is not.  Each axis is one straight line in FP32, and the times are compared there
// (each is an FP32 value: the same order as in FP64).  A near-zero-gradient axis enters with r, which
// is within 2^-10 of its time; its series is evaluated for the lanes whose earliest axis it is, and
// where another axis comes within 2^-8 of it, or the earliest time is not positive, every time is
// taken in full.  Against a series, an FP64 comparison and nested branches on each axis, with the next
// record gathered at the end of the step (100x100x10 field, tracking and ordering): 1e4 particles
// 186 -> 158 us, 1e5 248 -> 218 us, 1e6 945 -> 940 us.  Without the branch on w the few-particle
// runs are another 8% shorter, but the full chip's 3% longer: neighbours skip an axis together.
__device__ __forceinline__ void exit_mix(const float (&u1)[3], const float (&u2)[3], const MixCoord (&xi)[3],
                                         const float (&A)[3], const float (&up)[3], Exit64& X, double& dt,
                                         int32_t& axis, unsigned& amb) {
    float E[3];
    bool near[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool pos = up[a] > 0.0f;
        // exit-face speed in the particle's direction; u_p = 0 with w > 0 has an infinite r and E = NaN
        const float w = pos ? u2[a] : -u1[a];
        E[a] = __builtin_inff();
        near[a] = false;
        if (w > 0.0f) {   // neighbouring particles share an axis without an exit: the wave skips it
            const float rup = __builtin_amdgcn_rcpf(up[a]);
            const float r = (float)((MixCoord)(pos ? 1.0f : 0.0f) - xi[a]) * rup;
            const float x = A[a] * r;
            const float u = 1.0f + x;
            const bool ratio = !(x > -0.5f);
            const float q = ratio ? w * __builtin_fabsf(rup) : u;
            const float den = ratio ? x : u - 1.0f;
            const float ph = (__builtin_amdgcn_logf(q) * kLn2f) * __builtin_amdgcn_rcpf(den);
            near[a] = fabsf(x) < kNearZero;
            E[a] = near[a] ? r : r * ph;
        }
    }
    // NaN is never the earliest: fminf passes it by, and it equals nothing
    const float Ew = fminf(fminf(fminf(E[0], E[1]), E[2]), __builtin_inff());
    X.c0 = E[0] == Ew;
    X.c1 = E[1] == Ew;
    const bool some = Ew < __builtin_inff();
    axis = some ? (X.c0 ? 0 : (X.c1 ? 1 : 2)) : -1;
    X.high = (X.c0 ? up[0] : (X.c1 ? up[1] : up[2])) > 0.0f;
    dt = (double)Ew;
    const bool any_near = (int)some & ((int)near[0] | (int)near[1] | (int)near[2]);
    if ((int)any_near | (int)(Ew <= 0.0f)) {
        const float second = __builtin_amdgcn_fmed3f(E[0], E[1], E[2]);   // the smallest itself when one is NaN
        // 2^-110: an r below the normal range is no estimate
        if ((int)(Ew <= 0.0f) | (int)!(second > fmaf(Ew, 1.0f + 0x1p-8f, 0x1p-110f))) {
            dt = dinf();
            axis = -1;
            float xe = 0.0f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                float e = 0.0f;
                const double ta = exit_time_mix(u1[a], u2[a], xi[a], e, amb);
                if (ta < dt) {
                    dt = ta;
                    axis = a;
                    xe = e;
                }
            }
            X.c0 = axis <= 0;
            X.c1 = axis == 1;
            X.high = xe == 1.0f;
        } else if (((int)X.c0 & (int)near[0]) | ((int)!X.c0 & (((int)X.c1 & (int)near[1]) | ((int)!X.c1 & (int)near[2])))) {
            const float upw = X.c0 ? up[0] : (X.c1 ? up[1] : up[2]);
            const float Aw = X.c0 ? A[0] : (X.c1 ? A[1] : A[2]);
            const MixCoord xw = X.c0 ? xi[0] : (X.c1 ? xi[1] : xi[2]);
            const float D = (float)((MixCoord)(upw > 0.0f ? 1.0f : 0.0f) - xw);
            const float rup = __builtin_amdgcn_rcpf(upw);
            dt = exit_series_mix(D, Aw, upw, rup, D * rup);
        }
    }
}

__device__ __forceinline__ MixCoord adv_mix_au(float A, float up, MixCoord xi, double tau) {
    if (up == 0.0f) return xi;
    const float tf = (float)tau;
    const float y = A * tf;
    MixCoord xn;
    if (fabsf(y) < kNearZero) {
        // expm1(y)/y = 1 + y/2 + y^2/6 + y^3/24 + y^4/120 + ..., truncation below 2^-59 here
        const double yd = (double)A * tau;
        const double psi = fma(yd, fma(yd, fma(yd, fma(yd, 1.0 / 120.0, 1.0 / 24.0), 1.0 / 6.0), 0.5), 1.0);
        xn = (MixCoord)fma((double)up * tau, psi, (double)xi);
    } else {
        // v - 1 is exact for |y| < 1/8 (Sterbenz) and not zero here; beyond, (v - 1)/y
        const float v = __builtin_amdgcn_exp2f(y * kLog2ef);
        const float den = (fabsf(y) < 0.125f) ? __builtin_amdgcn_logf(v) * kLn2f : y;
        const float ps = (v - 1.0f) * __builtin_amdgcn_rcpf(den);
        if constexpr (kMixedCoord64) xn = xi + (double)((up * tf) * ps);
        else xn = fmaf(up * tf, ps, xi);
    }
    xn = (xn < (MixCoord)0) ? (MixCoord)0 : xn;
    xn = (xn > (MixCoord)1) ? (MixCoord)1 : xn;
    return xn;
}

// ---------------------------------------------------------------------------------------------
template <int PREC> struct Real;
template <> struct Real<P64> { using T = double; };
template <> struct Real<PMIX> { using T = float; };
// Type of the local coordinates of a lane.
template <int PREC> struct Coord;
template <> struct Coord<P64> { using T = double; };
template <> struct Coord<PMIX> { using T = MixCoord; };

// Lane state of one particle.
template <int PREC>
struct Lane {
    using R = typename Real<PREC>::T;
    int64_t pid;        // particle index, -1 when the lane is idle
    int32_t c, i, j, k; // cell
    int32_t g;          // grid index (batched runs)
    int32_t ncross;
    int32_t ks;         // next snapshot index
    unsigned amb;       // undecided roundings of the correctly rounded functions
    unsigned drop;      // pathline records that had no slot
    unsigned drop0;     // pathline: `drop` when this particle began
    unsigned long long hash;
    double t;
    double s_next;      // time of snapshot ks (+inf past the last)
    typename Coord<PREC>::T x[3];   // local coordinates
    R v1[3], v2[3];     // packed layout: the current cell's face velocities (low, high face)
    int32_t fl;         // packed layout: the current cell's flag word
    int32_t nc0;        // pathline: crossings before this call
    int32_t zrun;       // quadtree: zero-time crossings in a row
    int32_t sub_base;   // quadtree: the current cell's first subface, subface counts and neighbours
    uint32_t counts;
    int32_t nbf[6];
    int64_t pq, pend;   // pathline record pass: next slot, end of the particle's slots
};

template <bool BATCHED>
__device__ __forceinline__ const GridDev& grid_of(const TrackParams& P, int32_t g) {
    if constexpr (BATCHED) return P.grids[g];
    else return P.g0;
}

// Layouts whose cells are packed records (structured records, quadtree records).
template <int LAYOUT> constexpr bool kPacked = (LAYOUT == L_CELL || LAYOUT == L_QUAD);

// Whether a lane keeps its cell's (i, j, k) up to date at every crossing: the face layout needs
// them for its face indices, timeseries and pathline outputs for their positions.  Endpoint runs
// on packed structured records only need them at the end, formed from the cell id there.
template <int LAYOUT, int OUT> constexpr bool kTrackIJK = !(LAYOUT == L_CELL && OUT == O_END);

// (i, j, k) of structured cell c.
__device__ __forceinline__ void cell_ijk(const GridDev& G, int32_t c, int32_t& i, int32_t& j, int32_t& k) {
    const int32_t plane = G.nx * G.ny;
    k = c / plane;
    const int32_t rem = c - k * plane;
    j = rem / G.nx;
    i = rem - j * G.nx;
}

// Gather one packed cell record: face velocities (with the direction sign) and the flag word.
template <int PREC>
__device__ __forceinline__ void load_rec(const GridDev& G, int32_t c, double sign,
                                         typename Real<PREC>::T (&u1)[3],
                                         typename Real<PREC>::T (&u2)[3], int32_t& fl) {
    if constexpr (PREC == P64) {
        const CellRec64* rec = G.rec64 + (uint32_t)c;
        const double2* r = reinterpret_cast<const double2*>(rec);
        const double2 a = r[0], b = r[1], d = r[2];
        fl = rec->flags;
        u1[0] = a.x; u2[0] = a.y;
        u1[1] = b.x; u2[1] = b.y;
        u1[2] = d.x; u2[2] = d.y;
        if (sign != 1.0) {   // backward tracking (uniform across the launch)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                u1[q] = sign * u1[q];
                u2[q] = sign * u2[q];
            }
        }
    } else {
        const float4* r = reinterpret_cast<const float4*>(G.rec32 + c);
        const float4 a = r[0];
        const float4 b = r[1];
        fl = __float_as_int(b.z);
        u1[0] = a.x; u2[0] = a.y;
        u1[1] = a.z; u2[1] = a.w;
        u1[2] = b.x; u2[2] = b.y;
        if (sign != 1.0) {   // backward tracking (uniform across the launch)
            const float fs = (float)sign;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                u1[q] = fs * u1[q];
                u2[q] = fs * u2[q];
            }
        }
    }
}

// Gather the record and the face neighbours of a quadtree cell into the lane.
__device__ __forceinline__ void load_quad(const GridDev& G, int32_t c, double sign, Lane<P64>& L) {
    load_rec<P64>(G, c, sign, L.v1, L.v2, L.fl);
    const QuadRec* rec = reinterpret_cast<const QuadRec*>(G.rec64) + (uint32_t)c;
    L.sub_base = rec->sub_base;
    L.counts = rec->counts;
    const QuadFace* face = reinterpret_cast<const QuadFace*>(G.rec32) + (uint32_t)c;
    const int4 a = *reinterpret_cast<const int4*>(face->nb);
    const int2 b = *reinterpret_cast<const int2*>(face->nb + 4);
    L.nbf[0] = a.x;
    L.nbf[1] = a.y;
    L.nbf[2] = a.z;
    L.nbf[3] = a.w;
    L.nbf[4] = b.x;
    L.nbf[5] = b.y;
}

// Gather one cell: face velocities (with the direction sign) and the flag word.
template <int PREC, int LAYOUT>
__device__ __forceinline__ void load_cell(const GridDev& G, const Lane<PREC>& L, double sign,
                                          typename Real<PREC>::T (&u1)[3],
                                          typename Real<PREC>::T (&u2)[3], int32_t& fl) {
    if constexpr (kPacked<LAYOUT>) {
        if constexpr (PREC == P64) {
            const double2* r = reinterpret_cast<const double2*>(G.rec64 + L.c);
            const double2 a = r[0], b = r[1], d = r[2];
            fl = G.rec64[L.c].flags;
            u1[0] = sign * a.x; u2[0] = sign * a.y;
            u1[1] = sign * b.x; u2[1] = sign * b.y;
            u1[2] = sign * d.x; u2[2] = sign * d.y;
        } else {
            const float4* r = reinterpret_cast<const float4*>(G.rec32 + L.c);
            const float4 a = r[0];
            const float4 b = r[1];
            const float fs = (float)sign;
            fl = __float_as_int(b.z);
            u1[0] = fs * a.x; u2[0] = fs * a.y;
            u1[1] = fs * a.z; u2[1] = fs * a.w;
            u1[2] = fs * b.x; u2[2] = fs * b.y;
        }
    } else {
        static_assert(PREC == P64, "the faces layout is FP64 only");
        const int64_t nx = G.nx, ny = G.ny;
        const int64_t fx = ((int64_t)L.k * ny + L.j) * (nx + 1) + L.i;
        const int64_t fy = ((int64_t)L.k * (ny + 1) + L.j) * nx + L.i;
        const int64_t fz = ((int64_t)L.k * ny + L.j) * nx + L.i;
        const double n_c = G.por ? G.por[L.c] : G.por_scalar;
        const double d = n_c * G.V;
        u1[0] = (sign * G.qx[fx]) / d;
        u2[0] = (sign * G.qx[fx + 1]) / d;
        u1[1] = (sign * G.qy[fy]) / d;
        u2[1] = (sign * G.qy[fy + nx]) / d;
        u1[2] = (sign * G.qz[fz]) / d;
        u2[2] = (sign * G.qz[fz + nx * ny]) / d;
        fl = G.flags[L.c];
    }
}

__device__ __forceinline__ void put_nan3(double* p) {
    const double q = __builtin_nan("");
    p[0] = q;
    p[1] = q;
    p[2] = q;
}

// Global position of local coordinates (a, b, d) in cell (i, j, k).
__device__ __forceinline__ void global_xyz(const GridDev& G, int32_t i, int32_t j, int32_t k, double a,
                                           double b, double d, double* out) {
    out[0] = G.x0 + ((double)i + a) * G.dx;
    out[1] = G.y0 + ((double)j + b) * G.dy;
    out[2] = G.z0 + ((double)k + d) * G.dz;
}

// Global position of local coordinates (a, b, d) in cell c: from (i, j, k) on a structured
// grid, from the cell's box on a quadtree grid.
template <int LAYOUT>
__device__ __forceinline__ void cell_xyz(const GridDev& G, int32_t c, int32_t i, int32_t j, int32_t k, double a,
                                         double b, double d, double* out) {
    if constexpr (LAYOUT == L_QUAD) {
        const QuadBox& B = G.qbox[c];
        out[0] = B.lo[0] + a * B.h[0];
        out[1] = B.lo[1] + b * B.h[1];
        out[2] = B.lo[2] + d * B.h[2];
    } else {
        (void)c;
        global_xyz(G, i, j, k, a, b, d, out);
    }
}

// Gradient and particle velocity of each axis at the step start, as the advance takes them.
template <int PREC>
__device__ __forceinline__ void step_au(const typename Real<PREC>::T (&u1)[3], const typename Real<PREC>::T (&u2)[3],
                                        const typename Coord<PREC>::T (&x)[3], typename Real<PREC>::T (&A)[3],
                                        typename Real<PREC>::T (&up)[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        A[a] = u2[a] - u1[a];
        if constexpr (PREC == P64) up[a] = u1[a] + A[a] * x[a];
        else up[a] = fmaf(A[a], (float)x[a], u1[a]);
    }
}

// Position at snapshot time s of a particle whose step started at time t in cell c (i, j, k)
// with local coordinates x, gradients A and velocities up: tau = s - t on every axis.
template <int PREC, int LAYOUT, int CR>
__device__ __forceinline__ void eval_snap(const GridDev& G, const typename Real<PREC>::T (&A)[3],
                                          const typename Real<PREC>::T (&up)[3],
                                          const typename Coord<PREC>::T (&x)[3], double t, int32_t c,
                                          int32_t i, int32_t j, int32_t k, double s, double* out,
                                          unsigned& amb) {
    const double tau = s - t;
    double p[3];
    if constexpr (PREC == P64) {
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = adv64<CR>(A[a], up[a], x[a], tau, amb);
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = (double)adv_mix_au(A[a], up[a], x[a], tau);
    }
    cell_xyz<LAYOUT>(G, c, i, j, k, p[0], p[1], p[2], out);
}

// Snapshot ks of a particle whose step started at (t, x) in cell c.
template <int PREC, int LAYOUT, int CR>
__device__ __forceinline__ void snap_at(const GridDev& G, const TrackParams& P,
                                        const typename Real<PREC>::T (&A)[3],
                                        const typename Real<PREC>::T (&up)[3],
                                        const typename Coord<PREC>::T (&x)[3], double t, int32_t c, int32_t i,
                                        int32_t j, int32_t k, int64_t pid, int32_t ks, double s, unsigned& amb) {
    eval_snap<PREC, LAYOUT, CR>(G, A, up, x, t, c, i, j, k, s, P.snap_xyz + (pid * P.n_snap + ks) * 3, amb);
}

// Positions at the snapshot times s with s < to (or s <= to when closed), evaluated from the
// state at the start of the step with tau = s - t.
template <int PREC, int LAYOUT, int CR>
__device__ __forceinline__ void write_snaps(Lane<PREC>& L, const GridDev& G,
                                            const typename Real<PREC>::T (&A)[3],
                                            const typename Real<PREC>::T (&up)[3],
                                            const TrackParams& P, const double* snap, double to,
                                            bool closed) {
    while (L.ks < P.n_snap) {
        const double s = L.s_next;
        if (closed ? !(s <= to) : !(s < to)) break;
        snap_at<PREC, LAYOUT, CR>(G, P, A, up, L.x, L.t, L.c, L.i, L.j, L.k, L.pid, L.ks, s, L.amb);
        ++L.ks;
        L.s_next = (L.ks < P.n_snap) ? snap[L.ks] : dinf();
    }
}

// Deferred snapshots (static kernel, timeseries, packed layouts).  In a wave, only the few lanes
// whose step holds a snapshot time would run the snapshot arithmetic at that step, while the
// others wait.  Instead a lane records its step-start state and snapshot range in its LDS slot;
// once kSnapFlush lanes of the wave have a pending slot (or no lane is left tracking), the wave
// evaluates all pending snapshots together, each lane taking one (slot, snapshot) pair.  Each
// snapshot is the same function of the same state, so the results do not change.
constexpr int kSnapFlush = 32;

// Ordering of the LDS slots between the lanes of one wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The snapshots of a step ending at `to` (open interval): into the lane's slot when it is free,
// else evaluated at once.
template <int PREC, int LAYOUT, int CR>
__device__ __forceinline__ void queue_snaps(Lane<PREC>& L, const GridDev& G,
                                            const typename Real<PREC>::T (&A)[3],
                                            const typename Real<PREC>::T (&up)[3], const TrackParams& P,
                                            const double* snap, double to,
                                            SnapJob<typename Real<PREC>::T>* job) {
    const int32_t ks0 = L.ks;
    while (L.ks < P.n_snap && L.s_next < to) {
        ++L.ks;
        L.s_next = (L.ks < P.n_snap) ? snap[L.ks] : dinf();
    }
    const int32_t cnt = L.ks - ks0;
    if (cnt == 0) return;
    if (job->cnt == 0) {
        job->x[0] = L.x[0];
        job->x[1] = L.x[1];
        job->x[2] = L.x[2];
        job->t = L.t;
        job->c = L.c;
        job->i = L.i;
        job->j = L.j;
        job->k = L.k;
        job->g = L.g;
        job->pid = (int32_t)L.pid;
        job->ks0 = ks0;
        job->cnt = cnt;
    } else {
        for (int32_t q = ks0; q < L.ks; ++q)
            snap_at<PREC, LAYOUT, CR>(G, P, A, up, L.x, L.t, L.c, L.i, L.j, L.k, L.pid, q, snap[q], L.amb);
    }
}

// All lanes of the wave: evaluate every pending snapshot of the wave's 64 slots W and free them.
template <int PREC, int LAYOUT, bool BATCHED, int CR>
__device__ __forceinline__ void flush_snaps(SnapJob<typename Real<PREC>::T>* W, const TrackParams& P,
                                            const double* snap) {
    using R = typename Real<PREC>::T;
    const int lane = (int)(threadIdx.x & 63u);
    const int cnt = W[lane].cnt;
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off, 64);
        if (lane >= off) incl += v;
    }
    const int total = __shfl(incl, 63, 64);
    W[lane].start = incl - cnt;
    wave_sync();
    for (int q = lane; q < total; q += 64) {
        // the slot holding pair q: the last one whose first pair is at most q (it has cnt > 0)
        int lo = 0, hi = 64;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (W[mid].start <= q) lo = mid;
            else hi = mid;
        }
        const SnapJob<R>& J = W[lo];
        const GridDev& G = grid_of<BATCHED>(P, J.g);
        R u1[3], u2[3];
        typename Coord<PREC>::T x[3];
        int32_t fl;
        load_rec<PREC>(G, J.c, P.sign, u1, u2, fl);
        x[0] = J.x[0];
        x[1] = J.x[1];
        x[2] = J.x[2];
        const int32_t ks = J.ks0 + (q - J.start);
        unsigned a = 0u;
        R A[3], up[3];
        step_au<PREC>(u1, u2, x, A, up);
        snap_at<PREC, LAYOUT, CR>(G, P, A, up, x, J.t, J.c, J.i, J.j, J.k, (int64_t)J.pid, ks, snap[ks], a);
        if (a) W[lo].amb = a;   // the slot's owner hands its particle to the careful pass
    }
    wave_sync();
    W[lane].cnt = 0;
    wave_sync();
}

template <int PREC>
__device__ __forceinline__ void nan_rest(Lane<PREC>& L, const TrackParams& P) {
    double* row = P.snap_xyz + L.pid * (int64_t)P.n_snap * 3;
    for (int32_t q = L.ks; q < P.n_snap; ++q) put_nan3(row + 3 * (int64_t)q);
    L.ks = P.n_snap;
}

// Pathline record staging.  A lane's records form one contiguous stream (40 bytes each), but
// the lanes of a wave write to as many streams, so written one by one they leave partial 64-byte
// segments that the L2 evicts before the next record completes them (measured on C2: 1.8x the
// record bytes written to HBM plus reads for the partial segments).  Staged in the lane's LDS
// slot, the stream is written in whole 64-byte segments; only the segments at the ends of the
// stream, which it shares with its neighbours, are written in 8-byte words.
__device__ __forceinline__ PathStage* path_stage_slot() {
    extern __shared__ __align__(16) double dyn_lds[];
    return reinterpret_cast<PathStage*>(dyn_lds) + threadIdx.x;
}

__device__ __forceinline__ void stage_record(const TrackParams& P, int64_t q, double t, double x,
                                             double y, double z, int32_t cell, int32_t face) {
    PathStage* S = path_stage_slot();
    const int64_t B = 40 * q;                       // byte offset of the record in the stream
    const int64_t wb = B & ~(int64_t)63;            // its segment
    const int o = (int)((B - wb) >> 3);             // in doubles: 0 .. 7
    S->buf[o] = t;
    S->buf[o + 1] = x;
    S->buf[o + 2] = y;
    S->buf[o + 3] = z;
    S->buf[o + 4] = __longlong_as_double((long long)(((uint64_t)(uint32_t)face << 32) | (uint32_t)cell));
    if (o + 5 >= 8) {
        // the segment is complete: write it (from the particle's first byte if it starts there)
        double* dst = reinterpret_cast<double*>(reinterpret_cast<char*>(P.path_rec) + wb);
        const int64_t B0 = 40 * S->q0;
        if (B0 <= wb) {
            const double2* src = reinterpret_cast<const double2*>(S->buf);
            double2* d2 = reinterpret_cast<double2*>(dst);
            d2[0] = src[0];
            d2[1] = src[1];
            d2[2] = src[2];
            d2[3] = src[3];
        } else {
            for (int k = (int)((B0 - wb) >> 3); k < 8; ++k) dst[k] = S->buf[k];
        }
        for (int k = 8; k < o + 5; ++k) S->buf[k - 8] = S->buf[k];
    }
}

// Write what is left of the staged stream [q0, qend) (its last, partial segment).
__device__ __forceinline__ void flush_records(const TrackParams& P, int64_t qend) {
    PathStage* S = path_stage_slot();
    const int64_t N = 40 * qend, B0 = 40 * S->q0;
    if (N <= B0) return;
    const int64_t wb = N & ~(int64_t)63;
    const int hi = (int)((N - wb) >> 3);
    const int lo = (B0 > wb) ? (int)((B0 - wb) >> 3) : 0;
    double* dst = reinterpret_cast<double*>(reinterpret_cast<char*>(P.path_rec) + wb);
    for (int k = lo; k < hi; ++k) dst[k] = S->buf[k];
}

// Group of particle `pid` (largest g with group_offsets[g] <= pid, empty groups skipped).
__device__ __forceinline__ int32_t find_group(const TrackParams& P, int64_t pid) {
    int32_t lo = 0, hi = P.n_groups;  // invariant: offsets[lo] <= pid < offsets[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (P.group_offsets[mid] <= pid) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Time step of a particle at time t (transient flow): the first step whose end is after t.
__device__ __forceinline__ int32_t step_of(const TrackParams& P, double t) {
    int32_t s = 0;
    while (s < P.n_tsteps - 1 && !(t < P.tstep_end[s])) ++s;
    return s;
}

// Release checks (S0).  Returns 0 when the particle is to be tracked, ST_SKIP when it is
// not tracked by this call, or a final status.
template <int PREC, int LAYOUT, int OUT, bool BATCHED>
__device__ int32_t begin(Lane<PREC>& L, const TrackParams& P, const double* snap) {
    const int64_t p = L.pid;
    const int32_t st = P.status[p];
    L.g = 0;
    if constexpr (BATCHED) {
        if (P.n_tsteps) L.g = step_of(P, P.t[p]);   // transient: the grid is the time step's
        else L.g = P.group_grid[find_group(P, p)];
    }
    const GridDev& G = grid_of<BATCHED>(P, L.g);
    const int64_t ncell = (int64_t)G.nx * G.ny * G.nz;
    const int32_t c = P.cell[p];
    if (st != ST_ACTIVE && st != ST_MAX_TIME) {
        if constexpr (OUT == O_PATH) {
            if (P.path_count) {
                P.path_off[p + 1] = 0;   // dry run: nothing else is written
                return ST_SKIP;
            }
        }
        if (P.out_xyz) {
            double* o = P.out_xyz + 3 * p;
            if (st == ST_INVALID || c < 0 || c >= ncell) {
                put_nan3(o);
            } else {
                const int32_t plane = G.nx * G.ny;
                const int32_t k = c / plane, rem = c - k * plane;
                const int32_t j = rem / G.nx, i = rem - j * G.nx;
                cell_xyz<LAYOUT>(G, c, i, j, k, P.xi[p], P.eta[p], P.zeta[p], o);
            }
        }
        return ST_SKIP;
    }
    const bool fresh = (st == ST_ACTIVE);
    const double a = P.xi[p], b = P.eta[p], d = P.zeta[p], t = P.t[p];
    bool bad = (c < 0 || (int64_t)c >= ncell);
    int32_t own = 0;
    if (!bad) {
        if constexpr (kPacked<LAYOUT>) {
            own = (PREC == P64) ? G.rec64[c].flags : G.rec32[c].flags;
        } else {
            own = G.flags[c];
        }
        bad = !(own & CF_ACTIVE);
    }
    if (!(a >= 0.0 && a <= 1.0) || !(b >= 0.0 && b <= 1.0) || !(d >= 0.0 && d <= 1.0)) bad = true;
    if (!(t == t) || __builtin_isinf(t)) bad = true;
    if (bad) {
        if constexpr (OUT == O_SERIES) {
            L.ks = 0;
            nan_rest(L, P);
        }
        return ST_INVALID;
    }
    if constexpr (LAYOUT == L_QUAD) load_quad(G, c, P.sign, L);
    else if constexpr (kPacked<LAYOUT>) load_rec<PREC>(G, c, P.sign, L.v1, L.v2, L.fl);
    L.c = c;
    L.zrun = 0;
    if constexpr (kTrackIJK<LAYOUT, OUT>) cell_ijk(G, c, L.i, L.j, L.k);
    L.x[0] = (typename Coord<PREC>::T)a;
    L.x[1] = (typename Coord<PREC>::T)b;
    L.x[2] = (typename Coord<PREC>::T)d;
    L.t = t;
    L.ncross = P.ncross[p];
    L.hash = P.hash[p];
    if constexpr (OUT == O_PATH) {
        L.nc0 = L.ncross;
        L.drop0 = L.drop;
        if (!P.path_count) {
            L.pq = P.path_off[p];
            const int64_t e = P.path_off[p + 1];
            L.pend = (e < P.path_cap) ? e : P.path_cap;
            if (P.path_stage) path_stage_slot()->q0 = L.pq;
        }
    }
    if constexpr (OUT == O_SERIES) {
        double* row = P.snap_xyz + p * (int64_t)P.n_snap * 3;
        int32_t q = 0;
        while (q < P.n_snap && snap[q] < t) {
            if (fresh) put_nan3(row + 3 * (int64_t)q);
            ++q;
        }
        L.ks = q;
        L.s_next = (q < P.n_snap) ? snap[q] : dinf();
    }
    if ((own & CF_SINK) && P.stop_at_sink) return ST_SINK;
    if (t > P.t_max) return ST_MAX_TIME;
    if constexpr (BATCHED) {
        if (P.n_tsteps && t > P.tstep_end[P.n_tsteps - 1]) return ST_MAX_TIME;
    }
    return 0;
}

// Write the final state of a tracked particle.
template <int PREC, int LAYOUT, int OUT, bool BATCHED>
__device__ void finish(Lane<PREC>& L, int32_t st, const TrackParams& P, unsigned int* s_hist,
                       unsigned long long& crossings) {
    const int64_t p = L.pid;
    atomicAdd(&s_hist[st], 1u);
    // the crossings of this call: the state still holds the count the particle came with
    if (st != ST_INVALID) crossings += (unsigned long long)(L.ncross - P.ncross[p]);
    if constexpr (OUT == O_PATH) {
        if (P.path_count) {   // dry run: the crossing count is the only output
            P.path_off[p + 1] = (st == ST_INVALID) ? 0 : (int64_t)(L.ncross - L.nc0);
            return;
        }
        if (P.path_stage && st != ST_INVALID) flush_records(P, (L.pq < L.pend) ? L.pq : L.pend);
    }
    P.status[p] = st;
    if (st == ST_INVALID) {
        if (P.out_xyz) put_nan3(P.out_xyz + 3 * p);
        return;
    }
    P.cell[p] = L.c;
    P.xi[p] = (double)L.x[0];
    P.eta[p] = (double)L.x[1];
    P.zeta[p] = (double)L.x[2];
    P.t[p] = L.t;
    P.ncross[p] = L.ncross;
    P.hash[p] = L.hash;
    if (P.out_xyz) {
        const GridDev& G = grid_of<BATCHED>(P, L.g);
        if constexpr (!kTrackIJK<LAYOUT, OUT>) cell_ijk(G, L.c, L.i, L.j, L.k);
        cell_xyz<LAYOUT>(G, L.c, L.i, L.j, L.k, (double)L.x[0], (double)L.x[1], (double)L.x[2], P.out_xyz + 3 * p);
    }
    if constexpr (OUT == O_SERIES) nan_rest(L, P);
}

// Quadtree transfer (after the crossing through face f of axis `axis`).  Where the cell's face entry
// names the neighbour, its record is already in the lane and the face coordinates carry over.
// Otherwise the subface holding the exit point (the first in order on an edge between two) gives
// the neighbour; in it, a face coordinate carries over when both cells span the same range on that
// axis and is mapped through the global coordinate otherwise.  A particle handed round a point in
// kQuadZeroRun zero-time crossings in a row (face velocities of split faces are averages,
// so they can circulate there) stops as stranded.
constexpr int kQuadZeroRun = 16;

template <int PREC, int OUT>
__device__ __forceinline__ int32_t quad_transfer(Lane<PREC>& L, const GridDev& G, const TrackParams& P,
                                                 const double* snap, int32_t axis, int32_t f, double xe, double dt,
                                                 int32_t nb, int32_t sub_base, uint32_t counts) {
    if (nb == FACE_OUT) return ST_BOUNDARY;
    if (nb == FACE_SPLIT) {
        int32_t q0 = sub_base;
        for (int32_t g = 0; g < f; ++g) q0 += (int32_t)((counts >> (5 * g)) & 31u);
        const int32_t q1 = q0 + (int32_t)((counts >> (5 * f)) & 31u);
        const int ta1 = (axis == 0) ? 1 : 0;
        const int ta2 = (axis == 2) ? 1 : 2;
        const double t1 = (ta1 == 0) ? (double)L.x[0] : (double)L.x[1];
        const double t2 = (ta2 == 1) ? (double)L.x[1] : (double)L.x[2];
        // the last subface is taken when no earlier one holds the point, so it is never tested
        int32_t hit = q1 - 1;
        for (int32_t q = q0; q < q1 - 1; ++q) {
            const double4 r = G.sub_rect[q];
            if (r.x <= t1 && t1 <= r.z && r.y <= t2 && t2 <= r.w) {
                hit = q;
                break;
            }
        }
        nb = (q1 > q0) ? G.sub_nb[hit] : -1;
        if (nb < 0) return ST_BOUNDARY;
        load_quad(G, nb, P.sign, L);
        if (!(L.fl & CF_ACTIVE)) return ST_INACTIVE_NB;
        const QuadBox& B = G.qbox[L.c];
        const QuadBox& N = G.qbox[nb];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (a == axis) continue;
            if (N.lo[a] == B.lo[a] && N.h[a] == B.h[a]) continue;   // same span: unchanged
            const double x = B.lo[a] + (double)L.x[a] * B.h[a];
            double l = (x - N.lo[a]) / N.h[a];
            l = (l < 0.0) ? 0.0 : l;
            l = (l > 1.0) ? 1.0 : l;
            L.x[a] = l;
        }
    }
    const int32_t nfl = L.fl;
    if (!(nfl & CF_ACTIVE)) return ST_INACTIVE_NB;
    // constant indices only: the lane state stays in registers
    L.x[0] = (axis == 0) ? 1.0 - xe : L.x[0];
    L.x[1] = (axis == 1) ? 1.0 - xe : L.x[1];
    L.x[2] = (axis == 2) ? 1.0 - xe : L.x[2];
    L.c = nb;
    if ((nfl & CF_SINK) && P.stop_at_sink) return ST_SINK;
    if ((int64_t)L.ncross >= P.max_steps) return ST_STEP_CAP;
    if (dt == 0.0) {
        if (++L.zrun >= kQuadZeroRun) {
            if constexpr (OUT == O_SERIES) {
                // stranded on the circuit: the position holds up to t_max
                double* row = P.snap_xyz + L.pid * (int64_t)P.n_snap * 3;
                while (L.ks < P.n_snap && snap[L.ks] <= P.t_max) {
                    cell_xyz<L_QUAD>(G, L.c, 0, 0, 0, (double)L.x[0], (double)L.x[1], (double)L.x[2],
                                     row + 3 * (int64_t)L.ks);
                    ++L.ks;
                }
            }
            return ST_STRANDED;
        }
    } else {
        L.zrun = 0;
    }
    return 0;
}

// End of a time step (transient flow): the particle continues in the next step's field from the
// same cell and position; it stops there if the cell is inactive, or a sink with stop_at_sink.
template <int PREC, int LAYOUT, bool BATCHED>
__device__ __forceinline__ int32_t step_switch(Lane<PREC>& L, const TrackParams& P) {
    L.g += 1;
    const GridDev& G2 = grid_of<BATCHED>(P, L.g);
    int32_t own;
    if constexpr (kPacked<LAYOUT>) {
        load_rec<PREC>(G2, L.c, P.sign, L.v1, L.v2, L.fl);
        own = L.fl;
    } else {
        own = G2.flags[L.c];
    }
    if (!(own & CF_ACTIVE)) return ST_INACTIVE_NB;
    if ((own & CF_SINK) && P.stop_at_sink) return ST_SINK;
    return 0;
}

// FNV-1a over the cells left: h = (h ^ c) (2^40 + 0x1b3).
__device__ __forceinline__ void hash_cell(unsigned long long& h, int32_t c) {
    const uint32_t lo = (uint32_t)h ^ (uint32_t)c;
    const uint64_t m = (uint64_t)lo * 0x1b3u;
    const uint32_t hi = (uint32_t)(h >> 32) * 0x1b3u + (lo << 8) + (uint32_t)(m >> 32);
    h = ((unsigned long long)hi << 32) | (uint32_t)m;
}

// One cell crossing (S1-S7).  Returns 0 to continue, or the final status.  `job`: the lane's
// slot for deferred snapshots, or null to write them at once.
//
// FP64: bound by the issue of its VALU instructions when the chip is full, and by their dependent
// chain when it is not.  So the common path is straight-line: estimates, the record of the next
// cell (its gather hides behind the arithmetic), one lean exit time, two lean advances; undecided
// lanes repair their values in branches (an axis' advance in ~6% of the wave steps: small A tau, whose
// expm1 has few bits to spare).  1e6 particles through a 100x100x10 field: 686 -> 462 VALU instructions
// per 64 crossings, kernel 2.93 -> 1.90 ms; repairing the logarithm and each expm1 in place, instead
// of the whole exit time or both advances, took the last 3%.
template <int PREC, int LAYOUT, int OUT, bool BATCHED, int CR>
__device__ __forceinline__ int32_t track_step(Lane<PREC>& L, const TrackParams& P, const double* snap,
                                              SnapJob<typename Real<PREC>::T>* job = nullptr) {
    using R = typename Real<PREC>::T;
    using X = typename Coord<PREC>::T;
    // the careful pass decides every evaluation in the general functions
    constexpr bool kLean = PREC == P64 && CR == ptcr::CR_FLAG;
    const GridDev& G = grid_of<BATCHED>(P, L.g);
    R u1[3], u2[3];
    int32_t fl;
    if constexpr (kPacked<LAYOUT>) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u1[a] = L.v1[a];
            u2[a] = L.v2[a];
        }
        fl = L.fl;
    } else {
        load_cell<PREC, LAYOUT>(G, L, P.sign, u1, u2, fl);
    }

    // earliest reachable face; exact ties go to the lowest axis.  c0, c1: the exit axis is 0, 1
    // (0 when no face is reachable)
    double dt = dinf();
    int32_t axis = -1;
    R xe = 0;
    Exit64 ex;
    R A[3], up[3];   // gradient and particle velocity of each axis at the step start
    if constexpr (PREC == P64) {
        if constexpr (kLean) {
            estimate_exit64(u1, u2, L.x, ex);
            axis = ex.c0 ? 0 : (ex.c1 ? 1 : 2);
        } else {
            step_au<PREC>(u1, u2, L.x, ex.A, ex.up);
            ex.sure = false;
        }
        if (!ex.sure) {
            exit_exact64<CR>(u1, u2, L.x, dt, axis, xe, L.amb);
            ex.c0 = axis <= 0;
            ex.c1 = axis == 1;
            ex.high = xe == 1.0;
        }
        xe = ex.high ? 1.0 : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            A[a] = ex.A[a];
            up[a] = ex.up[a];
        }
    } else {
        step_au<PREC>(u1, u2, L.x, A, up);
        exit_mix(u1, u2, L.x, A, up, ex, dt, axis, L.amb);
        xe = ex.high ? 1.0f : 0.0f;
    }
    const bool c0 = ex.c0, c1 = !ex.c0 && ex.c1;
    const bool hi = ex.high;
    const int32_t f = 2 * axis + (hi ? 1 : 0);
    const int32_t step = hi ? 1 : -1;

    // the neighbour across the exit face, and whether the particle moves into it
    int32_t nc = L.c;
    bool moves = false;
    int32_t face = 0, sub_base = 0;   // quadtree: the exit face's entry, the cell's subfaces
    uint32_t counts = 0u;
    if constexpr (LAYOUT == L_QUAD) {
        const int32_t n0 = hi ? L.nbf[1] : L.nbf[0], n1 = hi ? L.nbf[3] : L.nbf[2], n2 = hi ? L.nbf[5] : L.nbf[4];
        face = c0 ? n0 : (c1 ? n1 : n2);
        sub_base = L.sub_base;
        counts = L.counts;
        load_quad(G, (int)(axis >= 0) & (int)(face >= 0) ? face : L.c, P.sign, L);
    }
    if constexpr (LAYOUT == L_CELL) {
        // cell id stride of the axis, selected from uniform values (no per-lane multiply)
        const int32_t stride = c0 ? 1 : (c1 ? G.nx : G.plane);
        moves = (int)(axis >= 0) & (int)!(((uint32_t)fl >> (f & 31)) & ((1u << NB_OUT) | (1u << NB_INACTIVE)));
        const int32_t beside = L.c + (hi ? stride : -stride);
        nc = moves ? beside : L.c;
        // its record is gathered ahead of the arithmetic that is left
        load_rec<PREC>(G, nc, P.sign, L.v1, L.v2, L.fl);
    }

    if constexpr (kLean) {
        const double d = exit_time64_fast<CR, true>(ex, ex.sure, L.amb);
        dt = ex.sure ? d : dt;
    }

    // time limit: t_max, or the end of the current time step when that comes first (transient
    // flow); a face reached exactly at the limit is crossed
    double lim = P.t_max;
    bool next_step = false;
    if constexpr (BATCHED) {
        if (P.n_tsteps) {
            const double e = P.tstep_end[L.g];
            if (e < lim) {
                lim = e;
                next_step = L.g + 1 < P.n_tsteps;
            }
        }
    }
    if (axis < 0 && __builtin_isinf(lim)) {
        if constexpr (OUT == O_SERIES) write_snaps<PREC, LAYOUT, CR>(L, G, A, up, P, snap, dinf(), true);
        return ST_STRANDED;
    }
    const double t_exit = L.t + dt;
    // The limit comes first: every axis moves analytically to it and no face is crossed.  The
    // two axes other than the exit axis (axis 0 when no face is reachable) move by the same
    // code as in a crossing step, so lanes of a wave that stop at a limit (or at the end of a
    // time step) and lanes that cross a face diverge only in the exit axis' own advance.
    const bool at_lim = t_exit > lim;
    const double tau = at_lim ? lim - L.t : dt;

    if constexpr (OUT == O_SERIES) {
        if (at_lim) write_snaps<PREC, LAYOUT, CR>(L, G, A, up, P, snap, lim, true);
        else if (job) queue_snaps<PREC, LAYOUT, CR>(L, G, A, up, P, snap, t_exit, job);
        else write_snaps<PREC, LAYOUT, CR>(L, G, A, up, P, snap, t_exit, false);
    }

    // the two other axes: (1, 2), (0, 2) or (0, 1)
    const bool c2 = !c0 && !c1;
    const R Ax = c0 ? A[1] : A[0], ux = c0 ? up[1] : up[0];
    const R Ay = c2 ? A[1] : A[2], uy = c2 ? up[1] : up[2];
    const X xa = c0 ? L.x[1] : L.x[0], xb = c2 ? L.x[1] : L.x[2];
    X na, nb;
    if constexpr (kLean) {
        const double ya = Ax * tau, yb = Ay * tau;
        const double Ea = expm1_fast<CR>(ya, ux, L.amb), Eb = expm1_fast<CR>(yb, uy, L.amb);
        na = adv64_end(Ea, ya, ux, xa, tau);
        nb = adv64_end(Eb, yb, uy, xb, tau);
        if (!((int)(__builtin_fabs(ya) <= 36.0) & (int)(__builtin_fabs(yb) <= 36.0) & (int)plain(xa, xb))) {
#pragma unroll 1
            for (int q = 0; q < 2; ++q) {
                const double n = adv64_au<CR>(q ? Ay : Ax, q ? uy : ux, q ? xb : xa, tau, L.amb);
                na = q ? na : n;
                nb = q ? n : nb;
            }
        }
    } else if constexpr (PREC == P64) {
        na = adv64_au<CR>(Ax, ux, xa, tau, L.amb);
        nb = adv64_au<CR>(Ay, uy, xb, tau, L.amb);
    } else {
        na = adv_mix_au(Ax, ux, xa, tau);
        nb = adv_mix_au(Ay, uy, xb, tau);
    }
    if (at_lim) {
        const R Ae = c0 ? A[0] : (c1 ? A[1] : A[2]), ue = c0 ? up[0] : (c1 ? up[1] : up[2]);
        const X xc = c0 ? L.x[0] : (c1 ? L.x[1] : L.x[2]);
        X ne;
        if constexpr (PREC == P64) {
            ne = adv64<CR>(Ae, ue, xc, tau, L.amb);
        } else {
            ne = adv_mix_au(Ae, ue, xc, tau);
        }
        L.x[0] = c0 ? ne : na;
        L.x[1] = c1 ? ne : (c0 ? na : nb);
        L.x[2] = c2 ? ne : nb;
        L.t = lim;
        if constexpr (BATCHED) {
            if (next_step) return step_switch<PREC, LAYOUT, BATCHED>(L, P);
        }
        return axis < 0 ? ST_STRANDED : ST_MAX_TIME;
    }

    L.t = t_exit;
    L.ncross += 1;
    hash_cell(L.hash, L.c);
    if constexpr (OUT == O_PATH) {
        // pathline record: the cell left, the face, the time and the position on the face
        if (!P.path_count) {
            const int64_t q = L.pq++;
            if (q >= 0 && q < L.pend) {
                // one 40-byte record: a particle's records form one contiguous stream
                double xyz[3];
                cell_xyz<LAYOUT>(G, L.c, L.i, L.j, L.k, (double)(c0 ? (X)xe : na), (double)(c1 ? (X)xe : (c0 ? na : nb)),
                                 (double)(c2 ? (X)xe : nb), xyz);
                if (P.path_stage) {
                    stage_record(P, q, L.t, xyz[0], xyz[1], xyz[2], L.c, f);
                } else {
                    PathRec r;
                    r.t = L.t;
                    r.x = xyz[0];
                    r.y = xyz[1];
                    r.z = xyz[2];
                    r.cell = L.c;
                    r.face = f;
                    P.path_rec[q] = r;
                }
            } else {
                L.drop += 1u;
            }
        }
    }

    // the exit coordinate: on the face left, or on the same face seen from the neighbour
    if constexpr (LAYOUT == L_QUAD) {
        L.x[0] = c0 ? xe : na;
        L.x[1] = c1 ? xe : (c0 ? na : nb);
        L.x[2] = c2 ? xe : nb;
        return quad_transfer<PREC, OUT>(L, G, P, snap, axis, f, xe, dt, face, sub_base, counts);
    }
    int32_t nfl_sink, stop = 0;
    if constexpr (LAYOUT == L_CELL) {
        nfl_sink = (fl >> (NB_SINK + f)) & 1;
        if (!moves) stop = ((fl >> (NB_OUT + f)) & 1) ? ST_BOUNDARY : ST_INACTIVE_NB;
    } else {
        const int32_t ii = L.i + (axis == 0 ? step : 0);
        const int32_t jj = L.j + (axis == 1 ? step : 0);
        const int32_t kk = L.k + (axis == 2 ? step : 0);
        nfl_sink = 0;
        if (ii < 0 || ii >= G.nx || jj < 0 || jj >= G.ny || kk < 0 || kk >= G.nz) {
            stop = ST_BOUNDARY;
        } else {
            nc = (kk * G.ny + jj) * G.nx + ii;
            const int32_t nfl = G.flags[nc];
            if (!(nfl & CF_ACTIVE)) stop = ST_INACTIVE_NB;
            nfl_sink = (nfl & CF_SINK) ? 1 : 0;
        }
        moves = stop == 0;
    }
    const X xn = (hi != moves) ? (X)1 : (X)0;
    L.x[0] = c0 ? xn : na;
    L.x[1] = c1 ? xn : (c0 ? na : nb);
    L.x[2] = c2 ? xn : nb;
    if (!moves) return stop;
    L.c = nc;
    if constexpr (kTrackIJK<LAYOUT, OUT>) {
        L.i += c0 ? step : 0;
        L.j += c1 ? step : 0;
        L.k += c2 ? step : 0;
    }
    if (nfl_sink && P.stop_at_sink) return ST_SINK;
    if (L.ncross >= (int32_t)P.max_steps) return ST_STEP_CAP;   // max_steps < 2^31
    return 0;
}

// Block-level setup shared by both kernels: LDS tables, snapshot times and counters.
struct BlockCounters {
    unsigned int hist[8];
    unsigned long long cross;
    unsigned int amb;
    unsigned int drop;
};

template <bool TS> struct BlockShared;
template <> struct BlockShared<false> : BlockCounters {};
template <> struct BlockShared<true> : BlockCounters {
    double snap[kMaxSnapLds];
};

template <int PREC, bool TS>
__device__ __forceinline__ const double* block_setup(BlockShared<TS>& S, const TrackParams& P) {
    if (threadIdx.x < 8) S.hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        S.cross = 0ull;
        S.amb = 0u;
        S.drop = 0u;
    }
    if constexpr (PREC == P64) ptcr::lds_tables_init();   // the FP32 path has no table lookups
    const double* snap = P.snap_times;
    if constexpr (TS) {
        if (P.n_snap <= kMaxSnapLds) {
            for (int q = threadIdx.x; q < P.n_snap; q += blockDim.x) S.snap[q] = P.snap_times[q];
            snap = S.snap;
        }
    }
    __syncthreads();
    return snap;
}

__device__ __forceinline__ void block_flush(BlockCounters& S, const TrackParams& P,
                                            unsigned long long crossings, unsigned amb,
                                            unsigned drop) {
    // wave-level reduction of the crossing count, one LDS atomic per wave
    for (int off = 32; off > 0; off >>= 1) crossings += __shfl_down(crossings, off, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(&S.cross, crossings);
    if (amb) atomicAdd(&S.amb, amb);
    if (drop) atomicAdd(&S.drop, drop);
    __syncthreads();
    if (threadIdx.x == 0 && S.amb) atomicAdd(&P.counters->cr_ambiguous, (unsigned long long)S.amb);
    if (threadIdx.x == 0 && S.drop) atomicAdd(&P.counters->path_dropped, (unsigned long long)S.drop);
    if (threadIdx.x < 8 && S.hist[threadIdx.x])
        atomicAdd(&P.counters->status[threadIdx.x], (unsigned long long)S.hist[threadIdx.x]);
    if (threadIdx.x == 0 && S.cross) atomicAdd(&P.counters->crossings, S.cross);
}

// At the end of a particle in the fast FP64 kernels: if one of its correctly rounded evaluations
// was left undecided (L.amb != 0; a value within 2^-96 of a rounding midpoint, which the fast
// kernels do not settle -- that would take registers their loop does not have), hand it to the
// careful pass instead of finishing it.  Its input state in memory is untouched, so the careful
// kernel tracks it again from there; this call's crossings of it are taken back and nothing of it
// is written back.  Returns false (finish it) when there is no free entry; the undecided
// evaluations are then counted as such.
template <int PREC, int OUT>
__device__ __forceinline__ bool hand_off(Lane<PREC>& L, const TrackParams& P) {
    const unsigned long long q = atomicAdd(&P.counters->recheck_tracks, 1ull);
    const unsigned amb = L.amb;
    L.amb = 0u;
    if (q < (unsigned long long)P.recheck_cap) {
        P.recheck_pid[q] = (int32_t)L.pid;
        if constexpr (OUT == O_PATH) L.drop = L.drop0;
        return true;
    }
    atomicAdd(&P.counters->cr_ambiguous, (unsigned long long)amb);
    return false;
}

// Finish a particle of the fast kernels (st > 0), or hand it to the careful pass.
template <int PREC, int LAYOUT, int OUT, bool BATCHED>
__device__ __forceinline__ void finish_fast(Lane<PREC>& L, int32_t st, const TrackParams& P, unsigned int* s_hist,
                                            unsigned long long& crossings) {
    if constexpr (PREC == P64) {
        if (L.amb && hand_off<PREC, OUT>(L, P)) return;
    }
    finish<PREC, LAYOUT, OUT, BATCHED>(L, st, P, s_hist, crossings);
}

// ---------------------------------------------------------------------------------------------
// Waves per SIMD the register allocator is asked to fit.  FP64: four (110 to 128 VGPRs, scratch in two
// quadtree kernels only).  Five (96) spill live loop values: call times of four / five, 1e6 particles 1.93 /
// 1.99 ms, 6e6 in 64 groups 12.1 / 15.5, 2e5 with 100 snapshots 2.04 / 2.61, 5e5 transient 1.49 / 1.88.
// Asked for three, the kernels take up to 141: 1 to 2% shorter endpoint runs, 0.53 -> 0.50 ms on the
// quadtree, but 2.04 -> 2.24 with 100 snapshots.  Mixed: eight for endpoint runs (six: 1e6 particles 0.97 ->
// 0.95 ms, 5e5 transient 0.76 -> 0.83), six for timeseries and pathlines (eight spill: 2e5 with 100
// snapshots 1.12 -> 1.41 ms, 2e5 pathlines 0.98 -> 1.23).
// Rounding mode of the fast kernels: undecided evaluations go to the careful pass.
constexpr int kFastCr = ptcr::CR_FLAG;

template <int PREC, int OUT>
constexpr int kWavesStatic = waves_static(PREC, OUT);
// Persistent kernel: FP64 three (137 to 168 VGPRs).  Four spill 20 to 196 bytes per lane: call times of
// three / four, 1e6 particles 2.55 / 2.72 ms, 4e6 with wells, ordered, 12.3 / 13.5 and unordered 13.0 /
// 14.7 (the static kernel: 11.2 ordered, 17.7 unordered), 3e5 on a quadtree 0.84 / 0.99, 2e5 pathlines 1.85 /
// 2.53.  Mixed six for endpoint runs (1e6: eight 1.42 -> 1.82 ms), four otherwise.
template <int PREC, int OUT>
constexpr int kWavesPersistent = PREC == P64 ? 3 : (OUT == O_END ? 6 : 4);

template <int PREC, int LAYOUT, int OUT, bool BATCHED>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWavesStatic<PREC, OUT>)))
k_track_static(TrackParams P) {
    // Block b runs on die b mod 8.  The slots are dealt to the dies in chunks of kDieChunk
    // consecutive blocks, round robin: a die's concurrent blocks hold neighbouring particles
    // (they share record lines in its L2), and every die sweeps the whole ordered work, so no die
    // is left with a heavier part of it (gridDim.x is a multiple of 8 * kDieChunk).
    const int64_t die = blockIdx.x % kXcd, j = blockIdx.x / kXcd;
    const int64_t blk = ((j / kDieChunk) * kXcd + die) * kDieChunk + j % kDieChunk;
    if (blk * blockDim.x >= P.n) return;   // the whole block is padding
    const int64_t slot = blk * blockDim.x + threadIdx.x;
    __shared__ BlockShared<OUT == O_SERIES> S;
    const double* snap = block_setup<PREC, OUT == O_SERIES>(S, P);
    unsigned long long crossings = 0;
    Lane<PREC> L;
    L.amb = 0u;
    L.drop = 0u;
    if constexpr (OUT == O_SERIES && kPacked<LAYOUT>) {
        // timeseries: the wave steps its lanes together so that it can evaluate the deferred
        // snapshots of all of them at once
        using J = SnapJob<typename Real<PREC>::T>;
        extern __shared__ __align__(16) double dyn_lds[];   // blockDim.x slots
        J* jobs = reinterpret_cast<J*>(dyn_lds);
        J* W = jobs + (threadIdx.x & ~63u);
        jobs[threadIdx.x].cnt = 0;
        jobs[threadIdx.x].amb = 0u;
        wave_sync();
        int32_t st = ST_SKIP;
        if (slot < P.n) {
            L.pid = P.order ? (int64_t)P.order[slot] : slot;
            st = begin<PREC, LAYOUT, OUT, BATCHED>(L, P, snap);
        }
        for (;;) {
            if (st == 0) st = track_step<PREC, LAYOUT, OUT, BATCHED, kFastCr>(L, P, snap, &jobs[threadIdx.x]);
            wave_sync();
            const unsigned long long pend = __ballot(jobs[threadIdx.x].cnt > 0);
            const unsigned long long live = __ballot(st == 0);
            if (pend != 0ull && (__popcll(pend) >= kSnapFlush || live == 0ull))
                flush_snaps<PREC, LAYOUT, BATCHED, kFastCr>(W, P, snap);
            if (live == 0ull) break;
        }
        L.amb |= jobs[threadIdx.x].amb;   // undecided snapshots evaluated for this lane by the wave
        if (st > 0) finish_fast<PREC, LAYOUT, OUT, BATCHED>(L, st, P, S.hist, crossings);
    } else {
        if (slot < P.n) {
            L.pid = P.order ? (int64_t)P.order[slot] : slot;
            int32_t st = begin<PREC, LAYOUT, OUT, BATCHED>(L, P, snap);
            while (st == 0) st = track_step<PREC, LAYOUT, OUT, BATCHED, kFastCr>(L, P, snap);
            if (st > 0) finish_fast<PREC, LAYOUT, OUT, BATCHED>(L, st, P, S.hist, crossings);
        }
    }
    block_flush(S, P, crossings, L.amb, L.drop);
}

// Lane 0's value of a 64-bit quantity as a wave-uniform (scalar) value.
__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

template <int PREC, int LAYOUT, int OUT, bool BATCHED>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWavesPersistent<PREC, OUT>)))
k_track_persistent(TrackParams P) {
    __shared__ BlockShared<OUT == O_SERIES> S;
    const double* snap = block_setup<PREC, OUT == O_SERIES>(S, P);
    unsigned long long crossings = 0;
    const unsigned long long n = (unsigned long long)P.n;
    const int refill = P.refill;
    const int steps = P.steps_per_refill;
    const unsigned long long chunk = (unsigned long long)P.chunk;
    // Wave-uniform state: the wave's current chunk [cnext, cend) of queue slots, claimed with one
    // atomic; idle lanes are refilled from it at every refill point.
    unsigned long long cnext = 0, cend = 0;
    bool exhausted = false;  // every die's segment is empty
    // The slots are split into kXcd segments; a wave first drains its own die's segment
    // (L2 locality), then the following ones.
    const unsigned long long seg = (n + kXcd - 1) / kXcd;
    const int die = blockIdx.x % kXcd;
    int tried = 0;           // segments found empty so far (wave-uniform)
    Lane<PREC> L;
    L.amb = 0u;
    L.drop = 0u;
    L.pid = -1;
    for (;;) {
        const unsigned long long idle = __ballot(L.pid < 0);
        const int nidle = __popcll(idle);
        const unsigned long long avail = cend - cnext;
        if (nidle > 0 && (nidle >= refill || nidle == 64) && (avail > 0 || !exhausted)) {
            unsigned long long nbase = 0, nlen = 0;
            while (avail < (unsigned long long)nidle && !exhausted && nlen == 0) {
                const int sg = (die + tried) % kXcd;
                const unsigned long long lo = (unsigned long long)sg * seg;
                const unsigned long long hi = (lo + seg < n) ? lo + seg : n;
                // one claim covers every idle lane: at least a chunk, more when more lanes are idle
                // (a wave's first fill takes 64 consecutive slots, as in the static kernel)
                const unsigned long long want = (unsigned long long)nidle - avail;
                const unsigned long long amount = want > chunk ? want : chunk;
                unsigned long long base = 0;
                if ((threadIdx.x & 63) == 0) base = atomicAdd(&P.counters->queue[sg], amount);
                base = lo + uniform_u64(base);   // lane 0's claim, kept in scalar registers
                if (base < hi) {
                    nbase = base;
                    nlen = (hi - base < amount) ? hi - base : amount;
                }
                if (base + amount >= hi) {
                    ++tried;
                    if (tried == kXcd) exhausted = true;
                }
            }
            if (L.pid < 0) {
                const unsigned long long rank =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
                long long slot = -1;
                if (rank < avail) slot = (long long)(cnext + rank);
                else if (rank - avail < nlen) slot = (long long)(nbase + (rank - avail));
                if (slot >= 0) {
                    L.pid = P.order ? (int64_t)P.order[slot] : slot;
                    const int32_t st = begin<PREC, LAYOUT, OUT, BATCHED>(L, P, snap);
                    if (st != 0) {
                        if (st > 0) finish<PREC, LAYOUT, OUT, BATCHED>(L, st, P, S.hist, crossings);
                        L.pid = -1;
                    }
                }
            }
            if (avail >= (unsigned long long)nidle) {
                cnext += (unsigned long long)nidle;
            } else {
                const unsigned long long used = (unsigned long long)nidle - avail;
                cnext = nbase + (used < nlen ? used : nlen);
                cend = nbase + nlen;
            }
        }
        if (__ballot(L.pid >= 0) == 0ull) {
            if (exhausted && cnext >= cend) break;
            continue;
        }
        for (int s = 0; s < steps; ++s) {
            if (L.pid >= 0) {
                const int32_t st = track_step<PREC, LAYOUT, OUT, BATCHED, kFastCr>(L, P, snap);
                if (st != 0) {
                    finish_fast<PREC, LAYOUT, OUT, BATCHED>(L, st, P, S.hist, crossings);
                    L.pid = -1;
                }
            }
        }
    }
    block_flush(S, P, crossings, L.amb, L.drop);
}

// ---------------------------------------------------------------------------------------------
// One lane per axis: four lanes of a wave track one particle (lanes 4q .. 4q + 3; the lanes of axis
// 2 are a pair that computes the same).  FP64, packed structured records, static schedule.
//
// A wave alone on its SIMD issues one instruction every ~7 cycles whatever they depend on, so a call
// whose particles leave the chip empty takes its longest track times the instructions of a step.
// With the axes side by side a step has about half of them: one exit time and one advance instead
// of three estimates, an exit time and two advances, and hardly any selects.  Every lane evaluates
// its own axis' correctly rounded exit time, so the earliest one is found exactly and no estimates
// are needed.  An undecided rounding hands the particle over only where the track uses the value: the
// exit time of an axis that is within the selection margin of the earliest, and the advance of an axis
// that no face stops.  It pays while its four times as many waves are at most two per SIMD.  Call times
// against one lane per particle: 1,000 particles on 2,200-step paths 1.66 / 2.54 ms, 10,000 1.72 /
// 2.56, 30,000 2.38 / 2.66; 4,096 backward 152 / 267 us; 5,000 pathlines 373 / 619 us; 10,000 with
// 100 snapshots 0.64 / 1.09 ms; near the limit of the rule, at 32,000 particles: pathlines 592 / 672 us, 100
// snapshots 870 / 1,131, transient 370 / 454, with wells 570 / 717, to the outlet 254 / 289.
template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const uint64_t b = ptcr::bits_of(v);
    return ptcr::of_bits(((uint64_t)(uint32_t)dpp<CTRL>((int32_t)(b >> 32)) << 32) | (uint32_t)dpp<CTRL>((int32_t)b));
}
constexpr int quad_perm(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
// The two other axes, seen from lanes of axes (0, 1, 2, 2); one lane's value for the whole quad.
constexpr int kNext = quad_perm(1, 2, 0, 0), kOther = quad_perm(2, 0, 1, 1);
constexpr int kLane0 = quad_perm(0, 0, 0, 0), kLane1 = quad_perm(1, 1, 1, 1), kLane2 = quad_perm(2, 2, 2, 2);

// Own-axis velocities and the flag word of a cell.
__device__ __forceinline__ void load_axis(const GridDev& G, int32_t c, int32_t axis, double sign, double& u1, double& u2,
                                          int32_t& fl) {
    const CellRec64* rec = G.rec64 + (uint32_t)c;
    const double2 v = reinterpret_cast<const double2*>(rec)[axis];
    fl = rec->flags;
    u1 = v.x;
    u2 = v.y;
    if (sign != 1.0) {   // backward tracking (uniform across the launch)
        u1 = sign * u1;
        u2 = sign * u2;
    }
}

template <int OUT, bool BATCHED>
__global__ void __launch_bounds__(kBlock) k_track_axes(TrackParams P) {
    constexpr int CR = kFastCr;
    __shared__ BlockShared<OUT == O_SERIES> S;
    const double* snap = block_setup<P64, OUT == O_SERIES>(S, P);
    unsigned long long crossings = 0;
    Lane<P64> L;
    L.amb = 0u;
    L.drop = 0u;
    const int64_t slot = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
    const int lane = (int)(threadIdx.x & 3u);
    const int32_t own = lane < 3 ? lane : 2;
    if (slot < P.n) {   // the same for the lanes of a quad, as every status below
        L.pid = P.order ? (int64_t)P.order[slot] : slot;
        int32_t st = begin<P64, L_CELL, OUT, BATCHED>(L, P, snap);
        double x = 0.0, u1 = 0.0, u2 = 0.0;
        int32_t fl = 0, idx = 0;
        if (st >= 0 && st != ST_INVALID) {
            x = own == 0 ? L.x[0] : (own == 1 ? L.x[1] : L.x[2]);
            u1 = own == 0 ? L.v1[0] : (own == 1 ? L.v1[1] : L.v1[2]);
            u2 = own == 0 ? L.v2[0] : (own == 1 ? L.v2[1] : L.v2[2]);
            fl = L.fl;
            if constexpr (kTrackIJK<L_CELL, OUT>) idx = own == 0 ? L.i : (own == 1 ? L.j : L.k);
        }
        while (st == 0) {
            const GridDev& G = grid_of<BATCHED>(P, L.g);
            // exit time of the own axis (exit_time64)
            Exit64 ex;
            ex.Aw = u2 - u1;
            ex.upw = u1 + ex.Aw * x;
            const bool pos = ex.upw > 0.0, neg = ex.upw < 0.0;
            const bool out2 = u2 > 0.0, out1 = u1 < 0.0;
            ex.ue = pos ? u2 : u1;
            ex.D = (pos ? 1.0 : 0.0) - x;
            const bool feasible = ((int)pos & (int)out2) | ((int)neg & (int)out1);
            // the ranges of exit_time64_fast's quotients
            const double low = __builtin_fmin(__builtin_fmin(__builtin_fabs(ex.D), __builtin_fabs(ex.upw)), __builtin_fabs(ex.ue));
            const double high = __builtin_fmax(__builtin_fabs(ex.upw), __builtin_fabs(ex.Aw));
            bool ok = (int)(low >= 0x1p-100) & (int)(high <= 0x1p100);
            unsigned undecided = 0u;
            double dt = exit_time64_fast<CR, false>(ex, ok, undecided);
            int32_t face = 4 * own + (pos ? 2 : 0);   // bit 0: an exit time of -0.0
            if (feasible && !ok) {
                dt = exit_core64<CR>(ex.Aw, ex.upw, ex.D, ex.ue, undecided);
                dt = dt < dinf() ? dt : dinf();   // a time that is NaN is never the earliest
                face |= (int32_t)(ptcr::bits_of(dt) >> 63);   // zeros arise here only
                dt = __builtin_fabs(dt);
            }
            dt = feasible ? dt : dinf();
            // the earliest axis, ties to the lowest: face 2 axis + high of the smallest key, bits 1 to 3.  The
            // step's time is that of this axis with its sign, -0.0 to a face at 0 and +0.0 to one at 1, which
            // shows in the other axes' coordinates of -0.0 and in a time of -0.0; the minimum of both zeros
            // need not be it.  (The sign in the key: 10,000 particles on 2,200-step paths 1,723 -> 1,740 us;
            // as a branch on a time of zero 1,801.)
            const double d1 = dpp<kNext>(dt), d2 = dpp<kOther>(dt);
            const double dtm = __builtin_fmin(__builtin_fmin(dt, d1), d2);
            if (undecided && dt <= dtm * (1.0 + kFilterMargin)) L.amb += undecided;
            const int32_t key = (dt == dtm) ? face : 14;
            const int32_t fs = min(min(key, dpp<kNext>(key)), dpp<kOther>(key));
            const int32_t f = fs >> 1;
            const double dtw = ptcr::of_bits(ptcr::bits_of(dtm) | ((uint64_t)(uint32_t)fs << 63));
            const bool none = !(dtm < dinf());
            const int32_t axis = fs >> 2;
            const bool hi = fs & 2;
            const bool mine = !none && own == axis;

            const int32_t stride = axis == 0 ? 1 : (axis == 1 ? G.nx : G.plane);
            const bool moves = (int)!none & (int)!(((uint32_t)fl >> f) & ((1u << NB_OUT) | (1u << NB_INACTIVE)));
            const int32_t beside = L.c + (hi ? stride : -stride);
            const int32_t nc = moves ? beside : L.c;
            const int32_t fl0 = fl;
            double v1, v2;
            load_axis(G, nc, own, P.sign, v1, v2, fl);

            double lim = P.t_max;
            bool next_step = false;
            if constexpr (BATCHED) {
                if (P.n_tsteps) {
                    const double e = P.tstep_end[L.g];
                    if (e < lim) {
                        lim = e;
                        next_step = L.g + 1 < P.n_tsteps;
                    }
                }
            }
            // own coordinate after s, and its global value
            auto place = [&](double s, bool need = true) {
                return adv64<CR>(ex.Aw, ex.upw, x, s, L.amb, need);
            };
            auto world = [&](double xl) {
                const double o = own == 0 ? G.x0 : (own == 1 ? G.y0 : G.z0), d = own == 0 ? G.dx : (own == 1 ? G.dy : G.dz);
                return o + ((double)idx + xl) * d;
            };
            if (none && __builtin_isinf(lim)) {
                if constexpr (OUT == O_SERIES) {   // stranded for good: every snapshot left
                    for (; L.ks < P.n_snap; ++L.ks)
                        P.snap_xyz[(L.pid * P.n_snap + L.ks) * 3 + own] = world(place(snap[L.ks] - L.t));
                }
                st = ST_STRANDED;
                break;
            }
            const double t_exit = L.t + dtw;
            const bool at_lim = t_exit > lim;
            if constexpr (OUT == O_SERIES) {
                const double to = at_lim ? lim : t_exit;
                while (L.ks < P.n_snap && (at_lim ? L.s_next <= to : L.s_next < to)) {
                    P.snap_xyz[(L.pid * P.n_snap + L.ks) * 3 + own] = world(place(L.s_next - L.t));
                    ++L.ks;
                    L.s_next = (L.ks < P.n_snap) ? snap[L.ks] : dinf();
                }
            }
            const double xn = place(at_lim ? lim - L.t : dtw, (int)at_lim | (int)!mine);
            if (at_lim) {
                x = xn;
                L.t = lim;
                st = none ? ST_STRANDED : ST_MAX_TIME;
                if constexpr (BATCHED) {
                    if (next_step) {   // the same cell in the next step's field
                        L.g += 1;
                        load_axis(grid_of<BATCHED>(P, L.g), L.c, own, P.sign, u1, u2, fl);
                        st = !(fl & CF_ACTIVE) ? ST_INACTIVE_NB : (((fl & CF_SINK) && P.stop_at_sink) ? ST_SINK : 0);
                    }
                }
                continue;
            }
            L.t = t_exit;
            L.ncross += 1;
            hash_cell(L.hash, L.c);
            if constexpr (OUT == O_PATH) {
                if (!P.path_count) {
                    const int64_t q = L.pq++;
                    if (q >= 0 && q < L.pend) {
                        // the quad writes the 40-byte record: x, y, z, and time, cell and face
                        double* r = reinterpret_cast<double*>(P.path_rec + q);
                        if (lane < 3) {
                            r[1 + own] = world(mine ? (hi ? 1.0 : 0.0) : xn);
                        } else {
                            r[0] = L.t;
                            r[4] = ptcr::of_bits(((uint64_t)(uint32_t)f << 32) | (uint32_t)L.c);
                        }
                    } else if (lane == 0) {
                        L.drop += 1u;
                    }
                }
            }
            x = mine ? ((hi != moves) ? 1.0 : 0.0) : xn;
            if (!moves) {
                st = ((fl0 >> (NB_OUT + f)) & 1) ? ST_BOUNDARY : ST_INACTIVE_NB;
                continue;
            }
            L.c = nc;
            u1 = v1;
            u2 = v2;
            if constexpr (kTrackIJK<L_CELL, OUT>) idx += mine ? (hi ? 1 : -1) : 0;
            if (((fl0 >> (NB_SINK + f)) & 1) && P.stop_at_sink) st = ST_SINK;
            else if (L.ncross >= (int32_t)P.max_steps) st = ST_STEP_CAP;
        }
        // the first lane ends the particle, with the other lanes' coordinates and roundings
        const uint32_t amb = L.amb;
        L.amb = amb | (uint32_t)dpp<kNext>((int32_t)amb) | (uint32_t)dpp<kOther>((int32_t)amb);
        const double x0 = dpp<kLane0>(x), x1 = dpp<kLane1>(x), x2 = dpp<kLane2>(x);
        int32_t i = 0, j = 0, k = 0;
        if constexpr (kTrackIJK<L_CELL, OUT>) {
            i = dpp<kLane0>(idx);
            j = dpp<kLane1>(idx);
            k = dpp<kLane2>(idx);
        }
        if (st > 0) {
            L.x[0] = x0;
            L.x[1] = x1;
            L.x[2] = x2;
            L.i = i;
            L.j = j;
            L.k = k;
            if (lane == 0) finish_fast<P64, L_CELL, OUT, BATCHED>(L, st, P, S.hist, crossings);
        }
        if (lane != 0) L.amb = 0u;
    }
    block_flush(S, P, crossings, L.amb, L.drop);
}

// End of a call, one block, after every counter update: the counters go to the host block, or to the
// caller's counts (the fields of pt_summary that the device computes, in the order PT_COUNT_* of
// pt.h), and are cleared for the next run.  Part of the careful pass where there is one.  Without
// the copy command, its event and the reset kernel a call of 1000 particles takes 88 instead of
// 99 us, of which its tracking kernel 51 (events carried by the kernels' own launches: 93).
__device__ void publish(const TrackParams& P) {
    __shared__ unsigned long long w[32];
    const int t = (int)threadIdx.x;
    unsigned long long* c = reinterpret_cast<unsigned long long*>(P.counters);
    if (t < 32) {
        const unsigned long long v = __hip_atomic_load(c + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        w[t] = v;
        if (P.host_counters)
            __hip_atomic_store(reinterpret_cast<unsigned long long*>(P.host_counters) + t, v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(c + t, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __threadfence_system();
    __syncthreads();
    if (P.counts && t == 0) {
        const Counters& k = *reinterpret_cast<const Counters*>(w);
        int64_t tracked = 0;
        for (int q = 0; q < 8; ++q) {
            P.counts[2 + q] = (int64_t)k.status[q];
            tracked += (int64_t)k.status[q];
        }
        P.counts[0] = (int64_t)k.crossings;
        P.counts[1] = tracked;
        P.counts[10] = (int64_t)k.cr_ambiguous;
        P.counts[11] = P.path_pass == 1 ? (int64_t)k.crossings
                                        : (P.path_pass == 2 ? (int64_t)k.crossings - (int64_t)k.path_dropped : 0);
        P.counts[12] = P.path_pass == 2 ? (int64_t)k.path_dropped : 0;
        P.counts[13] = (int64_t)k.recheck_tracks;
        P.counts[14] = 0;
        P.counts[15] = 0;
    }
}

// The same as a kernel of its own, for calls without a careful pass.
__global__ void __launch_bounds__(64) k_publish(TrackParams P) { publish(P); }

// Careful pass, FP64: the particles the tracking kernel handed over are tracked again from their
// input state with every correctly rounded evaluation decided exactly (CR_EXACT), one thread per
// particle, snapshots and pathline records written again in full.  The list is usually empty; the
// grid is fixed and strides over it.  Its last block publishes the counters.
template <int LAYOUT, int OUT, bool BATCHED>
__global__ void __launch_bounds__(kBlock) k_track_careful(TrackParams P) {
    __shared__ BlockShared<OUT == O_SERIES> S;
    __shared__ bool last;
    const unsigned long long cnt = P.counters->recheck_tracks;
    const int64_t n = (int64_t)(cnt < (unsigned long long)P.recheck_cap ? cnt : (unsigned long long)P.recheck_cap);
    if (n == 0) {   // uniform across the grid (publishing clears a count that is 0)
        if (blockIdx.x == 0) publish(P);
        return;
    }
    const double* snap = block_setup<P64, OUT == O_SERIES>(S, P);
    unsigned long long crossings = 0;
    Lane<P64> L;
    L.amb = 0u;
    L.drop = 0u;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        L.pid = P.recheck_pid[q];
        int32_t st = begin<P64, LAYOUT, OUT, BATCHED>(L, P, snap);
        while (st == 0) st = track_step<P64, LAYOUT, OUT, BATCHED, ptcr::CR_EXACT>(L, P, snap);
        if (st > 0) finish<P64, LAYOUT, OUT, BATCHED>(L, st, P, S.hist, crossings);
    }
    block_flush(S, P, crossings, L.amb, L.drop);
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&P.counters->done, 1ull) == (unsigned long long)gridDim.x - 1ull;
    __syncthreads();
    if (last) {
        __threadfence();
        publish(P);
    }
}

// Allocation-free entry point: write the argument's bytes to dst.
__global__ void __launch_bounds__(256) k_fill(FillArgs A) {
    for (uint32_t q = threadIdx.x; q < A.nbytes; q += blockDim.x) A.dst[q] = A.bytes[q];
}

__global__ void __launch_bounds__(256) k_reset(ResetParams R) {
    unsigned long long* w = reinterpret_cast<unsigned long long*>(R.c);
    const int n = sizeof(Counters) / sizeof(unsigned long long);
    if ((int)threadIdx.x < n) w[threadIdx.x] = 0ull;
    for (int q = threadIdx.x; q < R.nsuper; q += blockDim.x) R.total[q] = 0u;
}

// ---------------------------------------------------------------------------------------------
// Block-wide inclusive scan of one value per thread: within each wave by shuffles, then the sums
// of the waves before it (two barriers; a scan in LDS over 1024 threads took twenty).  `part`:
// one entry per wave.
template <class T>
__device__ __forceinline__ T block_scan(T* part, T x) {
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T v = __shfl_up(x, off, 64);
        if (lane >= off) x += v;
    }
    __syncthreads();   // `part` may still be read from an earlier scan
    if (lane == 63) part[wave] = x;
    __syncthreads();
    for (int q = 0; q < wave; ++q) x += part[q];
    return x;
}

// Spatial ordering: the particles sorted by their starting cell (bucket), in two levels.  A
// returning global atomic for every particle runs at the L2 atomic units' ~25 G/s on random
// buckets, which made a one-level counting sort of 1.8e7 particles take 1 ms; here a tile makes one
// per super-bucket it holds.  Bound by launches and by the latency of each kernel's few loads up to
// ~1e6 particles: three kernels instead of six with a scan of the tile counts, 1e5 particles
// 57 -> 30 us, 1e6 67 -> 45 us, 1.8e7 462 -> 376 us.  The order inside a bucket is arbitrary: it only
// changes which lanes and dies process which particles, never a result.

// The group of particle p: the last group whose first particle is at or before p, searched in
// [lo, n_groups).
__device__ __forceinline__ int32_t group_at(const int64_t* offsets, int32_t lo, int32_t n_groups, int64_t p) {
    int32_t hi = n_groups;   // invariant: offsets[lo] <= p < offsets[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (offsets[mid] <= p) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Bucket of particle p.  Called with the lanes of a wave on consecutive particles (the first
// active lane on the lowest): the group of that lane is searched once with wave-uniform values,
// and only lanes past the end of its group search on their own.
__device__ __forceinline__ uint32_t sort_bucket(const SortParams& S, int64_t p) {
    int64_t key = 0;
    if (S.n_groups > 0) {
        const int64_t p0 = (int64_t)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)p >> 32)) << 32) |
                                     __builtin_amdgcn_readfirstlane((uint32_t)p));
        const int32_t g0 = group_at(S.group_offsets, 0, S.n_groups, p0);
        const int64_t end0 = (g0 + 1 < S.n_groups) ? S.group_offsets[g0 + 1] : INT64_MAX;
        const int32_t g = (p < end0) ? g0 : group_at(S.group_offsets, g0 + 1, S.n_groups, p);
        key = S.grid_base[S.group_grid[g]];
    }
    const int32_t c = S.cell[p];
    const int32_t st = S.status[p];
    if (c < 0 || (st != ST_ACTIVE && st != ST_MAX_TIME)) return 0u;
    key += c;
    const int64_t b = key >> S.shift;
    return (uint32_t)(b < S.nbuckets ? b : S.nbuckets - 1);
}

// Level 1: each tile keeps its particles' buckets, counts them per super-bucket, and claims a
// range of each super-bucket.
__global__ void __launch_bounds__(1024) k_sort_tiles(SortParams S) {
    __shared__ unsigned c[kMaxSuper];
    for (int q = threadIdx.x; q < S.nsuper; q += blockDim.x) c[q] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * S.tile;
    for (int q = threadIdx.x; q < S.tile; q += blockDim.x) {
        const int64_t p = base + q;
        if (p < S.n) {
            const uint32_t b = sort_bucket(S, p);
            S.bucket[p] = b;
            atomicAdd(&c[b / (uint32_t)S.fine], 1u);
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < S.nsuper; q += blockDim.x) {
        const unsigned v = c[q];
        if (v) S.cnt[(int64_t)blockIdx.x * S.nsuper + q] = atomicAdd(&S.total[q], v);
    }
}

// The first slot of each super-bucket, into at[0 .. nsuper): every block sums the totals itself.
__device__ __forceinline__ void super_starts(const SortParams& S, unsigned* at, unsigned* part) {
    const int per = (S.nsuper + (int)blockDim.x - 1) / (int)blockDim.x;
    const int q0 = (int)threadIdx.x * per;
    const int q1 = (q0 + per < S.nsuper) ? q0 + per : S.nsuper;
    unsigned sum = 0u;
    for (int q = q0; q < q1; ++q) sum += S.total[q];
    unsigned run = block_scan<unsigned>(part, sum) - sum;
    for (int q = q0; q < q1; ++q) {
        const unsigned v = S.total[q];
        at[q] = run;
        run += v;
    }
}

// Level 1, placement: each tile writes its particles (index and bucket) from the first slot of
// its share of each super-bucket on, ranked by LDS atomics.
__global__ void __launch_bounds__(1024) k_sort_spread(SortParams S) {
    __shared__ unsigned at[kMaxSuper];
    __shared__ unsigned part[16];
    super_starts(S, at, part);
    __syncthreads();
    // super-buckets that the tile does not hold have no entry in cnt: what is read for them is not used
    for (int q = threadIdx.x; q < S.nsuper; q += blockDim.x) at[q] += S.cnt[(int64_t)blockIdx.x * S.nsuper + q];
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * S.tile;
    for (int q = threadIdx.x; q < S.tile; q += blockDim.x) {
        const int64_t p = base + q;
        if (p < S.n) {
            const uint32_t b = S.bucket[p];
            const unsigned k = atomicAdd(&at[b / (uint32_t)S.fine], 1u);
            S.sidx[k] = (int32_t)p;
            S.sbucket[k] = b;
        }
    }
}

// Level 2: one block per super-bucket orders its range [lo, hi) by bucket: an LDS histogram of
// its `fine` buckets, the histogram's exclusive prefix sum, then LDS-atomic ranks.
__global__ void __launch_bounds__(kFineBlock) k_sort_fine(SortParams S) {
    __shared__ unsigned h[kFineMax];
    __shared__ unsigned part[16];
    __shared__ unsigned range[2];
    const int s = blockIdx.x;
    super_starts(S, h, part);
    __syncthreads();
    if (threadIdx.x == 0) {
        range[0] = h[s];
        range[1] = h[s] + S.total[s];
    }
    __syncthreads();
    const int64_t lo = range[0], hi = range[1];
    if (lo == hi) return;   // uniform: an empty super-bucket
    const uint32_t b0 = (uint32_t)s * (uint32_t)S.fine;
    for (int q = threadIdx.x; q < S.fine; q += kFineBlock) h[q] = 0u;
    __syncthreads();
    for (int64_t i = lo + threadIdx.x; i < hi; i += kFineBlock) atomicAdd(&h[S.sbucket[i] - b0], 1u);
    __syncthreads();
    // exclusive prefix sum of h[0, fine): each thread a run of consecutive buckets
    const int per = (S.fine + kFineBlock - 1) / kFineBlock;
    const int q0 = (int)threadIdx.x * per;
    const int q1 = (q0 + per < S.fine) ? q0 + per : S.fine;
    unsigned sum = 0u;
    for (int q = q0; q < q1; ++q) sum += h[q];
    unsigned run = block_scan<unsigned>(part, sum) - sum;
    for (int q = q0; q < q1; ++q) {
        const unsigned v = h[q];
        h[q] = run;
        run += v;
    }
    __syncthreads();
    for (int64_t i = lo + threadIdx.x; i < hi; i += kFineBlock) {
        const unsigned r = atomicAdd(&h[S.sbucket[i] - b0], 1u);
        S.order[lo + r] = S.sidx[i];
    }
}

// ---------------------------------------------------------------------------------------------
// Pathline offsets: inclusive prefix sum, in place, of the per-particle crossing counts written
// by the count pass (v = path_offsets + 1), and path_offsets[0] = 0.


// Tile b (kScanTile elements): scan within the tile, tile total to part[b].
__global__ void __launch_bounds__(kScanBlock) k_scan_tiles(ScanParams S) {
    __shared__ int64_t part[kScanBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer];
    int64_t sum = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        v[q] = (base + q < S.n) ? S.v[base + q] : 0;
        sum += v[q];
    }
    const int64_t incl = block_scan<int64_t>(part, sum);
    int64_t run = incl - sum;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        run += v[q];
        if (base + q < S.n) S.v[base + q] = run;
    }
    if (threadIdx.x == kScanBlock - 1) S.part[blockIdx.x] = incl;
}

// One workgroup: exclusive scan of the tile totals; writes the leading zero.
__global__ void __launch_bounds__(kScanBlock) k_scan_partials(ScanParams S) {
    __shared__ int64_t part[kScanBlock / 64];
    const int64_t per = (S.ntiles + kScanBlock - 1) / kScanBlock;
    const int64_t lo = (int64_t)threadIdx.x * per;
    const int64_t hi = (lo + per < S.ntiles) ? lo + per : S.ntiles;
    int64_t sum = 0;
    for (int64_t q = lo; q < hi; ++q) sum += S.part[q];
    int64_t run = block_scan<int64_t>(part, sum) - sum;
    for (int64_t q = lo; q < hi; ++q) {
        const int64_t h = S.part[q];
        S.part[q] = run;
        run += h;
    }
    if (threadIdx.x == 0 && S.head) *S.head = 0;
}

// Tile b adds the total of the tiles before it.
__global__ void __launch_bounds__(kScanBlock) k_scan_add(ScanParams S) {
    const int64_t add = S.part[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int64_t q = threadIdx.x; q < kScanTile; q += kScanBlock)
        if (base + q < S.n) S.v[base + q] += add;
}

// Quadtree grid load: each face's total flow (its subfaces summed in order), the velocities
// u = Q / (n V), the own flags, the first subface and the per-face subface counts.
__global__ void __launch_bounds__(256) k_build_quad(BuildQuadParams B) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= B.ncell) return;
    const QuadBox& X = B.box[c];
    const double V = (X.h[0] * X.h[1]) * X.h[2];
    const double n_c = B.por ? B.por[c] : B.por_scalar;
    const int32_t own = B.flags ? B.flags[c] : CF_ACTIVE;
    double Q[6];
    bool finite = true;
    uint32_t counts = 0u;
    for (int f = 0; f < 6; ++f) {
        const int32_t a = B.sub_off[6 * c + f], b = B.sub_off[6 * c + f + 1];
        double q = 0.0;
        for (int32_t s = a; s < b; ++s) {
            finite = finite && __builtin_isfinite(B.sub_q[s]);
            q += B.sub_q[s];
        }
        Q[f] = q;
        counts |= (uint32_t)(b - a) << (5 * f);
    }
    if (!finite) atomicOr(&B.err[0], 1);
    if (!(n_c > 0.0) || !__builtin_isfinite(n_c)) atomicOr(&B.err[1], 1);
    if (own & ~(CF_ACTIVE | CF_SINK)) atomicOr(&B.err[2], 1);
    if (B.balance_tol >= 0.0 && (own & CF_ACTIVE) && !(own & CF_SINK) && finite) {
        const double net = (Q[0] - Q[1]) + (Q[2] - Q[3]) + (Q[4] - Q[5]);
        double gross = 0.0;
        for (int32_t s = B.sub_off[6 * c]; s < B.sub_off[6 * c + 6]; ++s) gross += fabs(B.sub_q[s]);
        if (fabs(net) > B.balance_tol * gross) atomicOr(&B.err[3], 1);
    }
    const double d = n_c * V;
    QuadRec r;
    for (int f = 0; f < 6; ++f) r.u[f] = Q[f] / d;
    r.flags = own & (CF_ACTIVE | CF_SINK);
    r.sub_base = B.sub_off[6 * c];
    r.counts = counts;
    r.pad0 = 0;
    B.rec[c] = r;
    QuadFace F;
    for (int f = 0; f < 6; ++f) {
        const int32_t a = B.sub_off[6 * c + f], b = B.sub_off[6 * c + f + 1];
        int32_t nb = FACE_SPLIT;
        if (b == a) {
            nb = FACE_OUT;
        } else if (b == a + 1) {
            nb = B.sub_nb[a];
            if (nb >= 0) {
                const QuadBox& N = B.box[nb];
                for (int t = 0; t < 3; ++t)
                    if (t != (f >> 1) && !(N.lo[t] == X.lo[t] && N.h[t] == X.h[t])) nb = FACE_SPLIT;
            }
        }
        F.nb[f] = nb;
    }
    F.pad[0] = F.pad[1] = 0;
    B.face[c] = F;
}

// Grid load: validate the field and build both packed records of every cell.
__global__ void __launch_bounds__(256) k_build(BuildParams B) {
    const GridDev& G = B.g;
    const int64_t ncell = (int64_t)G.nx * G.ny * G.nz;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncell) return;
    const int64_t nx = G.nx, ny = G.ny, nz = G.nz;
    const int64_t plane = nx * ny;
    const int64_t k = c / plane, rem = c - k * plane;
    const int64_t j = rem / nx, i = rem - j * nx;
    const int64_t fx = (k * ny + j) * (nx + 1) + i;
    const int64_t fy = (k * (ny + 1) + j) * nx + i;
    const int64_t fz = (k * ny + j) * nx + i;
    const double q[6] = {G.qx[fx], G.qx[fx + 1], G.qy[fy], G.qy[fy + nx], G.qz[fz], G.qz[fz + plane]};
    const double n_c = G.por ? G.por[c] : G.por_scalar;
    const int32_t own = G.flags ? G.flags[c] : CF_ACTIVE;
    bool finite = true;
    for (int f = 0; f < 6; ++f) finite = finite && __builtin_isfinite(q[f]);
    if (!finite) atomicOr(&B.err[0], 1);
    if (!(n_c > 0.0) || !__builtin_isfinite(n_c)) atomicOr(&B.err[1], 1);
    if (own & ~(CF_ACTIVE | CF_SINK)) atomicOr(&B.err[2], 1);
    if (B.balance_tol >= 0.0 && (own & CF_ACTIVE) && !(own & CF_SINK) && finite) {
        const double net = (q[0] - q[1]) + (q[2] - q[3]) + (q[4] - q[5]);
        const double gross = fabs(q[0]) + fabs(q[1]) + fabs(q[2]) + fabs(q[3]) + fabs(q[4]) + fabs(q[5]);
        if (fabs(net) > B.balance_tol * gross) atomicOr(&B.err[3], 1);
    }
    const double d = n_c * G.V;
    int32_t word = own & (CF_ACTIVE | CF_SINK);
    const int64_t ncoord[3] = {i, j, k};
    const int64_t ndim[3] = {nx, ny, nz};
    const int64_t nstride[3] = {1, nx, plane};
    for (int f = 0; f < 6; ++f) {
        const int a = f >> 1;
        const int64_t s = (f & 1) ? 1 : -1;
        const int64_t cc = ncoord[a] + s;
        if (cc < 0 || cc >= ndim[a]) {
            word |= 1 << (NB_OUT + f);
        } else {
            const int32_t nf = G.flags ? G.flags[c + s * nstride[a]] : CF_ACTIVE;
            if (!(nf & CF_ACTIVE)) word |= 1 << (NB_INACTIVE + f);
            if (nf & CF_SINK) word |= 1 << (NB_SINK + f);
        }
    }
    CellRec64 r64;
    CellRec32 r32;
    for (int f = 0; f < 6; ++f) {
        const double u = q[f] / d;
        r64.u[f] = u;
        r32.u[f] = (float)u;
    }
    r64.flags = word;
    r64.pad0 = 0;
    r64.pad1 = 0.0;
    r32.flags = word;
    r32.pad0 = 0;
    B.rec64[c] = r64;
    B.rec32[c] = r32;
}

template <int PREC, int LAYOUT, int OUT, bool BATCHED>
const void* pick_sched(int sched) {
    if (sched == S_STATIC) return reinterpret_cast<const void*>(&k_track_static<PREC, LAYOUT, OUT, BATCHED>);
    return reinterpret_cast<const void*>(&k_track_persistent<PREC, LAYOUT, OUT, BATCHED>);
}

template <int PREC, int LAYOUT, int OUT>
const void* pick_batched(const KernelKey& k) {
    return k.batched ? pick_sched<PREC, LAYOUT, OUT, true>(k.sched) : pick_sched<PREC, LAYOUT, OUT, false>(k.sched);
}

template <int PREC, int LAYOUT>
const void* pick_out(const KernelKey& k) {
    if (k.out == O_SERIES) return pick_batched<PREC, LAYOUT, O_SERIES>(k);
    if (k.out == O_PATH) return pick_batched<PREC, LAYOUT, O_PATH>(k);
    return pick_batched<PREC, LAYOUT, O_END>(k);
}

}  // namespace

const void* track_kernel(const KernelKey& k) {
    if (k.layout == L_QUAD) {   // FP64, single grid
        if (k.out == O_SERIES) return pick_sched<P64, L_QUAD, O_SERIES, false>(k.sched);
        if (k.out == O_PATH) return pick_sched<P64, L_QUAD, O_PATH, false>(k.sched);
        return pick_sched<P64, L_QUAD, O_END, false>(k.sched);
    }
    if (k.precision == PMIX) return pick_out<PMIX, L_CELL>(k);
    if (k.layout == L_FACES) return pick_out<P64, L_FACES>(k);
    return pick_out<P64, L_CELL>(k);
}

template <int OUT>
const void* pick_axes(const KernelKey& k) {
    return k.batched ? reinterpret_cast<const void*>(&k_track_axes<OUT, true>)
                     : reinterpret_cast<const void*>(&k_track_axes<OUT, false>);
}

const void* axes_kernel(const KernelKey& k) {
    if (k.out == O_SERIES) return pick_axes<O_SERIES>(k);
    if (k.out == O_PATH) return pick_axes<O_PATH>(k);
    return pick_axes<O_END>(k);
}

template <int LAYOUT, int OUT>
const void* pick_careful(const KernelKey& k) {
    return k.batched ? reinterpret_cast<const void*>(&k_track_careful<LAYOUT, OUT, true>)
                     : reinterpret_cast<const void*>(&k_track_careful<LAYOUT, OUT, false>);
}

template <int LAYOUT>
const void* pick_careful_out(const KernelKey& k) {
    if (k.out == O_SERIES) return pick_careful<LAYOUT, O_SERIES>(k);
    if (k.out == O_PATH) return pick_careful<LAYOUT, O_PATH>(k);
    return pick_careful<LAYOUT, O_END>(k);
}

const void* careful_kernel(const KernelKey& k) {
    if (k.layout == L_QUAD) {   // single grid
        if (k.out == O_SERIES) return reinterpret_cast<const void*>(&k_track_careful<L_QUAD, O_SERIES, false>);
        if (k.out == O_PATH) return reinterpret_cast<const void*>(&k_track_careful<L_QUAD, O_PATH, false>);
        return reinterpret_cast<const void*>(&k_track_careful<L_QUAD, O_END, false>);
    }
    if (k.layout == L_FACES) return pick_careful_out<L_FACES>(k);
    return pick_careful_out<L_CELL>(k);
}

const void* reset_kernel() { return reinterpret_cast<const void*>(&k_reset); }
const void* fill_kernel() { return reinterpret_cast<const void*>(&k_fill); }
const void* publish_kernel() { return reinterpret_cast<const void*>(&k_publish); }
const void* sort_tiles_kernel() { return reinterpret_cast<const void*>(&k_sort_tiles); }
const void* sort_spread_kernel() { return reinterpret_cast<const void*>(&k_sort_spread); }
const void* sort_fine_kernel() { return reinterpret_cast<const void*>(&k_sort_fine); }
const void* scan_tiles_kernel() { return reinterpret_cast<const void*>(&k_scan_tiles); }
const void* scan_partials_kernel() { return reinterpret_cast<const void*>(&k_scan_partials); }
const void* scan_add_kernel() { return reinterpret_cast<const void*>(&k_scan_add); }
const void* build_kernel() { return reinterpret_cast<const void*>(&k_build); }
const void* build_quad_kernel() { return reinterpret_cast<const void*>(&k_build_quad); }

}  // namespace pt
