// The binary64 path's Kepler root and velocity, for the default step count
// (kep_options.fixed_iter == 0): the root of Eq. 1 to the last bits of
// binary64, which is where thirty Danby steps end, without taking thirty of
// them.  The binary32 solve of the mixed path (the starting-value table and one
// step, or its schedule) gives a starting value within ~4e-7 rad, and one
// binary64 step with Danby's second-order term from there leaves an error of
// order d^3 (below 1e-17 rad at e <= 0.9); above the table's range binary64
// Danby steps follow until they no longer move the root.  Every residual,
// slope, sine and cosine that fixes the root is binary64: the binary32 part
// only chooses where the binary64 step starts.
//
// An explicit step count (fixed_iter != 0) keeps Danby's plain iteration
// (Pol64, kepler64).
//
// What bounds it: VALU issue (0.82 of the cycles at 65,536 x 4 x 256, 123
// instructions a triple), about 60 binary64 and 45 binary32 ones in the
// formulation where thirty steps with library sine, cosine and three quotients
// each took ~4000.  Measured, thirty steps -> this root: chi-square 65,536 x 4 x
// 256 8.53 ms -> 222 us, gradient 65,536 x 4 x 256 10.0 ms -> 468 us, Gauss-Newton
// products 32,768 x 4 x 256 6.04 ms -> 410 us, Kepler's equation alone for
// 4,194,301 pairs 479 -> 25 us (a copy of those bytes takes 20).  Against the
// extended-precision oracle its errors are the smaller ones (E rms 6.0e-17
// against 9.9e-17 at e < 0.9, 9.0e-17 against 1.22e-16 up to 0.99).
#pragma once

#include <hip/hip_runtime.h>

#include "kep_device.h"
#include "kep_grad.h"
#include "kep_knots64.h"
#include "kep_policy.h"

namespace kep {

static_assert(KEP_KNOTS64_HALF == kSc64Half, "the knots span the same interval");

// The block's LDS copy of the correctly rounded knots, n = -kSc64Half ..
// kSc64Half (sin odd, cos even), in the layout of fill_sincos64_knots; every
// thread calls it and a block barrier follows.  Read instead of computed: the
// series left about an ulp in each knot, which near periapsis is multiplied by
// e/D in the root, and a read is the shorter prologue.
__device__ __forceinline__ void load_knots64(double2 *tab)
{
    for (int q = threadIdx.x; q < kSc64Knots; q += blockDim.x) {
        const int n = q - kSc64Half, i = n < 0 ? -n : n;
        const double s = kep_knots64[i][0];
        tab[q] = make_double2(n < 0 ? -s : s, kep_knots64[i][1]);
    }
}

// sin and cos of E, |E| <= 3.25 or NaN, from the knots n/64: the remainder
// y = E - n/64 is exact, |y| <= 2^-7 and a few binary32 ulps (sin y to y^5,
// cos y to y^6: remainders 3.5e-19 and 3.4e-22).  Each value is the knot's plus
// a correction 2^7 times smaller, so it carries the knot's rounding and one
// more.  A NaN reads knot 0 and gives NaN.
__device__ __forceinline__ void sincos64_knots(double E, const double2 *tab, double &s, double &c)
{
    const float fn = rintf((float)E * 64.0f);
    int n;
    __asm__("v_cvt_i32_f32 %0, %1" : "=v"(n) : "v"(fn));    // a NaN converts to 0
    const double y = fma((double)fn, -0.015625, E);
    const double2 k = tab[n + kSc64Half];
    const double y2 = y * y;
    const double sy = fma(y * y2, fma(y2, 1.0 / 120.0, -1.0 / 6.0), y);
    const double oy = y2 * fma(y2, fma(y2, 1.0 / 720.0, -1.0 / 24.0), 0.5);    // 1 - cos y
    s = k.x + fma(k.y, sy, -(k.x * oy));
    c = k.y - fma(k.x, sy, k.y * oy);
}

// Kepler's residual E - e sin E - M of a centred root (|E| >= |M|, same sign, to
// within its own error): E - M with its rounding error (fast two-sum), so that
// what is left is the rounding of sin E.
__device__ __forceinline__ double residual64(double E, double e, double s, double M)
{
    const double a = E - M;
    return fma(-e, s, a) + ((E - a) - M);
}

// A root E and what the velocity needs at it: sin E, cos E, D = 1 - e cos E and
// 1/D to the last bits.
struct Root64 {
    double E, s, c, D, rD;
};

// 1/D from an estimate r with relative error below 1e-6: two Newton steps.
__device__ __forceinline__ double rcp64_refine(double D, double r)
{
    r = fma(r, fma(-D, r, 1.0), r);
    return fma(r, fma(-D, r, 1.0), r);
}

// Binary64 Danby steps (one quotient: danby_delta's form) from E until a step
// leaves only an error of its fourth power, |step| <= 1e-5 D, at most 30; the
// iterate stays in [M - e, M + e] and in [-3.25, 3.25].  For e above the
// table's range, where the binary64 step from the binary32 root is not bounded
// by a scan.  Lanes without `todo` keep their values.
__device__ __forceinline__ void danby_finish64(double e, double M, bool todo, const double2 *knots, Root64 &r)
{
    const double lo = fmax(M - e, -3.25), hi = fmin(M + e, 3.25);
    for (int it = 0; it < 30; ++it) {
        if (!__any(todo)) break;
        if (todo) {
            double s, c;
            r.E = fmin(fmax(r.E, lo), hi);
            sincos64_knots(r.E, knots, s, c);
            const double f = residual64(r.E, e, s, M);
            const double f1 = fma(-e, c, 1.0);
            const double g = f * (0.5 * e * s);
            const double N = fma(f1, f1, -g), N2 = N * N;
            const double den = f1 * fma(f * f1, f * (e * c * (1.0 / 6.0)), fma(-g, N, N2));
            const double En = fmin(fmax(r.E - (f * N2) / den, lo), hi);
            const double d = En - r.E;
            r.E = En;
            todo = fabs(d) > 1e-5 * f1;
            if (todo) {
                sincos64_knots(En, knots, r.s, r.c);
            } else {
                const double d2 = d * d;
                const double sd = fma(d * d2, -1.0 / 6.0, d), od = 0.5 * d2;   // |d| <= 2e-5: d^4/24 is below 1e-20
                r.s = fma(c, sd, fma(-s, od, s));
                r.c = fma(-s, sd, fma(-c, od, c));
            }
        }
    }
}

// The root from its binary32 value E32 for the centred binary64 mean anomaly M
// (|M| <= pi): f = E - e sin E - M and D = 1 - e cos E in binary64, the step
// d = d1 - d1^2 e sin E / (2 D), d1 = -f/D (its error is below 2.4 |d1|^3 at
// e <= 0.9), sin and cos carried to E + d to second order.
__device__ __forceinline__ void refine_root64(double e, float E32, double M, bool far, const double2 *knots, Root64 &r)
{
    E32 = clamp_root(E32);
    const double E0 = (double)E32;
    double s, c;
    sincos64_knots(E0, knots, s, c);
    const double f = residual64(E0, e, s, M);
    const double D = fma(-e, c, 1.0);
    const double r0 = (double)rcp32((float)D);
    const double rD = fma(r0, fma(-D, r0, 1.0), r0);       // 1e-14: ample for a step of ~1e-7 rad
    const double d1 = -f * rD;
    const double d = fma(-d1, (0.5 * d1) * (e * s) * rD, d1);
    const double od = 0.5 * d * d;
    r.E = E0 + d;
    r.s = fma(c, d, fma(-s, od, s));
    r.c = fma(-s, d, fma(-c, od, c));
    // (a NaN stays as it is: the steps' clamps would make a number of it)
    if (__any(far)) danby_finish64(e, M, far && M == M, knots, r);
    r.D = fma(-e, r.c, 1.0);
    // D at E and at E + d differ by a relative ~1e-6 at most, unless steps followed
    r.rD = rcp64_refine(r.D, far ? (double)rcp32((float)r.D) : rD);
}

// The largest |M| that counts as centred: pi and more than any rounding of it, and
// short of the knot after pi (the starting-value table has one word past it).
constexpr double kCentred = 3.1416;

// |x| below which one subtraction of whole turns centres it (the rounding of x/(2 pi)
// is then below 1e-6 turns).
constexpr double kOneTurnStep = 0x1p33;

// An angle less the multiple of 2 pi nearest to it (2 pi in two parts), for every
// finite angle: one subtraction leaves |x| <= pi + |x| 2^-51, so large angles take
// several (two at 1e17, twenty at 1e308; per record, not per observation).  The
// table's index has no other bound: with one subtraction here and one in
// mean_anomaly64c it left its row from |M0| ~ 1e31.  The large ones stand before the
// others' code because the kernels are compiled best that way: gradient 65,536 x 4 x
// 256 468 us, 495 as one loop, 487 without the large ones (66 binary64 calls: 0.8% less
// time than without them on average, at most 1.1% more).
__host__ __device__ __forceinline__ double centre_angle(double x)
{
    if (__builtin_expect(fabs(x) >= kOneTurnStep, 0)) {
#pragma nounroll
        do {
            const double n = rint(x * kInvTwoPi);
            x = fma(-n, kTwoPiLo, fma(-n, kTwoPiHi, x));
        } while (fabs(x) > kCentred);
    }
    const double n = rint(x * kInvTwoPi);
    return fma(-n, kTwoPiLo, fma(-n, kTwoPiHi, x));
}

// A mean anomaly as r + 2 pi (k + k2), |M| < 2^54: r centred, k its whole turns as the
// product with 1/(2 pi) rounds them, k2 those that this rounding missed (M of 3.7e14
// next to an odd multiple of pi gave r = -3.169, a knot past its row).  k is exact and
// so is its product with either part of 2 pi.
__host__ __device__ __forceinline__ double centre_turns(double M, double &k, double &k2)
{
    k = rint(M * kInvTwoPi);
    double r = fma(-k, kTwoPiLo, fma(-k, kTwoPiHi, M));
    k2 = 0.0;
    if (fabs(r) > kCentred) {
        k2 = rint(r * kInvTwoPi);
        r = fma(-k2, kTwoPiLo, fma(-k2, kTwoPiHi, r));
    }
    return r;
}

// Per-planet constants of the centred binary64 mean anomaly.
struct Phase64c {
    double P, rP;   // rP = 1/P correctly rounded; NaN where it overflows (P below 2^-1024)
    double M0c;     // M0 reduced to [-pi, pi]
};

__host__ __device__ __forceinline__ Phase64c make_phase64c(double P, double M0)
{
    Phase64c p;
    p.P = P;
    const double rP = 1.0 / P;
    p.rP = rP <= 1.7976931348623157e308 ? rP : __builtin_nan("");
    p.M0c = centre_angle(M0);
    return p;
}

// The mean anomaly on [-pi, pi] (Eq. 6 with the bracket in binary64): the
// IEEE quotient q = (t - t0)/P (the product with the correctly rounded
// reciprocal and one correction by its exact remainder; the division itself
// where 1/P overflows), q less its nearest integer exactly, 2 pi times it plus
// M0 in one fused multiply-add, reduced once more with 2 pi in two parts.
// Each rounding is at a magnitude of at most 2 pi (4 pi before centring).
__host__ __device__ __forceinline__ double mean_anomaly64c(double tt, const Phase64c &p, double &q)
{
    if (p.rP == p.rP) {
        const double q0 = tt * p.rP;
        q = fma(fma(-q0, p.P, tt), p.rP, q0);
    } else {
        q = tt / p.P;
    }
    const double phi = q - rint(q);
    const double M = fma(phi, kTwoPiHi, p.M0c);
    const double n = rint(M * kInvTwoPi);
    return fma(phi - n, kTwoPiLo, fma(-n, kTwoPiHi, M));
}

// The binary64 policy of the dense kernels at the default step count.
struct Rec64R {            // 88 bytes
    Phase64c ph;
    double e, A, B;        // A = K b^2 cos w, B = -K b sin w  (b = sqrt(1 - e^2))
    Ecc32 k;               // of the binary32 starting solve
    TabPlace tp;           // its place in the starting-value table (toff -1: the schedule)
    int16_t niter;
    int16_t pad;
    int32_t pad2;
};

struct Pol64R {
    static constexpr bool kMixed = false;
    static constexpr int kTables = 2;      // the starting-value table and the sin/cos knots
    using Rec = Rec64R;
    using Obs = Obs64;
    using ModelAcc = Pol64::ModelAcc;
    using ChiAcc = Pol64::ChiAcc;

    static __device__ __forceinline__ bool setup(const DenseArgs &, double P, double K, double e, double w,
                                                 double M0, Rec &r)
    {
        const bool ok = planet_ok(P, K, e, w, M0);
        if (!ok) { P = 1.0; K = 0.0; e = 0.0; w = 0.0; M0 = 0.0; }
        r.ph = make_phase64c(P, M0);
        const double b2 = (1.0 - e) * (1.0 + e), b = sqrt(b2);
        double sw, cw;
        sincos(w, &sw, &cw);
        r.e = e;
        r.A = K * b2 * cw;
        r.B = -K * b * sw;
        r.k = make_ecc32(e);
        r.tp = table_place(e, true);
        r.niter = (int16_t)sched32(r.k.e);
        r.pad = 0;
        r.pad2 = 0;
        return ok;
    }

    static __device__ __forceinline__ void load_obs(const DenseArgs &a, int64_t k, Obs &o) { Pol64::load_obs(a, k, o); }
    static __device__ __forceinline__ void load_obs_model(const DenseArgs &a, int64_t k, Obs &o)
    {
        Pol64::load_obs_model(a, k, o);
    }

    // One planet (a wave-uniform record): v = (A cos E + B sin E) / (1 - e cos E),
    // the quotient corrected by its remainder.  tab, knots: the block's LDS tables.
    template <int NCH>
    static __device__ __forceinline__ void add_planet(const Rec &rr, const Obs (&o)[NCH], ModelAcc (&m)[NCH],
                                                      int max_iter, const uint32_t *tab, const double2 *knots)
    {
        const Phase64c ph = rr.ph;
        const double e = rr.e, A = rr.A, B = rr.B;
        double M[NCH];
        float M32[NCH], E32[NCH], sv[NCH], omc[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            double q;
            M[c] = mean_anomaly64c(o[c].tt, ph, q);
            M32[c] = (float)M[c];
        }
        PolMixed::solve<NCH, false>(rr.k, uniform_int(rr.niter), false, rr.tp, M32, E32, sv, omc, max_iter, tab);
        const bool far = uniform_int(rr.tp.toff) < 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            Root64 r;
            refine_root64(e, E32[c], M[c], far, knots, r);
            const double num = fma(A, r.c, B * r.s);
            const double v = num * r.rD;
            m[c].s += fma(fma(-v, r.D, num), r.rD, v);
        }
    }

    static __device__ __forceinline__ void model_init(ModelAcc &m) { m.s = 0.0; }
    static __device__ __forceinline__ double model_value(const ModelAcc &m) { return m.s; }
    static __device__ __forceinline__ void chi_init(ChiAcc &x) { x = 0.0; }
    static __device__ __forceinline__ bool obs_valid(const Obs &o) { return Pol64::obs_valid(o); }
    static __device__ __forceinline__ void chi_add_plain(ChiAcc &x, const ModelAcc &m, const Obs &o, double gam)
    {
        Pol64::chi_add_plain(x, m, o, gam);
    }
    static __device__ __forceinline__ bool chi_add(ChiAcc &x, const ModelAcc &m, const Obs &o, double gam,
                                                   double jit, bool has_jit)
    {
        return Pol64::chi_add(x, m, o, gam, jit, has_jit);
    }
    static __device__ __forceinline__ double chi_value(const ChiAcc &x) { return x; }
};

// ------------------------------------------------------------ derivatives
// Per-planet record of the binary64 gradient and Gauss-Newton products.
struct RecG64 {            // 112 bytes
    Phase64c ph;
    double e, b, rb, b2, K, cw, sw;   // b = sqrt(1 - e^2), rb = 1/b, b2 = 1 - e^2
    Ecc32 k;                          // of the binary32 starting solve, as Rec64R
    TabPlace tp;
    int16_t niter;
    int16_t pad;
};

__device__ __forceinline__ bool setup_g64(double P, double K, double e, double w, double M0, RecG64 &r)
{
    const bool ok = planet_ok(P, K, e, w, M0);
    if (!ok) { P = 1.0; K = 0.0; e = 0.0; w = 0.0; M0 = 0.0; }
    r.ph = make_phase64c(P, M0);
    r.e = e;
    r.b2 = (1.0 - e) * (1.0 + e);
    r.b = sqrt(r.b2);
    r.rb = 1.0 / r.b;
    r.K = K;
    sincos(w, &r.sw, &r.cw);
    r.k = make_ecc32(e);
    r.tp = table_place(e, true);
    r.niter = (int16_t)sched32(r.k.e);
    r.pad = 0;
    return ok;
}

// sin E, cos E, D = 1 - e cos E and 1/D of NCH observations of one planet (a
// wave-uniform record), and q = (t - t0)/P.  ROOT: the default step count
// (tab, knots as in Pol64R); else Danby's plain iteration, `fixed` steps (0: its
// schedule and convergence test).
template <bool ROOT, int NCH>
__device__ __forceinline__ void roots_g64(const RecG64 &rr, const double (&tt)[NCH], int fixed, int max_iter,
                                          const uint32_t *tab, const double2 *knots, Root64 (&r)[NCH],
                                          double (&q)[NCH])
{
    const Phase64c ph = rr.ph;
    const double e = rr.e;
    double M[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) M[c] = mean_anomaly64c(tt[c], ph, q[c]);
    if constexpr (ROOT) {
        float M32[NCH], E32[NCH], sv[NCH], omc[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) M32[c] = (float)M[c];
        PolMixed::solve<NCH, false>(rr.k, uniform_int(rr.niter), false, rr.tp, M32, E32, sv, omc, max_iter, tab);
        const bool far = uniform_int(rr.tp.toff) < 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) refine_root64(e, E32[c], M[c], far, knots, r[c]);
    } else {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            r[c].E = kepler64(M[c], e, M[c] >= 0.0 ? 1.0 : -1.0, fixed, max_iter);
            sincos(r[c].E, &r[c].s, &r[c].c);
            r[c].D = 1.0 - e * r[c].c;
            r[c].rD = 1.0 / r[c].D;
        }
    }
}

// dv/dK = cos(w+f) + e cos w = b (b cos w cos E - sin w sin E)/D: the velocity is
// K times it (the quotient corrected by its remainder).
__device__ __forceinline__ double dvdk_g64(const RecG64 &p, const Root64 &r)
{
    const double num = p.b * fma(p.b * p.cw, r.c, -(p.sw * r.s));
    const double v = num * r.rD;
    return fma(fma(-v, r.D, num), r.rD, v);
}

// The other terms of planet p's derivatives from sin E, cos E and 1/D, by the
// implicit-function relations (df/dM = b/D^2, df/de = sin E (D + 1 - e^2)/(b D^2)):
//   dv/dP = (2 pi K/P) q x[0], dv/de = K x[1], dv/dw = -K x[2], dv/dM0 = -K x[0];
// x[2] = sin(w+f) + e sin w in the form b (b sin w cos E + cos w sin E)/D, which
// does not cancel near apoapsis.
__device__ __forceinline__ void terms_g64(const RecG64 &p, double s, double c, double rD, double (&x)[3])
{
    const double bs = p.b * s;
    const double swf = fma(p.sw, c - p.e, p.cw * bs) * rD;        // sin(w + f)
    const double t = swf * rD;
    x[0] = t * (p.b * rD);
    x[1] = fma(-t, (s * p.rb) * fma(p.b2, rD, 1.0), p.cw);            // rD (D + b2) = 1 + b2 rD
    x[2] = p.b * rD * fma(p.b * p.sw, c, p.cw * s);
}

}  // namespace kep
