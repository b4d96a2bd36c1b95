// fv_fast.h -- the face arithmetic of fv_physics.h for cells of ordinary magnitude, in fewer
// instructions and with the same results, bit for bit.
//
// What bounds the stencil kernels is the issue of FP64 instructions, and half of a WENO3 + HLLC
// face is division and square root: a division as the compiler expands it (operands scaled, two
// Newton steps, a rounding step, fix-ups for every special operand) takes 61 cycles of a SIMD per
// wavefront, a square root 86, a fused multiply-add about 5 and the reciprocal estimate 17
// (measured, 8 wavefronts per SIMD). Three things are saved here:
//   * no scaling and no fix-up: those only matter for operands near the ends of the exponent
//     range, for zeros, infinities and NaN;
//   * one reciprocal for several denominators: 1/d_i = (1/(d_1 d_2 ..)) times the other ones,
//     then the last Newton step for each by itself. The rounding step q + (a - b q) y of every
//     quotient stays, so each is correctly rounded as before;
//   * exact rewriting: a factor of two moved through a product (fma(2t, q/2, x) = fma(t, q, x)),
//     minimum and maximum as single instructions, the physical flux only of the side of the
//     contact that the HLLC flux takes, selections made only where some lane needs them.
// All of this holds while no intermediate result leaves the normal range. That is made certain
// from two sides. Every cell that a face reads has to be "tame": each field zero or of magnitude
// 2^-200 .. 2^50 (the kernels look at the cells when they load them). And the quantities formed
// at a face that a division or a root depends on have to lie in the windows below; a face tells
// whether they do (the functions here return it). A wavefront with a face that they do not hold
// for, or whose cells are not tame, computes its faces with fv_physics.h instead.
//
// Measured with the whole step (SSP-RK; before and after): 2D 1024^2 WENO3 + HLLC, 16 steps,
// 2144 -> 1986 us; 256 samples of 256^2, 4 steps, 7.57 -> 6.88 ms; multilevel MUSCL + HLL run
// 55.7 -> 47.7 ms; 3D 200 x 161 x 130, 3 steps, 3.04 -> 2.81 ms; the face of the 2D kernel went
// from 363 VALU instructions with 15 reciprocal or root estimates to 312 with 8. With the short Roe,
// shallow-water and ideal MHD fluxes: 1000 x 601 Roe, 5 steps, 601 -> 539 us; 1000 x 750 shallow
// water, HLL, 8 steps, 490 -> 460 us; 512^2 MHD, Rusanov, 8 steps, 480 -> 463 us.
//
// Bounds behind the windows: a difference or a combination of tame values is zero or at least
// 2^-252 (one cancellation loses at most 52 bits); a WENO3 denominator lies in [2^-41, 2^212]
// and the product of four of them in [2^-164, 2^848]; with density and squared sound speed in
// [2^-100, 2^100], every speed is below 2^154 and every numerator is zero or above 2^-900, so
// remainders a - b q (106 bits below a) never become subnormal. Roe's averages and strengths,
// whose squared sound speed has that window too, and shallow water, with g h in the place of the
// squared sound speed, stay within the same bounds.
#pragma once

#include "fv_physics.h"

namespace fvk {

constexpr int kTameLo = -200, kTameHi = 50;   // exponents, as frexp gives them

// ---------------------------------------------------------------- quotients and roots

// 1/d to 2^-48 (the hardware estimate is good to 2^-24.3, one Newton step).
__device__ __forceinline__ double recip48(double d)
{
    const double y = __builtin_amdgcn_rcp(d);
    return __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
}

// y[i] = 1/d[i] within half a unit in the last place (2^-97 before its rounding) for N
// denominators whose product stays in the normal range, from one hardware reciprocal.
//
// The rounding step of a quotient can then fail where the reciprocal lies within that error of the
// middle of two numbers and has come out as the wrong one: denominators an odd number of units
// below a power of two (of all ones, whose reciprocal is 2^k (1 + 2^-53 + 2^-106), to about 30
// units), under the few numerators whose quotient is next to a middle itself (a power of two
// under all ones; 0x16666666666663 under 2 - 5 * 2^-52). One denominator by itself gets these
// right, since the hardware estimate does (this is the sequence that a division expands to).
// SHARP gets them right for several, with a cubic last step: one more operation each, taken where
// both operands come from the same few values of a nearly uniform flow. A WENO3 denominator and
// its numerator, sums of squares of squares and products with them, meet them by chance only
// (2^-44 for the denominator, times that of the numerator).
template <int N, bool SHARP = false>
__device__ __forceinline__ void recips(const double (&d)[N], double (&y)[N])
{
    if constexpr (N == 1) {
        y[0] = recip48(d[0]);
    } else if constexpr (N == 2) {
        const double r = recip48(d[0] * d[1]);
        y[0] = r * d[1];
        y[1] = r * d[0];
    } else {
        static_assert(N == 4, "one, two or four denominators");
        const double d01 = d[0] * d[1], d23 = d[2] * d[3];
        const double r = recip48(d01 * d23);
        const double r01 = r * d23, r23 = r * d01;
        y[0] = r01 * d[1];
        y[1] = r01 * d[0];
        y[2] = r23 * d[3];
        y[3] = r23 * d[2];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double e = __builtin_fma(-d[i], y[i], 1.0);
        if constexpr (SHARP) e = __builtin_fma(e, e, e);
        y[i] = __builtin_fma(e, y[i], y[i]);
    }
}

// a/b correctly rounded, with y from recips().
__device__ __forceinline__ double quotient(double a, double b, double y)
{
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}

// 1/b correctly rounded.
__device__ __forceinline__ double inverse(double b)
{
    const double d[1] = {b};
    double y[1];
    recips(d, y);
    return __builtin_fma(__builtin_fma(-b, y[0], 1.0), y[0], y[0]);
}

// sqrt(x) correctly rounded: Goldschmidt's iteration for the root g and half its reciprocal h
// from the hardware estimate, then two corrections by the residual x - g^2.
__device__ __forceinline__ double root(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    double h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

// ---------------------------------------------------------------- windows

// Running range of the high words of positive doubles (ordered like the doubles; a negative
// value falls below every positive one, infinities and NaN above every finite one).
struct HighRange {
    int lo = 0x7fffffff, hi = 0;
    __device__ __forceinline__ void add(double x)
    {
        const int h = __double2hiint(x);
        lo = h < lo ? h : lo;
        hi = h > hi ? h : hi;
    }
    // every value in [2^E0, 2^E1)
    template <int E0, int E1>
    __device__ __forceinline__ bool within() const
    {
        return lo >= ((1023 + E0) << 20) && hi < ((1023 + E1) << 20);
    }
};

// x in [2^E0, 2^E1), or -x if NEG.
template <int E0, int E1, bool NEG = false>
__device__ __forceinline__ bool in_window(double x)
{
    const uint32_t h = (uint32_t)__double2hiint(x) - ((uint32_t)(1023 + E0) << 20) - (NEG ? 0x80000000u : 0u);
    return h < ((uint32_t)(E1 - E0) << 20);
}

// Running exponents of the fields of loaded cells (a zero counts as exponent 0, as do
// infinities and NaN, which `bits` catches).
struct CellRange {
    int lo = 0, hi = 0;
    uint32_t bits = 0;
    template <bool FINITE>
    __device__ __forceinline__ void add(double v)
    {
        const int e = __builtin_amdgcn_frexp_exp(v);
        lo = e < lo ? e : lo;
        hi = e > hi ? e : hi;
        if (FINITE) {
            const uint32_t b = (uint32_t)__double2hiint(v) << 1;
            bits = b > bits ? b : bits;
        }
    }
    __device__ __forceinline__ bool tame() const
    {
        return lo > kTameLo && hi <= kTameHi && bits < 0xffe00000u;
    }
};

// Minimum and maximum of finite values (single instructions).
__device__ __forceinline__ double fmin1(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double fmax1(double a, double b) { return __builtin_fmax(a, b); }

// ---------------------------------------------------------------- reconstruction

// minmod of finite values: one of the two terms is always a zero.
__device__ __forceinline__ double minmod_finite(double a, double b)
{
    return fmax1(fmin1(a, b), 0.0) + fmin1(fmax1(a, b), 0.0);
}

// Numerators and denominators of weno3(a, b, c) and weno3(d, c, b) from the smoothness terms
// t = ((difference)^2 + eps)^2 of (a, b), (b, c) and (c, d).
__device__ __forceinline__ void weno3_terms(double a, double b, double c, double d, double tab,
                                            double tbc, double tcd, double* n, double* den)
{
    // 2 t1 (b + c)/2 + t0 (3b - a)/2 = t1 (b + c) + (t0/2)(3b - a)
    const double s = b + c, h = 0.5 * tbc;
    n[0] = __builtin_fma(tab, s, h * __builtin_fma(3.0, b, -a));
    n[1] = __builtin_fma(tcd, s, h * __builtin_fma(3.0, c, -d));
    den[0] = __builtin_fma(2.0, tab, tbc);
    den[1] = __builtin_fma(2.0, tcd, tbc);
}

// Smoothness term of two neighbouring cells (the sign of the difference does not matter).
__device__ __forceinline__ double weno3_smooth(double a, double b)
{
    const double d = b - a;
    const double t = __builtin_fma(d, d, 1e-6);
    return t * t;
}

// WENO3 states of every field at a face; terms(q, n, den) gives a field's two numerators and
// denominators. Two fields at a time: four denominators share a reciprocal.
template <int NF, class Terms>
__device__ __forceinline__ void weno3_states(const Terms& terms, double* UL, double* UR)
{
#pragma unroll
    for (int q = 0; q + 1 < NF; q += 2) {
        double n[4], d[4], y[4];
        terms(q, n, d);
        terms(q + 1, n + 2, d + 2);
        recips(d, y);
        UL[q] = quotient(n[0], d[0], y[0]);
        UR[q] = quotient(n[1], d[1], y[1]);
        UL[q + 1] = quotient(n[2], d[2], y[2]);
        UR[q + 1] = quotient(n[3], d[3], y[3]);
    }
    if constexpr (NF % 2) {
        constexpr int q = NF - 1;
        double n[2], d[2], y[2];
        terms(q, n, d);
        recips(d, y);
        UL[q] = quotient(n[0], d[0], y[0]);
        UR[q] = quotient(n[1], d[1], y[1]);
    }
}

// Left and right states of every field at a face from at(q, j), field q of cell i - 2 + j.
struct Reconstruct {
    template <int RECON, int NF, class Cells>
    __device__ __forceinline__ void states(const Cells& at, double* UL, double* UR)
    {
        if constexpr (RECON == REC_FIRST) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                UL[q] = at(q, 1);
                UR[q] = at(q, 2);
            }
        } else if constexpr (RECON == REC_MUSCL) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const double b = at(q, 1), c = at(q, 2), m = c - b;
                UL[q] = __builtin_fma(0.5, minmod_finite(b - at(q, 0), m), b);
                UR[q] = __builtin_fma(-0.5, minmod_finite(m, at(q, 3) - c), c);
            }
        } else if constexpr (RECON == REC_ENO2) {
#pragma unroll
            for (int q = 0; q < NF; ++q)
                reconstruct<REC_ENO2>(at(q, 0), at(q, 1), at(q, 2), at(q, 3), UL[q], UR[q]);
        } else {
            weno3_states<NF>([&](int q, double* n, double* d) {
                const double a = at(q, 0), b = at(q, 1), c = at(q, 2), e = at(q, 3);
                weno3_terms(a, b, c, e, weno3_smooth(a, b), weno3_smooth(b, c), weno3_smooth(e, c), n, d);
            }, UL, UR);
        }
    }
};

// The same for the faces of a march along one axis, each a cell further than the one before:
// WENO3 keeps the smoothness terms of the last two pairs of cells, and forms one of three anew.
template <int RECON, int NF>
struct MarchReconstruct {
    static constexpr bool KEEP = RECON == REC_WENO3;
    double ta[KEEP ? NF : 1], tb[KEEP ? NF : 1];   // of cells 0 and 1, 1 and 2 of the next face

    template <class Cells>
    __device__ __forceinline__ void start(const Cells& at)
    {
        if constexpr (KEEP) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                ta[q] = weno3_smooth(at(q, 0), at(q, 1));
                tb[q] = weno3_smooth(at(q, 1), at(q, 2));
            }
        }
    }
    template <int, int, class Cells>
    __device__ __forceinline__ void states(const Cells& at, double* UL, double* UR)
    {
        if constexpr (KEEP) {
            weno3_states<NF>([&](int q, double* n, double* d) {
                const double a = at(q, 0), b = at(q, 1), c = at(q, 2), e = at(q, 3);
                const double tc = weno3_smooth(e, c);
                weno3_terms(a, b, c, e, ta[q], tb[q], tc, n, d);
                ta[q] = tb[q];
                tb[q] = tc;
            }, UL, UR);
        } else {
            Reconstruct().states<RECON, NF>(at, UL, UR);
        }
    }
};

// ---------------------------------------------------------------- Euler

// Primitives of both sides of a face. False unless densities and squared sound speeds are
// positive and in [2^-100, 2^100).
template <int DIM>
__device__ __forceinline__ bool euler_prims(const double* UL, const double* UR, const Phys& ph,
                                            EulerPrim<DIM>& wl, EulerPrim<DIM>& wr)
{
    wl.ir = inverse(UL[0]);
    wr.ir = inverse(UR[0]);
    double kl = 0.0, kr = 0.0;   // twice the kinetic energies
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        wl.u[k] = UL[1 + k] * wl.ir;
        wr.u[k] = UR[1 + k] * wr.ir;
        kl = (k == 0) ? UL[1] * wl.u[0] : kl + (UL[1 + k] * wl.u[k]);
        kr = (k == 0) ? UR[1] * wr.u[0] : kr + (UR[1 + k] * wr.u[k]);
    }
    wl.p = ph.gm1 * __builtin_fma(-0.5, kl, UL[DIM + 1]);
    wr.p = ph.gm1 * __builtin_fma(-0.5, kr, UR[DIM + 1]);
    const double xl = (ph.gamma * wl.p) * wl.ir, xr = (ph.gamma * wr.p) * wr.ir;
    wl.c = root(xl);
    wr.c = root(xr);
    HighRange r;
    r.add(UL[0]);
    r.add(UR[0]);
    r.add(xl);
    r.add(xr);
    return r.within<-100, 100>();
}

// Some lane of the wavefront has c.
__device__ __forceinline__ bool any_lane(bool c) { return __ballot(c) != 0ull; }

// HLL's combination of NF fields with physical fluxes FL, FR and speeds SL < SR.
template <int NF>
__device__ __forceinline__ bool hll_tame(const double* UL, const double* UR, const double* FL,
                                         const double* FR, double SL, double SR, double* Fh)
{
    const double d[1] = {SR - SL};
    double y[1];
    recips(d, y);
    const double slsr = SL * SR;
#pragma unroll
    for (int q = 0; q < NF; ++q)
        Fh[q] = quotient(((SR * FL[q]) - (SL * FR[q])) + (slsr * (UR[q] - UL[q])), d[0], y[0]);
    const bool takeL = (SL >= 0.0), takeR = (SR <= 0.0);
    if (any_lane(takeL || takeR)) {
#pragma unroll
        for (int q = 0; q < NF; ++q) Fh[q] = takeL ? FL[q] : (takeR ? FR[q] : Fh[q]);
    }
    return in_window<-150, 155>(d[0]);
}

// The HLLC flux of euler_numflux. The side K that decides (the supersonic side, or the side of
// the contact) is chosen first, and only its physical flux and star state are formed.
template <int DIM>
__device__ __forceinline__ bool hllc_tame(const double* UL, const double* UR, const EulerPrim<DIM>& wl,
                                          const EulerPrim<DIM>& wr, int nd, double* Fh)
{
    constexpr int NF = DIM + 2;
    const double uL = pick<DIM>(wl.u, nd), uR = pick<DIM>(wr.u, nd);
    const double SL = fmin1(uL - wl.c, uR - wr.c);
    const double SR = fmax1(uL + wl.c, uR + wr.c);
    const double eL = SL - uL, eR = SR - uR;
    const double DL = UL[0] * eL;
    const double DR = UR[0] * eR;
    const double num = (wr.p - wl.p) + __builtin_fma(pick<DIM>(UL + 1, nd), eL, -(pick<DIM>(UR + 1, nd) * eR));
    const double den[1] = {DL - DR};
    double y1[1];
    recips(den, y1);
    const double Ss = quotient(num, den[0], y1[0]);
    const bool takeL = (SL >= 0.0), takeR = (SR <= 0.0);
    const bool left = takeL || (!takeR && Ss >= 0.0);
    const double SK = left ? SL : SR;
    const double DK = left ? DL : DR;
    const double uK = left ? uL : uR;
    const double pK = left ? wl.p : wr.p;
    const double irK = left ? wl.ir : wr.ir;
    double UK[NF], vK[DIM];
#pragma unroll
    for (int q = 0; q < NF; ++q) UK[q] = left ? UL[q] : UR[q];
#pragma unroll
    for (int k = 0; k < DIM; ++k) vK[k] = (k == nd) ? uK : (left ? wl.u[k] : wr.u[k]);
    double FK[NF];
    FK[0] = pick<DIM>(UK + 1, nd);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const double a = UK[1 + k] * uK;
        FK[1 + k] = (k == nd) ? (a + pK) : a;
    }
    FK[DIM + 1] = (UK[DIM + 1] + pK) * uK;
    const double d2[2] = {SK - Ss, DK};
    double y2[2];
    recips<2, true>(d2, y2);
    const double f = quotient(DK, d2[0], y2[0]);
    double Us[NF];
    Us[0] = f;
#pragma unroll
    for (int k = 0; k < DIM; ++k) Us[1 + k] = (k == nd) ? (f * Ss) : (f * vK[k]);
    Us[DIM + 1] = f * __builtin_fma(UK[DIM + 1], irK, (Ss - uK) * (Ss + quotient(pK, DK, y2[1])));
#pragma unroll
    for (int q = 0; q < NF; ++q) Fh[q] = __builtin_fma(SK, Us[q] - UK[q], FK[q]);
    if (any_lane(takeL || takeR)) {
#pragma unroll
        for (int q = 0; q < NF; ++q) Fh[q] = (takeL || takeR) ? FK[q] : Fh[q];
    }
    return in_window<-60, 300, true>(den[0]) && in_window<-300, 300>(d2[0] * d2[1]);
}

// harten_fix of both speeds: its division where some lane is inside a fan.
__device__ __forceinline__ void harten_tame(double l1, double fan1, double l3, double fan3, double& g1,
                                            double& g3)
{
    g1 = fabs(l1);
    g3 = fabs(l3);
    if (any_lane(g1 < fan1 || g3 < fan3)) {
        g1 = harten_fix(l1, fan1);
        g3 = harten_fix(l3, fan3);
    }
}

// The Roe flux of euler_numflux: one reciprocal for the averages, one for the strengths (eight
// divisions and three more roots before).
template <int DIM>
__device__ __forceinline__ bool roe_tame(const double* UL, const double* UR, const EulerPrim<DIM>& wl,
                                         const EulerPrim<DIM>& wr, const double* FL, const double* FR,
                                         int nd, double* Fh, const Phys& ph)
{
    const double sqL = root(UL[0]);
    const double sqR = root(UR[0]);
    const double wsum[1] = {sqL + sqR};
    double yw[1];
    recips(wsum, yw);
    const double hL = (UL[DIM + 1] + wl.p) * wl.ir;
    const double hR = (UR[DIM + 1] + wr.p) * wr.ir;
    double ua[DIM];
#pragma unroll
    for (int k = 0; k < DIM; ++k) ua[k] = quotient((sqL * wl.u[k]) + (sqR * wr.u[k]), wsum[0], yw[0]);
    const double ha = quotient((sqL * hL) + (sqR * hR), wsum[0], yw[0]);
    double usq = ua[0] * ua[0];
#pragma unroll
    for (int k = 1; k < DIM; ++k) usq = usq + (ua[k] * ua[k]);
    const double csq[1] = {ph.gm1 * (ha - (0.5 * usq))};
    const double ca = root(csq[0]);
    double yc[1];
    recips(csq, yc);
    const double c2 = 2.0 * csq[0], y2 = 0.5 * yc[0];
    const double rhoa = sqL * sqR;
    const double una = pick<DIM>(ua, nd);
    const double unL = pick<DIM>(wl.u, nd), unR = pick<DIM>(wr.u, nd);
    const double jr = UR[0] - UL[0];
    const double jp = wr.p - wl.p;
    const double rj = (rhoa * ca) * (unR - unL);
    const double s1 = quotient(jp - rj, c2, y2);
    const double s2 = jr - quotient(jp, csq[0], yc[0]);
    const double s3 = quotient(jp + rj, c2, y2);
    const double fan1 = 0.5 * fmax1(0.0, (unR - wr.c) - (unL - wl.c));
    const double fan3 = 0.5 * fmax1(0.0, (unR + wr.c) - (unL + wl.c));
    double l1, l3;
    harten_tame(una - ca, fan1, una + ca, fan3, l1, l3);
    const double g1 = l1 * s1, g2 = fabs(una) * s2, g3 = l3 * s3;
    double gs[DIM];
#pragma unroll
    for (int k = 0; k < DIM; ++k) gs[k] = fabs(una) * (rhoa * (wr.u[k] - wl.u[k]));
    double diss[DIM + 2];
    diss[0] = (g1 + g2) + g3;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const bool n = (k == nd);
        double t = (g1 * (n ? (ua[k] - ca) : ua[k])) + (g2 * ua[k]);
        t = n ? t : (t + gs[k]);
        diss[1 + k] = t + (g3 * (n ? (ua[k] + ca) : ua[k]));
    }
    double te = (g1 * (ha - (una * ca))) + (g2 * (0.5 * usq));
#pragma unroll
    for (int k = 0; k < DIM; ++k) te = (k == nd) ? te : (te + (gs[k] * ua[k]));
    diss[DIM + 1] = te + (g3 * (ha + (una * ca)));
#pragma unroll
    for (int q = 0; q < DIM + 2; ++q) Fh[q] = 0.5 * ((FL[q] + FR[q]) - diss[q]);
    return in_window<-100, 100>(csq[0]);
}

// ---------------------------------------------------------------- shallow water

// swe_numflux; depths and squared celerities in [2^-100, 2^100).
template <int DIM, int FLUX>
__device__ __forceinline__ bool swe_tame(const double* UL, const double* UR, int nd, double* Fh,
                                         const Phys& ph)
{
    constexpr int NF = DIM + 1;
    SwePrim<DIM> wl, wr;
    wl.ih = inverse(UL[0]);
    wr.ih = inverse(UR[0]);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        wl.u[k] = UL[1 + k] * wl.ih;
        wr.u[k] = UR[1 + k] * wr.ih;
    }
    const double xl = ph.grav * UL[0], xr = ph.grav * UR[0];
    wl.c = root(xl);
    wr.c = root(xr);
    HighRange r;
    r.add(UL[0]);
    r.add(UR[0]);
    r.add(xl);
    r.add(xr);
    double FL[NF], FR[NF];
    swe_flux<DIM>(UL, wl, nd, FL, ph);
    swe_flux<DIM>(UR, wr, nd, FR, ph);
    const double uL = pick<DIM>(wl.u, nd), uR = pick<DIM>(wr.u, nd);
    if constexpr (FLUX == FLUX_RUSANOV) {
        const double s = fmax1(fabs(uL) + wl.c, fabs(uR) + wr.c);
#pragma unroll
        for (int q = 0; q < NF; ++q) Fh[q] = 0.5 * ((FL[q] + FR[q]) - (s * (UR[q] - UL[q])));
        return r.within<-100, 100>();
    } else if constexpr (FLUX == FLUX_HLL) {
        const double SL = fmin1(uL - wl.c, uR - wr.c);
        const double SR = fmax1(uL + wl.c, uR + wr.c);
        return hll_tame<NF>(UL, UR, FL, FR, SL, SR, Fh) && r.within<-100, 100>();
    } else {
        const double sqL = root(UL[0]);
        const double sqR = root(UR[0]);
        const double xa = ph.grav * (0.5 * (UL[0] + UR[0]));
        r.add(xa);
        const double ca = root(xa);
        const double d[2] = {sqL + sqR, ca};
        double y[2];
        recips<2, true>(d, y);
        double ua[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) ua[k] = quotient((sqL * wl.u[k]) + (sqR * wr.u[k]), d[0], y[0]);
        const double una = pick<DIM>(ua, nd);
        const double jh = UR[0] - UL[0];
        const double jq = (pick<DIM>(UR + 1, nd) - pick<DIM>(UL + 1, nd)) - (una * jh);
        const double jc = quotient(jq, d[1], y[1]);
        const double s1 = 0.5 * (jh - jc);
        const double s2 = 0.5 * (jh + jc);
        const double fan1 = 0.5 * fmax1(0.0, (uR - wr.c) - (uL - wl.c));
        const double fan2 = 0.5 * fmax1(0.0, (uR + wr.c) - (uL + wl.c));
        double l1, l2;
        harten_tame(una - ca, fan1, una + ca, fan2, l1, l2);
        const double g1 = l1 * s1, g2 = l2 * s2;
        double diss[NF];
        diss[0] = g1 + g2;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            const bool n = (k == nd);
            double t = g1 * (n ? (una - ca) : ua[k]);
            t = n ? t : (t + (fabs(una) * ((UR[1 + k] - UL[1 + k]) - (ua[k] * jh))));
            diss[1 + k] = t + (g2 * (n ? (una + ca) : ua[k]));
        }
#pragma unroll
        for (int q = 0; q < NF; ++q) Fh[q] = 0.5 * ((FL[q] + FR[q]) - diss[q]);
        return r.within<-100, 100>();
    }
}

// ---------------------------------------------------------------- ideal MHD

// Primitives and fast speed of one side; false unless the density and a^2 + b^2 are in [2^-100,
// 2^100) and the discriminant is zero or in [2^-400, 2^400).
__device__ __forceinline__ bool mhd_side(const double* U, int nd, const Phys& ph, MhdPrim& w, double& cf)
{
    w.ir = inverse(U[0]);
#pragma unroll
    for (int k = 0; k < 3; ++k) w.u[k] = U[1 + k] * w.ir;
    const double ke = 0.5 * (((U[1] * w.u[0]) + (U[2] * w.u[1])) + (U[3] * w.u[2]));
    w.pb = 0.5 * (((U[5] * U[5]) + (U[6] * U[6])) + (U[7] * U[7]));
    w.p = ph.gm1 * ((U[4] - ke) - w.pb);
    const double a2 = (ph.gamma * w.p) * w.ir;
    const double b2 = (2.0 * w.pb) * w.ir;
    const double bn = (nd == 0) ? U[5] : ((nd == 1) ? U[6] : U[7]);
    const double bn2 = (bn * bn) * w.ir;
    const double s = a2 + b2;
    const double disc = fmax1(0.0, (s * s) - ((4.0 * a2) * bn2));
    const bool some = in_window<-400, 400>(disc);
    const double rd = some ? root(disc) : 0.0;
    cf = root(0.5 * (s + rd));
    HighRange r;
    r.add(U[0]);
    r.add(s);
    return (some || disc == 0.0) && r.within<-100, 100>();
}

// mhd_numflux.
template <int FLUX>
__device__ __forceinline__ bool mhd_tame(const double* UL, const double* UR, int nd, double* Fh,
                                         const Phys& ph)
{
    MhdPrim wl, wr;
    double cL, cR;
    const bool okL = mhd_side(UL, nd, ph, wl, cL), okR = mhd_side(UR, nd, ph, wr, cR);
    double FL[8], FR[8];
    mhd_flux(UL, wl, nd, FL);
    mhd_flux(UR, wr, nd, FR);
    const double uL = (nd == 0) ? wl.u[0] : ((nd == 1) ? wl.u[1] : wl.u[2]);
    const double uR = (nd == 0) ? wr.u[0] : ((nd == 1) ? wr.u[1] : wr.u[2]);
    if constexpr (FLUX == FLUX_RUSANOV) {
        const double s = fmax1(fabs(uL) + cL, fabs(uR) + cR);
#pragma unroll
        for (int q = 0; q < 8; ++q) Fh[q] = 0.5 * ((FL[q] + FR[q]) - (s * (UR[q] - UL[q])));
        return okL && okR;
    } else {
        const double SL = fmin1(uL - cL, uR - cR);
        const double SR = fmax1(uL + cL, uR + cR);
        return hll_tame<8>(UL, UR, FL, FR, SL, SR, Fh) && okL && okR;
    }
}

// ---------------------------------------------------------------- fluxes

// Whether the flux has a short form, to be used with this reconstruction. (WENO3 states of ideal
// MHD's eight fields in front of a short flux took 194 registers, where 114 hold the general one.)
template <int EQ, int RECON, int FLUX>
constexpr bool short_flux()
{
    if (EQ == EQ_EULER)
        return FLUX == FLUX_RUSANOV || FLUX == FLUX_HLL || FLUX == FLUX_HLLC || FLUX == FLUX_ROE;
    return EQ == EQ_SWE || (EQ == EQ_MHD && RECON != REC_WENO3);
}

// Numerical flux at a face from tame cells; false where the windows do not hold.
template <int DIM, int EQ, int RECON, int FLUX>
__device__ __forceinline__ bool numflux_tame(const double* UL, const double* UR, int nd, double* Fh,
                                             const Phys& ph)
{
    if constexpr (EQ == EQ_EULER && short_flux<EQ, RECON, FLUX>()) {
        constexpr int NF = DIM + 2;
        EulerPrim<DIM> wl, wr;
        const bool ok = euler_prims<DIM>(UL, UR, ph, wl, wr);
        if constexpr (FLUX == FLUX_HLLC) {
            return hllc_tame<DIM>(UL, UR, wl, wr, nd, Fh) && ok;
        } else {
            double FL[NF], FR[NF];
            euler_flux<DIM>(UL, wl, nd, FL);
            euler_flux<DIM>(UR, wr, nd, FR);
            const double uL = pick<DIM>(wl.u, nd), uR = pick<DIM>(wr.u, nd);
            if constexpr (FLUX == FLUX_ROE) {
                return roe_tame<DIM>(UL, UR, wl, wr, FL, FR, nd, Fh, ph) && ok;
            } else if constexpr (FLUX == FLUX_RUSANOV) {
                const double s = fmax1(fabs(uL) + wl.c, fabs(uR) + wr.c);
#pragma unroll
                for (int q = 0; q < NF; ++q) Fh[q] = 0.5 * ((FL[q] + FR[q]) - (s * (UR[q] - UL[q])));
                return ok;
            } else {
                const double SL = fmin1(uL - wl.c, uR - wr.c);
                const double SR = fmax1(uL + wl.c, uR + wr.c);
                return hll_tame<NF>(UL, UR, FL, FR, SL, SR, Fh) && ok;
            }
        }
    } else if constexpr (EQ == EQ_SWE) {
        return swe_tame<DIM, FLUX>(UL, UR, nd, Fh, ph);
    } else if constexpr (EQ == EQ_MHD && short_flux<EQ, RECON, FLUX>()) {
        return mhd_tame<FLUX>(UL, UR, nd, Fh, ph);
    } else {
        numflux<DIM, EQ, FLUX>(UL, UR, nd, Fh, ph);
        return true;
    }
}

// ---------------------------------------------------------------- one face

// Whether faces of this scheme have a shorter form for tame cells.
template <int EQ, int RECON, int FLUX>
constexpr bool has_tame_face()
{
    if (RECON == REC_CELLS4) return false;
    return RECON == REC_WENO3 || RECON == REC_MUSCL || short_flux<EQ, RECON, FLUX>();
}

// Whether a cell that is not finite has to be seen when it is loaded. With Euler's windowed
// fluxes a NaN reaches the density or the squared sound speed of the face (from the conserved
// fields, or through the reciprocal that WENO3's fields share) and fails the window there.
// minmod's minimum and maximum drop a NaN, and the other fluxes have no window on every field.
template <int EQ, int RECON, int FLUX>
constexpr bool cells_need_finite()
{
    return RECON == REC_MUSCL || EQ != EQ_EULER || !short_flux<EQ, RECON, FLUX>();
}

// Cells around a face. reread() gives the same values to the general path in a form that keeps the
// compiler from holding what the short path computed from them (differences, smoothness terms)
// until then: that took 50 registers of the 3D marching kernel.
// In LDS: field q of cell i - 2 + j at s[q * QS + (j - 2) * STRIDE].
template <int QS, int STRIDE>
struct LdsCells {
    const double* su;
    int c;
    __device__ __forceinline__ double operator()(int q, int j) const { return su[q * QS + c + (j - 2) * STRIDE]; }
    __device__ __forceinline__ LdsCells reread() const
    {
        LdsCells r{su, c};
        asm volatile("" : "+v"(r.c));
        return r;
    }
};

// The same for cells in registers: each value as if new.
template <class Cells>
struct Reread {
    const Cells& at;
    __device__ __forceinline__ double operator()(int q, int j) const
    {
        double v = at(q, j);
        asm volatile("" : "+v"(v));
        return v;
    }
};

// Cells of a face in registers: cell i - 2 + j at w[j - 2 + G].
template <int NF, int G>
struct RowCells {
    const double (&w)[2 * G][NF];
    __device__ __forceinline__ double operator()(int q, int j) const { return w[j - 2 + G][q]; }
    __device__ __forceinline__ Reread<RowCells> reread() const { return Reread<RowCells>{*this}; }
};

// Flux at the face with normal axis ND between cells i - 1 and i; at(q, j): field q of cell
// i - 2 + j (j = 1, 2 only for first order). tame: uniform over the wavefront. rec: how the short
// path reconstructs (once not tame, a march stays so: its kept terms are not used again).
template <int DIM, int EQ, int RECON, int FLUX, int ND, class Cells, class Rec>
__device__ __forceinline__ void face_flux(const Cells& at, const Phys& ph, bool tame, double* F, Rec& rec)
{
    constexpr int NF = NumFields<DIM, EQ>::value;
    if constexpr (has_tame_face<EQ, RECON, FLUX>()) {
        if (tame) {
            double UL[NF], UR[NF];
            rec.template states<RECON, NF>(at, UL, UR);
            const bool ok = numflux_tame<DIM, EQ, RECON, FLUX>(UL, UR, ND, F, ph);
            if (!any_lane(!ok)) return;
        }
    }
    double UL[NF], UR[NF];
    const auto cell = at.reread();
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        if constexpr (RECON == REC_FIRST)
            reconstruct<RECON>(0.0, cell(q, 1), cell(q, 2), 0.0, UL[q], UR[q]);
        else
            reconstruct<RECON>(cell(q, 0), cell(q, 1), cell(q, 2), cell(q, 3), UL[q], UR[q]);
    }
    numflux<DIM, EQ, FLUX>(UL, UR, ND, F, ph);
}

template <int DIM, int EQ, int RECON, int FLUX, int ND, class Cells>
__device__ __forceinline__ void face_flux(const Cells& at, const Phys& ph, bool tame, double* F)
{
    Reconstruct rec;
    face_flux<DIM, EQ, RECON, FLUX, ND>(at, ph, tame, F, rec);
}

}  // namespace fvk
