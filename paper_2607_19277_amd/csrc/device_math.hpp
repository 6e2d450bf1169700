// device_math.hpp -- per-cell / per-face device arithmetic shared by the
// gfx950 kernels: the Euler update (AGILE 1.0, Sec. 2.3.1 equations;
// Table 1 solvers HLL, HLLC, LF), ideal MHD with GLM cleaning (Sec. 2.3.3)
// and special relativistic hydrodynamics (Sec. 2.3.4); minmod and van Leer
// slopes (Sec. 3.1).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace agile {

// ---------------------------------------------------------------------------
// arithmetic helpers

// reciprocal: hardware estimate (relative error below 5e-8 on gfx950)
// refined by one Newton step, which squares the error: below 3e-15, measured
// at most 20 ulp over 2^-60 .. 2^60
__device__ __forceinline__ double rcp64(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
// square root of zero or a positive normal number: hardware reciprocal
// square root refined by two Goldschmidt steps and a final residual
// correction (~1 ulp); zero maps to zero (the iteration alone would give
// 0 * inf)
__device__ __forceinline__ double sqrt64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, x);
    return x == 0.0 ? 0.0 : fma(d, h, g);
}
// FP32: the hardware's own
__device__ __forceinline__ float rcpR(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsqR(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float sqrtR(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float fminR(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float absR(float a) { return __builtin_fabsf(a); }
__device__ __forceinline__ float fmaxR(float a, float b) { return __builtin_fmaxf(a, b); }

// minmod(a, b) = median(a, b, 0): 0 unless a and b have the same sign, else
// the argument of smaller magnitude (a and b equal on ties).
__device__ __forceinline__ double minmod(double a, double b) {
    return __builtin_fmax(__builtin_fmin(a, b), __builtin_fmin(__builtin_fmax(a, b), 0.0));
}
__device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }

// The limited slope of a cell is used only as w +- slope/2.  half_slope<LIM>
// returns the slope times 1/2 / HALF<LIM>, so that the factor falls into the
// fma of that sum (minmod) or away (van Leer).
// LIM 0: minmod(a, b).  LIM 1: half of van Leer's slope, the harmonic mean
// 2ab/(a + b) when a and b have the same strict sign (ab > 0), else 0.
template <int LIM>
constexpr double HALF = LIM == 1 ? 1.0 : 0.5;
__device__ __forceinline__ double harmonic(double a, double b) {
    const double t = a * b, s = a + b;
    const double r = __builtin_amdgcn_rcp(s);
    const double q = t * r;                        // the Newton step of the
    const double h = fma(q, fma(-s, r, 1.0), q);   // reciprocal, on the product
    return t > 0.0 ? h : 0.0;
}
__device__ __forceinline__ float harmonic(float a, float b) {
    const float t = a * b;
    return t > 0.0f ? t * rcpR(a + b) : 0.0f;
}
template <int LIM, typename R>
__device__ __forceinline__ R half_slope(R a, R b) {
    if constexpr (LIM == 1) return harmonic(a, b);
    else return minmod(a, b);
}
// the slopes of the two cells that share the difference b: of (a, b) and of
// (b, c).  FP64 minmod(x, b) = x clamped to between 0 and b: the bounds are
// formed once for both, 6 operations instead of 8.
template <int LIM, typename R>
__device__ __forceinline__ void half_slopes(R a, R b, R c, R &s0, R &s1) {
    if constexpr (LIM == 0 && sizeof(R) == 8) {
        const R lo = __builtin_fmin(b, 0.0), hi = __builtin_fmax(b, 0.0);
        s0 = __builtin_fmax(__builtin_fmin(a, hi), lo);
        s1 = __builtin_fmax(__builtin_fmin(c, hi), lo);
    } else {
        s0 = half_slope<LIM>(a, b);
        s1 = half_slope<LIM>(b, c);
    }
}

// reciprocal square root of a positive normal number: hardware estimate
// refined by one Newton step (measured at most 36 ulp over 2^-60 .. 2^60)
__device__ __forceinline__ double rsq64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        unsigned long long w = __shfl_xor(v, o, 64);
        v = w > v ? w : v;
    }
    return v;
}

// ---------------------------------------------------------------------------
// Euler physics

// conserved -> primitives (rho, vx, vy, vz, p) with v = m (1/rho),
// p = (gamma-1)(e - rho v^2/2); returns whether rho > 0 and p > 0
__device__ __forceinline__ bool cons2prim(const double U[5], double gm1, double w[5]) {
    const double rho = U[0];
    const double r = rcp64(rho);
    const double vx = U[1] * r, vy = U[2] * r, vz = U[3] * r;
    const double vv = (vx * vx + vy * vy) + vz * vz;
    const double p = gm1 * (U[4] - 0.5 * rho * vv);
    w[0] = rho; w[1] = vx; w[2] = vy; w[3] = vz; w[4] = p;
    return rho > 0.0 && p > 0.0;
}

// IEEE quotients and roots of ordinary numbers.  The compiler's division and
// square root spend most of their operations on scaling, so that the whole
// exponent range works; for numbers between 2^-250 and 2^250 the Newton and
// Goldschmidt steps in their middle give the same, correctly rounded result
// by themselves, and quotients by one denominator can share its reciprocal:
//   r = newton_rcp(d);  n / d = quotient(n, d, r);  1 / d = quotient(1, d, r).
__device__ __forceinline__ bool ordinary(double x) {   // 2^-250 <= x < 2^250
    return unsigned(__double2hiint(x)) - 0x30500000u < 0x1f400000u;
}
__device__ __forceinline__ double newton_rcp(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}
__device__ __forceinline__ double quotient(double n, double d, double r) {
    const double q = n * r;
    return fma(fma(-d, q, n), r, q);
}
__device__ __forceinline__ double root(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}

// Cell signal rate s = ((|vx|+c)/dx + (|vy|+c)/dx) + (|vz|+c)/dx with
// c = sqrt(gamma p / rho), evaluated operation by operation with IEEE
// division and square root and no contraction, so that the CFL maximum is
// the same number as on the CPU.  Ordinary states take the short forms above
// (the same bits, 91 instructions instead of 170 in the last stage: SSP-RK2
// HLLC steps on 256^3 2% faster); a wave with any other state takes the
// general ones.
__device__ __forceinline__ double signal_rate(const double U[5], double gamma, double inv_dx, bool &ok) {
#pragma clang fp contract(off)
    const double rho = U[0];
    const double rr = newton_rcp(rho);
    double r = quotient(1.0, rho, rr);
    double vx = U[1] * r, vy = U[2] * r, vz = U[3] * r;
    double vv = (vx * vx + vy * vy) + vz * vz;
    double p = (gamma - 1.0) * (U[4] - 0.5 * rho * vv);
    const double gp = gamma * p;
    double c = root(quotient(gp, rho, rr));
    ok = ordinary(rho) & ordinary(gp);
    if (!ok) {
        r = 1.0 / rho;
        vx = U[1] * r; vy = U[2] * r; vz = U[3] * r;
        vv = (vx * vx + vy * vy) + vz * vz;
        p = (gamma - 1.0) * (U[4] - 0.5 * rho * vv);
        ok = rho > 0.0 && p > 0.0;
        c = __builtin_sqrt(gamma * p / rho);
    }
    double s = (__builtin_fabs(vx) + c) * inv_dx;
    s = s + (__builtin_fabs(vy) + c) * inv_dx;
    s = s + (__builtin_fabs(vz) + c) * inv_dx;
    return s;
}

// Conserved state and physical flux of a primitive state rotated to the face
// normal, (rho, u_n, u_t1, u_t2, p): mass rho u_n, momentum rho u u_n + p e_n,
// energy u_n (e + p) -- the Euler equations of Sec. 2.3.1.  (FP32; the FP64
// fluxes form neither.)
__device__ __forceinline__ void euler_UF(const float w[5], float igm1, float U[5], float F[5]) {
    using R = float;
    const R rho = w[0], un = w[1], v1 = w[2], v2 = w[3], p = w[4];
    const R vv = (un * un + v1 * v1) + v2 * v2;
    const R e = p * igm1 + R(0.5) * rho * vv;
    const R mn = rho * un;
    U[0] = rho; U[1] = mn; U[2] = rho * v1; U[3] = rho * v2; U[4] = e;
    F[0] = mn; F[1] = mn * un + p; F[2] = U[2] * un; F[3] = U[3] * un; F[4] = un * (e + p);
}

// sound speed c = sqrt(gamma p / rho), written as gamma p / sqrt(gamma p rho)
__device__ __forceinline__ float sound_speed(float rho, float p, float gamma) {
    const float gp = gamma * p;
    return gp * rsqR(gp * rho);
}

// HLL (RS = 0), HLLC (RS = 1) or local Lax-Friedrichs (RS = 2) flux across a
// face from rotated left / right primitive states, evaluated without branches.  Wave speeds of Davis:
// S_L = min(u_L - c_L, u_R - c_R), S_R = max(u_L + c_L, u_R + c_R).
// HLL: with a = max(S_R, 0), b = min(S_L, 0),
//   F = (a F_L - b F_R + a b (U_R - U_L)) / (a - b),
// which equals F_L for S_L >= 0, F_R for S_R <= 0 and the two-wave HLL flux
// otherwise.
// HLLC (Toro, Sec. 10.4): contact speed
//   S* = (p_R - p_L + rho_L u_L (S_L - u_L) - rho_R u_R (S_R - u_R)) / (rho_L (S_L - u_L) - rho_R (S_R - u_R)),
// upwind side K = L if S_L >= 0, R if S_R <= 0, else L iff S* >= 0; then
//   F = F_K in the supersonic cases, else
//   F*_K = (S*(S_K U_K - F_K) + S_K P_K D*)/(S_K - S*), D* = (0, 1, 0, 0, S*),
//   P_K = p_K + rho_K (S_K - u_K)(S* - u_K).
// Only side K's conserved state and flux are formed.
__device__ __forceinline__ void riemann_srhd(const float wL[5], const float wR[5], float g, float igm1, float F[5]);
__device__ __forceinline__ void riemann_srhd(const double wL[5], const double wR[5], double g, double igm1,
                                             double F[5]);

// FP32: the operations in the order of the formulas above.  The FP64 forms
// below need fewer operations but round differently, which in FP32 would move
// a state by about 1e-8 of itself per step.
template <int RS>
__device__ __forceinline__ void riemann_euler(const float wL[5], const float wR[5], float gamma, float igm1,
                                              float F[5]) {
    using R = float;
    const R cL = sound_speed(wL[0], wL[4], gamma);
    const R cR = sound_speed(wR[0], wR[4], gamma);
    const R uL = wL[1], uR = wR[1];
    const R SL = fminR(uL - cL, uR - cR);
    const R SR = fmaxR(uL + cL, uR + cR);
    if (RS == 2) {
        // local Lax-Friedrichs: F = ((F_L + F_R) - s (U_R - U_L))/2 with the
        // larger |u| + c of the two states
        R UL[5], FL[5], UR[5], FRt[5];
        euler_UF(wL, igm1, UL, FL);
        euler_UF(wR, igm1, UR, FRt);
        const R sp = fmaxR(absR(uL) + cL, absR(uR) + cR);
#pragma unroll
        for (int v = 0; v < 5; ++v) F[v] = R(0.5) * ((FL[v] + FRt[v]) - sp * (UR[v] - UL[v]));
    } else if (RS == 0) {
        R UL[5], FL[5], UR[5], FRt[5];
        euler_UF(wL, igm1, UL, FL);
        euler_UF(wR, igm1, UR, FRt);
        const R ap = fmaxR(SR, R(0)), bm = fminR(SL, R(0));
        const R inv = rcpR(ap - bm);
        const R ab = ap * bm;
#pragma unroll
        for (int v = 0; v < 5; ++v) F[v] = ((ap * FL[v] - bm * FRt[v]) + ab * (UR[v] - UL[v])) * inv;
    } else {
        const R dL = wL[0] * (SL - uL), dR = wR[0] * (SR - uR);
        const R Ss = ((wR[4] - wL[4]) + (uL * dL - uR * dR)) * rcpR(dL - dR);
        // bitwise logic: a short-circuit would become a branch
        const bool supL = SL >= R(0), supR = SR <= R(0);
        const bool left = supL | (!supR & (Ss >= R(0)));
        R w[5], U[5], Fk[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) w[v] = left ? wL[v] : wR[v];
        const R SK = left ? SL : SR;
        const R dK = left ? dL : dR;
        euler_UF(w, igm1, U, Fk);
        const R PK = w[4] + dK * (Ss - w[1]);
        const R inv = rcpR(SK - Ss);
        const R SP = SK * PK;
        const bool sup = supL | supR;
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            R t = Ss * (SK * U[v] - Fk[v]);
            if (v == 1) t = t + SP;
            if (v == 4) t = t + SP * Ss;
            F[v] = sup ? Fk[v] : t * inv;
        }
    }
}

// FP64 sound speed: c = gp / sqrt(gp rho) as in sound_speed, the Newton step
// of the reciprocal root applied to the product
__device__ __forceinline__ double sound_speed64(double rho, double p, double gamma) {
    const double gp = gamma * p;
    const double x = gp * rho;
    const double y = __builtin_amdgcn_rsq(x);
    const double c = gp * y;
    return fma(0.5 * c, fma(-x * y, y, 1.0), c);
}

// FP64: the same fluxes with the physical flux written as F = u U + p (0, 1, 0,
// 0, u), so that neither U nor F of a side is formed.
// HLL and Lax-Friedrichs are both al F_L + be F_R + k (U_L - U_R) with, for HLL,
// al = S_R+/(S_R+ - S_L-), be = -S_L-/(S_R+ - S_L-), k = S_R+ be, S+ = max(S, 0),
// S- = min(S, 0), and for Lax-Friedrichs al = be = 1/2, k = s/2.  With the mass
// flux M = al rho_L u_L + be rho_R u_R + k (rho_L - rho_R) and the right
// side's part B = (be u_R - k) rho_R of it, what the flow carries is M q_L + B
// (q_R - q_L) for q = u, v_t, v^2/2: differences of the sides before products.
// (Sums a U_L + b U_R with a = al u_L + k, b = be u_R - k take six
// operations fewer, LF / van Leer / SSP-RK3 steps on 256^3 4890 instead of 4980
// us, but in slow flow a rho_L and b rho_R cancel: densities were off by up to
// 1.5 times as much.)
// HLLC: across S_K the star state satisfies the jump conditions, so its flux
// is the physical flux of the state (rho*, S*, v_t, P_K, e*),
//   rho* = rho_K (S_K - u_K)/(S_K - S*),
//   e* = (e_K (S_K - u_K) - p_K u_K + P_K S*)/(S_K - S*).
// With S_K limited to S_L <= 0 or S_R >= 0 that flux is F_K itself when the
// flow is supersonic (S_K = 0 leaves rho* S* = rho_K u_K, and so on), so no
// case is selected after the side but S*/(S_K - S*) = -1 at S_K = 0: through the
// reciprocal of rcp64 the supersonic flux would be off by up to 20 ulp (1856-block
// blast 5180 -> 5205 us).  Davis' speeds give S_L < S* < S_R (the numerator of S* - S_L
// is at least gamma (p_L + p_R) - (p_R - p_L) > 0, and likewise on the right), so
// the sign of S* alone picks the side.
// The stage kernel is bound by its VALU work and latency, not by HBM, so the
// operation count is what matters: HLLC 71 instructions a face instead of
// 113.  With the shared minmod bounds above, a pass of ten steps of the
// 1856-block HLLC blast 6533 -> 6189 us, and of three LF / van Leer / SSP-RK3
// steps on 256^3 6804 -> 5667 us (when these fluxes came in).
template <int RS>
__device__ __forceinline__ void riemann_euler(const double wL[5], const double wR[5], double gamma, double igm1,
                                              double F[5]) {
    const double cL = sound_speed64(wL[0], wL[4], gamma);
    const double cR = sound_speed64(wR[0], wR[4], gamma);
    const double uL = wL[1], uR = wR[1];
    if (RS == 1) {
        const double SL = __builtin_fmin(uL - cL, uR - cR);
        const double SR = __builtin_fmax(uL + cL, uR + cR);
        const double dL = wL[0] * (SL - uL), dR = wR[0] * (SR - uR);
        const double num = fma(-uR, dR, fma(uL, dL, wR[4] - wL[4]));
        const double Ss = num * rcp64(dL - dR);
        const bool left = Ss >= 0.0;
        double w[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) w[v] = left ? wL[v] : wR[v];
        const double SK = left ? __builtin_fmin(SL, 0.0) : __builtin_fmax(SR, 0.0);
        const double u = w[1], p = w[4];
        const double du = SK - u;
        const double dK = w[0] * du;
        const double q = SK == 0.0 ? -1.0 : Ss * rcp64(SK - Ss);
        const double PK = fma(dK, Ss - u, p);
        const double vv = fma(w[3], w[3], fma(w[2], w[2], u * u));
        const double e = fma(0.5 * w[0], vv, p * igm1);
        const double t = PK * Ss;
        F[0] = dK * q;
        F[1] = fma(F[0], Ss, PK);
        F[2] = F[0] * w[2];
        F[3] = F[0] * w[3];
        F[4] = fma(fma(e, du, fma(-p, u, t)), q, t);
        return;
    }
    double al, be, k;
    if (RS == 2) {
        al = be = 0.5;
        k = 0.5 * __builtin_fmax(__builtin_fabs(uL) + cL, __builtin_fabs(uR) + cR);
    } else {
        const double sr = __builtin_fmax(__builtin_fmax(uL + cL, uR + cR), 0.0);
        const double sl = __builtin_fmin(__builtin_fmin(uL - cL, uR - cR), 0.0);
        const double inv = rcp64(sr - sl);
        al = sr * inv;
        be = -sl * inv;
        k = sr * be;
    }
    const double a = al * uL, b = be * uR;
    const double mR = b * wR[0];
    const double M = fma(k, wL[0] - wR[0], fma(a, wL[0], mR));
    const double B = fma(-k, wR[0], mR);
    const double vL = fma(wL[3], wL[3], fma(wL[2], wL[2], uL * uL));
    const double vR = fma(wR[3], wR[3], fma(wR[2], wR[2], uR * uR));
    F[0] = M;
    F[1] = fma(M, uL, fma(B, uR - uL, RS == 2 ? 0.5 * (wL[4] + wR[4]) : fma(al, wL[4], be * wR[4])));
    F[2] = fma(M, wL[2], B * (wR[2] - wL[2]));
    F[3] = fma(M, wL[3], B * (wR[3] - wL[3]));
    const double pu = fma(a, wL[4], b * wR[4]);   // e + p = gamma/(gamma - 1) p + rho v^2/2 on either side
    F[4] = fma(0.5, fma(M, vL, B * (vR - vL)), fma(igm1 * k, wL[4] - wR[4], fma(igm1, pu, pu)));
}

template <int RS, typename R>
__device__ __forceinline__ void riemann(const R wL[5], const R wR[5], R gamma, R igm1, R F[5]) {
    if constexpr (RS == 3) riemann_srhd(wL, wR, gamma, igm1, F);   // SRHD states (rho, u, p): local Lax-Friedrichs
    else riemann_euler<RS>(wL, wR, gamma, igm1, F);
}


// ---------------------------------------------------------------------------
// special relativistic hydrodynamics (c = 1), nvar 5: (D, m, tau)
// primitives (rho, u, p) with u = Gamma v the spatial four-velocity, ideal
// gas h = 1 + g/(g-1) p/rho (Sec. 2.3.4)

// con2prim by a 1-D root in xi = Gamma^2 rho h: with e = tau + D,
//   1/Gamma^2 = 1 - m^2/xi^2, rho = D/Gamma, p(xi) = (g-1)/g (xi/Gamma^2 - D/Gamma),
//   f(xi) = xi - p(xi) - e increases on (|m|, g e], f(|m|) <= 0 < f(g e);
// Newton steps from xi = e kept inside the bracket (bisection otherwise)
// until a step moves xi by at most 1e-15 xi (at most 100).  IEEE division and
// square root without contraction: the same iterates as on any machine.  The
// ghost prolongation and the regrid transfer use this form, so that their states
// are the same bits everywhere.
__device__ __forceinline__ bool srhd_con2prim(const double U[5], double g, double w[5]) {
#pragma clang fp contract(off)
    const double D = U[0], e = U[4] + U[0];
    const double m2 = (U[1] * U[1] + U[2] * U[2]) + U[3] * U[3];
    const double mm = __builtin_sqrt(m2);
    const double gg = (g - 1.0) / g;
    double lo = mm, hi = g * e;
    if (!(D > 0.0) || !(hi > lo)) {
        for (int v = 0; v < 5; ++v) w[v] = 1.0;
        return false;
    }
    double x = e;
    if (!(x > lo)) x = 0.5 * (lo + hi);
    bool conv = false;
    for (int it = 0; it < 100 && !conv; ++it) {
        const double q = m2 / (x * x);
        const double g2 = 1.0 - q;
        const double ig = __builtin_sqrt(g2);
        const double G = 1.0 / ig;
        const double p = gg * (x * g2 - D * ig);
        const double f = (x - p) - e;
        const double fp = 1.0 - gg * ((1.0 + q) - D * G * q / x);
        if (f > 0.0) hi = x;
        else if (f < 0.0) lo = x;
        double xn = x - f / fp;
        // a step within the tolerance converges, also on a bracket end
        conv = __builtin_fabs(xn - x) <= 1e-15 * xn;
        if (!conv && !(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
        x = xn;
    }
    const double g2 = 1.0 - m2 / (x * x);
    const double ig = __builtin_sqrt(g2);
    const double G = 1.0 / ig;
    const double rho = D * ig;
    const double p = gg * (x * g2 - D * ig);
    w[0] = rho;
    w[1] = (U[1] / x) * G;
    w[2] = (U[2] / x) * G;
    w[3] = (U[3] / x) * G;
    w[4] = p;
    return conv && rho > 0.0 && p > 0.0;
}

// reciprocal and reciprocal square root refined by two Newton steps
// (within about an ulp): the con2prim iteration below stops on its step
// size, which must stay above their rounding noise
__device__ __forceinline__ double rcp64x2(double x) {
    const double r = rcp64(x);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double rsq64x2(double x) {
    const double y = rsq64(x);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// The same root for the flux path, where the primitives need not be the same
// bits as elsewhere: reciprocals instead of IEEE division and square root, a
// start nearer the root, and Newton stops after a step of at most 1e-9 xi.  Newton converges
// quadratically there, so that step leaves an error far below rounding (the
// result agrees with the 1e-15 iteration to a few ulp), and the stopping
// test stays clear of the arithmetic's noise.
__device__ __forceinline__ bool srhd_con2prim_bracketed(const double U[5], double g, double w[5]) {
    const double D = U[0], e = U[4] + U[0];
    const double m2 = (U[1] * U[1] + U[2] * U[2]) + U[3] * U[3];
    const double gg = (g - 1.0) / g;
    double lo = __builtin_sqrt(m2), hi = g * e;
    if (!(D > 0.0) || !(hi > lo)) {
        for (int v = 0; v < 5; ++v) w[v] = 1.0;
        return false;
    }
    // start: the root at rest, xi = e + (g-1)(e - D), with the pressure part
    // scaled by 1 - m^2/e^2 (one Newton step fewer than xi = e on moving gas)
    double x = e + ((g - 1.0) * (e - D)) * (1.0 - m2 * rcp64x2(e * e));
    if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
    bool conv = false;
    for (int it = 0; it < 100 && !conv; ++it) {
        const double r = rcp64x2(x);
        const double q = (m2 * r) * r;
        const double g2 = 1.0 - q;
        const double G = rsq64x2(g2);
        const double ig = g2 * G;
        const double p = gg * (x * g2 - D * ig);
        const double f = (x - p) - e;
        const double fp = 1.0 - gg * ((1.0 + q) - ((D * G) * q) * r);
        if (f > 0.0) hi = x;
        else if (f < 0.0) lo = x;
        const double dx = f * rcp64x2(fp);
        double xn = x - dx;
        conv = __builtin_fabs(dx) <= 1e-9 * x;
        if (!conv && !(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
        x = xn;
    }
    const double r = rcp64x2(x);
    const double g2 = 1.0 - (m2 * r) * r;
    const double G = rsq64x2(g2);
    const double ig = g2 * G;
    const double rho = D * ig;
    const double p = gg * (x * g2 - D * ig);
    const double rG = r * G;
    w[0] = rho;
    w[1] = U[1] * rG;
    w[2] = U[2] * rG;
    w[3] = U[3] * rG;
    w[4] = p;
    return conv && rho > 0.0 && p > 0.0;
}

// The form every cell takes first: Newton alone, without the bracket's
// selects, in two parts.  Until a step is below 3e-5 xi reciprocals with one
// refinement do.  The steps that follow are accurate (their slope needs no
// refinement: its error of 5e-8 counts against the step alone), with the
// residual as (xi - e) - p, where the first difference is exact.  Newton's
// constant grows with Gamma^2 (about Gamma^2/6 for cold gas) and an error of xi
// with 2 Gamma^2 in 1/Gamma^2, so the last step must be below 1e-9 xi / Gamma^2:
// gas below Gamma of about 2 is done after one accurate step, faster gas takes
// a second one.  Against the root in extended precision the primitives are
// 0.85 times as far off as the bracketed form's (median over Gamma 1 to 128,
// p/rho 1e-4 to 100; nowhere further beyond the noise of rounding).  A lane that leaves (|m|, g e), does not
// converge (12 and 4 steps; at Gamma above 1000 the arithmetic's noise exceeds the bound)
// or has no state is left to the bracketed form.  The stage kernels of SRHD are
// bound by this iteration; per cell about 180 issue slots instead of 260 (with
// the flux below, three SSP-RK3 steps of the 256^3 shear layer 8520 -> 6965 us,
// with FP32 fluxes 6360 -> 5620 us; the bound that follows Gamma costs this
// mild gas nothing, 7021 -> 7006).
__device__ __forceinline__ bool srhd_con2prim_fast(const double U[5], double g, double w[5]) {
    const double D = U[0], e = U[4] + U[0];
    const double m2 = fma(U[3], U[3], fma(U[2], U[2], U[1] * U[1]));
    const double gg = (g - 1.0) / g;
    const double hi = g * e;
    double x = fma((g - 1.0) * (e - D), fma(-m2, __builtin_amdgcn_rcp(e * e), 1.0), e);
    bool fine = (D > 0.0) & (x * x > m2) & (x < hi), near = false;
    for (int it = 0; it < 12 && fine && !near; ++it) {
        const double r = rcp64(x);
        const double q = (m2 * r) * r;
        const double g2 = 1.0 - q;
        const double DG = D * rsq64(g2);
        const double f = fma(-(gg * g2), x - DG, x - e);
        const double fp = fma(-gg, fma(-(DG * q), r, 1.0 + q), 1.0);
        const double dx = f * __builtin_amdgcn_rcp(fp);
        x = x - dx;
        near = __builtin_fabs(dx) <= 3e-5 * x;
        fine = (x * x > m2) & (x < hi);
    }
    double r = 0.0;
    bool conv = false;
    for (int it = 0; it < 4 && near && !conv; ++it) {
        r = rcp64x2(x);
        const double q = (m2 * r) * r;
        const double g2 = 1.0 - q;
        const double DG = D * rsq64x2(g2);
        const double f = fma(-(gg * g2), x - DG, x - e);
        const double fp = fma(-gg, fma(-(DG * q), r, 1.0 + q), 1.0);
        const double dx = f * __builtin_amdgcn_rcp(fp);
        x = x - dx;
        conv = __builtin_fabs(dx) <= 1e-9 * (x * g2);
    }
    r = fma(r, fma(-x, r, 1.0), r);   // x moved by at most 1e-9 of itself
    const double g2 = 1.0 - (m2 * r) * r;
    const double G = rsq64x2(g2);
    const double ig = g2 * G;
    const double rho = D * ig;
    const double p = gg * (x * g2 - D * ig);
    const double rG = r * G;
    w[0] = rho;
    w[1] = U[1] * rG;
    w[2] = U[2] * rG;
    w[3] = U[3] * rG;
    w[4] = p;
    bool ok = rho > 0.0 && p > 0.0;
    if (!conv) ok = srhd_con2prim_bracketed(U, g, w);
    return ok;
}

// One reconstructed state (rho, u_n, u_t1, u_t2, p) at a face along the first
// velocity slot: its conserved values
//   D = Gamma rho, m = Gamma rho h u, tau = Gamma^2 rho h - p - D,
// its flux F = (D v_n, m v_n + p e_n, m_n - D v_n), and its largest
// |characteristic speed|
//   (|v_n| (1 - c_s^2) + sqrt(c_s^2 (1 - v^2)(1 - v^2 c_s^2 - v_n^2 (1 - c_s^2)))) / (1 - v^2 c_s^2),
// c_s^2 = g p / (rho h).  With s = 1/sqrt(1 + u^2): Gamma = (1 + u^2) s,
// v_n = u_n s, v^2 = u^2 s^2, so a state takes one reciprocal square root,
// two reciprocals and one square root.
__device__ __forceinline__ float srhd_face_state(const float w[5], float ghat, float g, float U[5], float F[5]) {
    using R = float;
    const R uu = (w[1] * w[1] + w[2] * w[2]) + w[3] * w[3];
    const R G2 = R(1) + uu;
    const R s = rsqR(G2);
    const R G = G2 * s;
    const R vn = w[1] * s;
    const R v2 = uu * (s * s);
    const R rhoh = w[0] + ghat * w[4];
    const R cs2 = (g * w[4]) * rcpR(rhoh);
    U[0] = G * w[0];
    const R Grh = G * rhoh;
    U[1] = Grh * w[1];
    U[2] = Grh * w[2];
    U[3] = Grh * w[3];
    U[4] = (G * Grh - w[4]) - U[0];
    F[0] = U[0] * vn;
    F[1] = U[1] * vn + w[4];
    F[2] = U[2] * vn;
    F[3] = U[3] * vn;
    F[4] = U[1] - F[0];
    R disc = (R(1) - v2) * ((R(1) - v2 * cs2) - (vn * vn) * (R(1) - cs2));
    disc = disc < R(0) ? R(0) : disc;
    return (absR(vn) * (R(1) - cs2) + sqrtR(cs2 * disc)) * rcpR(R(1) - v2 * cs2);
}

// local Lax-Friedrichs flux with the larger |characteristic speed| of the
// two reconstructed states (Table 1: the SRHD module offers LF)
// FP32: the operations in the order of the formulas above (see riemann_euler).
__device__ __forceinline__ void riemann_srhd(const float wL[5], const float wR[5], float g, float igm1, float F[5]) {
    using R = float;
    R UL[5], FL[5], UR[5], FR[5];
    const R ghat = g * igm1;
    const R sL = srhd_face_state(wL, ghat, g, UL, FL);
    const R sR = srhd_face_state(wR, ghat, g, UR, FR);
    const R sp = fmaxR(sL, sR);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = R(0.5) * ((FL[v] + FR[v]) - sp * (UR[v] - UL[v]));
}

// FP64: F = v_n U + p (0, 1, 0, 0, v_n), so that with a = (v_nL + s)/2, b =
// (v_nR - s)/2 (s the speed) F = a U_L + b U_R + the pressure terms, and
// neither U nor F of a side is formed -- but for mass and energy.  The energy
// flux m_n - D v_n keeps m_n = Gamma rho h u_n (through v_n it would take the
// error of the estimated Gamma three times), and the dissipation of both is
// formed from differences, so that it vanishes where the sides agree.  (As a U_L
// + b U_R throughout, energies after six steps were 1.92e-16 off against 64 bits
// instead of 1.79e-16; that saves six operations, 6914 instead of 7008 us for the
// three steps above.)  The speed is multiplied through by
// h = rho h, with c = g p: (|v_n| (h - c) + sqrt(c X)/Gamma)/(h - v^2 c),
// X = (h - v^2 c) - v_n^2 (h - c): one reciprocal and two reciprocal square
// roots a side.
__device__ __forceinline__ double srhd_face_speed(const double w[5], double ghat, double g, double &G, double &vn,
                                                  double &Gh) {
    const double uu = fma(w[3], w[3], fma(w[2], w[2], w[1] * w[1]));
    const double G2 = 1.0 + uu;
    const double s = rsq64(G2);
    G = G2 * s;
    vn = w[1] * s;
    const double h = fma(ghat, w[4], w[0]), c = g * w[4];
    Gh = G * h;
    const double den = fma(-(uu * (s * s)), c, h), hc = h - c;
    const double Y = __builtin_fmax(c * fma(-(vn * vn), hc, den), 1e-300);
    const double y = __builtin_amdgcn_rsq(Y), d = Y * y;
    const double root = fma(0.5 * d, fma(-d, y, 1.0), d);
    return fma(__builtin_fabs(vn), hc, s * root) * rcp64(den);
}
__device__ __forceinline__ void riemann_srhd(const double wL[5], const double wR[5], double g, double igm1,
                                             double F[5]) {
    double GL, GR, vL, vR, hL, hR;
    const double ghat = g * igm1;
    const double sL = srhd_face_speed(wL, ghat, g, GL, vL, hL);
    const double sR = srhd_face_speed(wR, ghat, g, GR, vR, hR);
    const double hs = 0.5 * __builtin_fmax(sL, sR);
    const double a = fma(0.5, vL, hs), b = fma(0.5, vR, -hs);
    const double DL = GL * wL[0], DR = GR * wR[0];
    const double kL = a * hL, kR = b * hR;
    const double eL = hL * GL, eR = hR * GR;   // tau + D + p
    const double tau = (eL - eR) + (wR[4] - wL[4]);   // tau_L - tau_R + D_L - D_R
    F[0] = fma(hs, DL - DR, 0.5 * fma(vL, DL, vR * DR));
    F[1] = fma(kL, wL[1], kR * wR[1]) + 0.5 * (wL[4] + wR[4]);
    F[2] = fma(kL, wL[2], kR * wR[2]);
    F[3] = fma(kL, wL[3], kR * wR[3]);
    F[4] = fma(hs, tau, fma(0.5, fma(hL, wL[1], hR * wR[1]), -F[0]));
}

// cell signal rate sum_d a_d / dx of a conserved SRHD state: the flux path's
// con2prim, then the largest |speed| along each axis as in srhd_face_state.
// Every kernel that forms the CFL signal of an SRHD state (the dt reduction,
// the last RK stage, the flux correction) calls this one function with the
// library's per-expression contraction, so they agree bitwise; against IEEE
// evaluation the rate differs by a few ulp.
__device__ __forceinline__ double srhd_signal(const double U[5], double g, double inv_dx, bool &ok) {
    double w[5];
    ok = srhd_con2prim_fast(U, g, w);
    const double uu = (w[1] * w[1] + w[2] * w[2]) + w[3] * w[3];
    const double is = rsq64(1.0 + uu);
    const double v2 = uu * (is * is);
    const double rhoh = w[0] + (g / (g - 1.0)) * w[4];
    const double cs2 = (g * w[4]) * rcp64(rhoh);
    const double ic = rcp64(1.0 - v2 * cs2);
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double vn = __builtin_fabs(w[1 + d]) * is;
        double disc = (1.0 - v2) * ((1.0 - v2 * cs2) - (vn * vn) * (1.0 - cs2));
        disc = disc < 0.0 ? 0.0 : disc;
        const double a = (vn * (1.0 - cs2) + sqrt64(cs2 * disc)) * ic;
        s = d == 0 ? a * inv_dx : s + a * inv_dx;
    }
    return s;
}

// ---------------------------------------------------------------------------
// ideal MHD with GLM cleaning (Sec. 2.3.3), nvar 9: (rho, m, e, B, psi)

// conserved -> primitives (rho, v, p, B, psi) with
// p = (gamma-1)((e - rho v^2/2) - B^2/2); returns whether rho > 0 and p > 0
__device__ __forceinline__ bool mhd_cons2prim(const double U[9], double gm1, double w[9]) {
    const double rho = U[0];
    const double r = rcp64(rho);
    const double vx = U[1] * r, vy = U[2] * r, vz = U[3] * r;
    const double vv = (vx * vx + vy * vy) + vz * vz;
    const double bb = (U[5] * U[5] + U[6] * U[6]) + U[7] * U[7];
    const double p = gm1 * ((U[4] - 0.5 * rho * vv) - 0.5 * bb);
    w[0] = rho; w[1] = vx; w[2] = vy; w[3] = vz; w[4] = p;
    w[5] = U[5]; w[6] = U[6]; w[7] = U[7]; w[8] = U[8];
    return rho > 0.0 && p > 0.0;
}

// Cell signal rate s = sum_d (|v_d| + c_f,d)/dx (summed x, y, z) and the GLM
// speed candidate cm = max_d (|v_d| + c_f,d), with the fast speed
// c_f^2 = ((a^2 + b^2) + sqrt((a^2 + b^2)^2 - 4 a^2 b_d^2))/2, a^2 = gamma p/rho,
// b^2 = |B|^2/rho, b_d^2 = B_d^2/rho; IEEE operations without contraction, so
// that dt and c_h are the same numbers as on the CPU.
__device__ __forceinline__ double mhd_signal(const double U[9], double gamma, double inv_dx, double &cm, bool &ok) {
#pragma clang fp contract(off)
    const double rho = U[0];
    const double rr = newton_rcp(rho);
    double r = quotient(1.0, rho, rr);
    double v[3] = {U[1] * r, U[2] * r, U[3] * r};
    double vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    const double bb = (U[5] * U[5] + U[6] * U[6]) + U[7] * U[7];
    double p = (gamma - 1.0) * ((U[4] - 0.5 * rho * vv) - 0.5 * bb);
    const double gp = gamma * p;
    double a2 = quotient(gp, rho, rr);
    double ss = a2 + quotient(bb, rho, rr);
    double c[3];
    ok = ordinary(rho) & ordinary(gp) & (bb == 0.0 || ordinary(bb));
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double bq = U[5 + d] * U[5 + d];
        const double disc = ss * ss - 4.0 * a2 * quotient(bq, rho, rr);
        ok &= ordinary(disc) & (bq == 0.0 || ordinary(bq));
        c[d] = root(0.5 * (ss + root(disc)));
    }
    if (!ok) {
        r = 1.0 / rho;
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] = U[1 + d] * r;
        vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
        p = (gamma - 1.0) * ((U[4] - 0.5 * rho * vv) - 0.5 * bb);
        ok = rho > 0.0 && p > 0.0;
        a2 = gamma * p / rho;
        ss = a2 + bb / rho;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double bd2 = U[5 + d] * U[5 + d] / rho;
            double disc = ss * ss - 4.0 * a2 * bd2;
            if (disc < 0.0) disc = 0.0;
            c[d] = __builtin_sqrt(0.5 * (ss + __builtin_sqrt(disc)));
        }
    }
    double s = 0.0;
    cm = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double a = __builtin_fabs(v[d]) + c[d];
        s = d == 0 ? a * inv_dx : s + a * inv_dx;
        cm = a > cm ? a : cm;
    }
    return s;
}

// MHD flux across a face from rotated primitive states (rho, u_n, u_t1, u_t2,
// p, B_n, B_t1, B_t2, psi).  GLM interface step of Dedner et al. (2002):
//   B_n* = (B_nL + B_nR)/2 - (psi_R - psi_L)/(2 c_h),
//   psi* = (psi_L + psi_R)/2 - c_h (B_nR - B_nL)/2,
// both sides take B_n*, the (B_n, psi) fluxes are (psi*, c_h^2 B_n*); HLL with
// Davis fast-speed bounds on the other seven components, in the clamped
// branch-free form F = ((a F_L - b F_R) + a b (U_R - U_L))/(a - b),
// a = max(S_R, 0), b = min(S_L, 0).  Physical flux along n: mass rho u_n,
// momentum rho u u_n + (p + B^2/2) e_n - B B_n, energy
// u_n (e + p + B^2/2) - B_n (u.B), induction u_n B - B_n u.
// FP32: the operations in the order of these formulas (see riemann_euler).
__device__ __forceinline__ void mhd_hll(const float wL[9], const float wR[9], float gamma, float igm1, float ch,
                                        float inv2ch, float F[9]) {
    using R = float;
    const R bn = R(0.5) * (wL[5] + wR[5]) - (wR[8] - wL[8]) * inv2ch;
    const R ps = R(0.5) * (wL[8] + wR[8]) - R(0.5) * ch * (wR[5] - wL[5]);
    R U[2][9], Fs[2][9], c[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const R *w = s ? wR : wL;
        const R rho = w[0], un = w[1], u1 = w[2], u2 = w[3], p = w[4], b1 = w[6], b2 = w[7];
        const R vv = (un * un + u1 * u1) + u2 * u2;
        const R bb = (bn * bn + b1 * b1) + b2 * b2;
        const R vb = (un * bn + u1 * b1) + u2 * b2;
        const R pt = p + R(0.5) * bb;
        const R e = (p * igm1 + R(0.5) * rho * vv) + R(0.5) * bb;
        const R mn = rho * un;
        U[s][0] = rho; U[s][1] = mn; U[s][2] = rho * u1; U[s][3] = rho * u2; U[s][4] = e;
        U[s][6] = b1; U[s][7] = b2;
        Fs[s][0] = mn;
        Fs[s][1] = mn * un + pt - bn * bn;
        Fs[s][2] = U[s][2] * un - b1 * bn;
        Fs[s][3] = U[s][3] * un - b2 * bn;
        Fs[s][4] = un * (e + pt) - bn * vb;
        Fs[s][6] = un * b1 - bn * u1;
        Fs[s][7] = un * b2 - bn * u2;
        const R r = rcpR(rho);
        const R a2 = gamma * p * r, B2 = bb * r, bd2 = bn * bn * r;
        const R sum = a2 + B2;
        const R disc = fmaxR(sum * sum - R(4) * a2 * bd2, R(0));
        c[s] = sqrtR(R(0.5) * (sum + sqrtR(disc)));
    }
    const R SL = fminR(wL[1] - c[0], wR[1] - c[1]);
    const R SR = fmaxR(wL[1] + c[0], wR[1] + c[1]);
    const R ap = fmaxR(SR, R(0)), bm = fminR(SL, R(0));
    const R inv = rcpR(ap - bm);
    const R ab = ap * bm;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        if (v == 5) continue;
        F[v] = ((ap * Fs[0][v] - bm * Fs[1][v]) + ab * (U[1][v] - U[0][v])) * inv;
    }
    F[5] = ps;
    F[8] = ch * ch * bn;
}

// FP64: the same flux as al F_L + be F_R + k (U_L - U_R), al, be and k as in
// riemann_euler, with F = u U + Phi for either side, Phi the pressure, tension
// and induction terms: M, B and differences before products as there (sums
// a U_L + b U_R lost the digits of slow flow: densities after ten steps 1.24e-16
// off against 64 bits instead of 0.93e-16; they took two steps of 18 944 blocks
// 22.22 instead of 22.51 ms), the normal tension taken from the pressures
// before they are weighted. Fast speed without division: with x = gamma p + B^2 and
// D = sqrt(x^2 - 4 gamma p B_n^2), c_f = sqrt((x + D)/(2 rho)) =
// (x + D)/sqrt(2 (x + D) rho); D^2 is kept above 1e-40 x^2, where D no longer
// counts, instead of 0.
__device__ __forceinline__ double mhd_fast_speed(double rho, double gp, double bb, double bn2) {
    const double x = gp + bb, x2 = x * x;
    const double q = __builtin_fmax(fma(-4.0 * gp, bn2, x2), 1e-40 * x2);
    const double y = __builtin_amdgcn_rsq(q), d = q * y;
    const double z = x + fma(0.5 * d, fma(-d, y, 1.0), d);
    const double s = (z + z) * rho;
    const double r = __builtin_amdgcn_rsq(s), c = z * r;
    return fma(0.5 * c, fma(-s * r, r, 1.0), c);
}
__device__ __forceinline__ void mhd_hll(const double wL[9], const double wR[9], double gamma, double igm1, double ch,
                                        double inv2ch, double F[9]) {
    const double bn = fma(0.5, wL[5] + wR[5], (wL[8] - wR[8]) * inv2ch);
    const double uL = wL[1], uR = wR[1];
    const double bn2 = bn * bn;
    const double bbL = fma(wL[7], wL[7], fma(wL[6], wL[6], bn2));
    const double bbR = fma(wR[7], wR[7], fma(wR[6], wR[6], bn2));
    const double cL = mhd_fast_speed(wL[0], gamma * wL[4], bbL, bn2);
    const double cR = mhd_fast_speed(wR[0], gamma * wR[4], bbR, bn2);
    const double sr = __builtin_fmax(__builtin_fmax(uL + cL, uR + cR), 0.0);
    const double sl = __builtin_fmin(__builtin_fmin(uL - cL, uR - cR), 0.0);
    const double inv = rcp64(sr - sl);
    const double al = sr * inv, be = -sl * inv;
    const double k = sr * be;
    const double a = al * uL, b = be * uR;
    const double mR = b * wR[0];
    const double M = fma(k, wL[0] - wR[0], fma(a, wL[0], mR));
    const double B = fma(-k, wR[0], mR);
    const double ptL = fma(0.5, bbL, wL[4]), ptR = fma(0.5, bbR, wR[4]);
    const double m1 = fma(al, wL[6], be * wR[6]), m2 = fma(al, wL[7], be * wR[7]);   // mean fields
    const double n1 = fma(al, wL[2], be * wR[2]), n2 = fma(al, wL[3], be * wR[3]);   // and velocities
    F[0] = M;
    F[1] = fma(M, uL, fma(B, uR - uL, fma(al, ptL - bn2, be * (ptR - bn2))));
    F[2] = fma(M, wL[2], fma(B, wR[2] - wL[2], -bn * m1));
    F[3] = fma(M, wL[3], fma(B, wR[3] - wL[3], -bn * m2));
    F[6] = fma(k, wL[6] - wR[6], fma(a, wL[6], fma(b, wR[6], -bn * n1)));
    F[7] = fma(k, wL[7] - wR[7], fma(a, wL[7], fma(b, wR[7], -bn * n2)));
    const double vvL = fma(wL[3], wL[3], fma(wL[2], wL[2], uL * uL));
    const double vvR = fma(wR[3], wR[3], fma(wR[2], wR[2], uR * uR));
    const double vbL = fma(wL[3], wL[7], fma(wL[2], wL[6], uL * bn));
    const double vbR = fma(wR[3], wR[7], fma(wR[2], wR[6], uR * bn));
    const double eL = fma(0.5, bbL, wL[4] * igm1), eR = fma(0.5, bbR, wR[4] * igm1);
    const double work = fma(a, ptL, fma(b, ptR, -bn * fma(al, vbL, be * vbR)));
    F[4] = fma(0.5, fma(M, vvL, B * (vvR - vvL)), fma(k, eL - eR, fma(a, eL, fma(b, eR, work))));
    F[5] = 0.5 * fma(-ch, wR[5] - wL[5], wL[8] + wR[8]);
    F[8] = ch * ch * bn;
}

} // namespace agile
