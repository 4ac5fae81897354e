// euler.h -- per-cell and per-face arithmetic of the Euler equations shared by
// the fused MUSCL-Hancock solver and its CTU variant: positivity test,
// limiters, physical fluxes, the Hancock predictor, Roe's flux with the
// Harten-Hyman entropy fix and the HLLE fallback, and the fixed-order
// per-group stats reduction.
//
// The kernels that use these functions are bound by VALU issue (float) or close
// to it (double), so the forms below are chosen for their instruction count.
// Each function contracts multiply-adds within one expression only (fp
// contract(on)), which makes its rounding a property of the source: a face state
// or a face flux has the same bits in every kernel and at every place it is
// inlined, whatever the register budget.  Against the plain forms (slopes with
// theta multiplied in, physical fluxes formed and then subtracted, the
// dissipation summed over all five waves; euler_mixed.h) the 256^3 padded step
// took 577 -> 556 us in float (1,247 -> 1,160 vector instructions per cell) and
// 1,070 -> 1,024 us in double, where they were taken.  Rounding error against 64-bit
// significands over smooth, supersonic and Mach-5 flows, relative to the plain forms:
// 0.97 to 0.99 in float, 0.99 to 1.00 in double (rms per variable).
#pragma once

#include "device_math.h"
#include "internal.h"

namespace gamer {
namespace {

template <typename T>
__device__ __forceinline__ bool physical(const T u[NV]) {
#pragma clang fp contract(on)
    // rho > 0 and p > 0  <=>  rho > 0 and 2 rho E > |m|^2
    return u[0] > T(0) && (u[0] + u[0]) * u[4] > u[1] * u[1] + u[2] * u[2] + u[3] * u[3];
}

// Generalised minmod over theta: 0 at extrema (a b <= 0), else sign(a) min(|a|,
// |b|, |a+b| / (2 theta)); k1 = 1 / (2 theta).  The slope is theta times this, and
// the factor is taken where the face values are formed (c.ht = theta / 2), which
// spares two multiplications per slope.  In float it is evaluated as med3(a,
// med3(b, k1 (a+b), 0), 0): the median with 0 is the two-argument minmod, and
// nesting it gives the same value bitwise whenever a and b share a sign (and 0
// otherwise).
__device__ __forceinline__ float limiter(float a, float b, float k1) {
#pragma clang fp contract(on)
    const float inner = __builtin_amdgcn_fmed3f(b, k1 * (a + b), 0.0f);
    return __builtin_amdgcn_fmed3f(a, inner, 0.0f);
}
// In double, without a branch: bs = b with the sign of a is positive exactly
// when a and b share a sign, and then |a| + bs = |a + b|; otherwise bs <= 0 and
// the clamp at 0 gives a zero slope (of either sign).
__device__ __forceinline__ double limiter(double a, double b, double k1) {
#pragma clang fp contract(on)
    const double aa = fabs(a);
    const double bs = __builtin_copysign(1.0, a) * b;
    const double m = fmin(aa, fmin(bs, k1 * (aa + bs)));
    return __builtin_copysign(fmax(m, 0.0), a);
}

// Limited slope along direction D in characteristic variables: the one-sided
// primitive differences a, b are projected on the left eigenvectors of the
// primitive system along D at the cell state, each wave's pair is limited,
// and the limited amplitudes are mapped back with the right eigenvectors.
// Component order (rho, normal velocity, two transverse velocities, p):
//   u - c: l = (0, -rho/2c, 0, 0, 1/2c^2), r = (1, -c/rho, 0, 0, c^2)
//   u (entropy): l = (1, 0, 0, 0, -1/c^2), r = (1, 0, 0, 0, 0)
//   u (shear, two): unit vectors of the transverse velocities
//   u + c: l = (0, rho/2c, 0, 0, 1/2c^2), r = (1, c/rho, 0, 0, c^2)
// h = rho/(2c), q = 1/(2c^2), cr = c/rho, c2 = c^2 of the cell.  Slopes over
// theta, as the limiter gives them.
template <int D, typename T>
__device__ __forceinline__ void char_slope(const T a[NV], const T b[NV], T h, T q, T cr, T c2,
                                           T k1, T dw[NV]) {
#pragma clang fp contract(on)
    constexpr int N = 1 + D, T1 = D == 0 ? 2 : 1, T2 = D == 2 ? 2 : 3;
    const T m0 = limiter(q * a[4] - h * a[N], q * b[4] - h * b[N], k1);
    const T m1 = limiter(a[0] - T(2) * q * a[4], b[0] - T(2) * q * b[4], k1);
    const T m4 = limiter(q * a[4] + h * a[N], q * b[4] + h * b[N], k1);
    dw[0] = m0 + m1 + m4;
    dw[N] = cr * (m4 - m0);
    dw[T1] = limiter(a[T1], b[T1], k1);
    dw[T2] = limiter(a[T2], b[T2], k1);
    dw[4] = c2 * (m0 + m4);
}

// Physical flux along direction D of a primitive state (rho, u_x, u_y, u_z, p).
template <int D, typename T>
__device__ __forceinline__ void flux_prim(const T w[NV], const Consts<T> &c, T f[NV]) {
#pragma clang fp contract(on)
    const T un = w[1 + D];
    const T e = w[4] * c.igm1 + c.half * w[0] * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
    const T mn = w[0] * un;
    f[0] = mn;
    f[1] = mn * w[1];
    f[2] = mn * w[2];
    f[3] = mn * w[3];
    f[1 + D] += w[4];
    f[4] = (e + w[4]) * un;
}

// Conserved variables of a primitive state.
template <typename T>
__device__ __forceinline__ void cons_prim(const T w[NV], const Consts<T> &c, T u[NV]) {
#pragma clang fp contract(on)
    u[0] = w[0];
    u[1] = w[0] * w[1];
    u[2] = w[0] * w[2];
    u[3] = w[0] * w[3];
    u[4] = w[4] * c.igm1 + c.half * w[0] * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
}

// One direction D of the half-step prediction: the two face states W0 -+ dW/2
// (dw: the slope over theta) as density, velocities, momentum along D and energy,
// and their flux difference taken into the increment,
//   S += F_D(minus) - F_D(plus),
// product by product: every term but the pressure's is one multiply-add (the
// pressure's is -dp of the slope), against a flux formed, subtracted and added.  The
// energy's larger product, the internal energy at Mach numbers below one, is the one
// that goes unrounded into the multiply-add (float: 6% off the mass flux's error).
template <typename T>
struct FacePair {
    T rho[2], u[2][3], mn[2], e[2];
};
template <int D, typename T>
__device__ __forceinline__ void face_pair(const T W0[NV], const T dw[NV], const Consts<T> &c, T S[NV],
                                          FacePair<T> &f) {
#pragma clang fp contract(on)
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        T w[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = side ? W0[v] + c.ht * dw[v] : W0[v] - c.ht * dw[v];
        const T r = w[0], p = w[4], un = w[1 + D];
        const T mn = r * un;
        const T e = p * c.igm1 + (c.half * r) * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
        f.rho[side] = r;
        f.mn[side] = mn;
        f.e[side] = e;
#pragma unroll
        for (int q = 0; q < 3; ++q) f.u[side][q] = w[1 + q];
        if (D == 0 && side == 0) {
            S[0] = mn;
#pragma unroll
            for (int q = 0; q < 3; ++q) S[1 + q] = mn * w[1 + q];
            S[4] = (e + p) * un;
        } else if (side == 0) {
            S[0] = S[0] + mn;
#pragma unroll
            for (int q = 0; q < 3; ++q) S[1 + q] = S[1 + q] + mn * w[1 + q];
            S[4] = S[4] + (e + p) * un;
        } else {
            S[0] = S[0] - mn;
#pragma unroll
            for (int q = 0; q < 3; ++q) S[1 + q] = S[1 + q] - mn * w[1 + q];
            S[4] = S[4] - (e + p) * un;
        }
    }
    S[1 + D] = S[1 + D] - c.theta * dw[4];
}

// Half-step prediction of one cell (conservative Hancock step, all three
// directions): face values W0 -+ dW_d/2, the common increment
//   S = dt/(2dh) sum_d [F_d(W0 - dW_d/2) - F_d(W0 + dW_d/2)],
// and Ub[d][0] (minus face), Ub[d][1] (plus face) = cons(W0 -+ dW_d/2) + S.
// dW: the slopes over theta.  Returns false if any of the six has rho <= 0 or
// p <= 0.
template <typename T>
__device__ __forceinline__ bool predict(const T W0[NV], const T dW[3][NV], T hdt,
                                        const Consts<T> &c, T Ub[3][2][NV]) {
#pragma clang fp contract(on)
    T S[NV];
    FacePair<T> f[3];
    face_pair<0>(W0, dW[0], c, S, f[0]);
    face_pair<1>(W0, dW[1], c, S, f[1]);
    face_pair<2>(W0, dW[2], c, S, f[2]);
#pragma unroll
    for (int v = 0; v < NV; ++v) S[v] = S[v] * hdt;
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            T *U = Ub[d][side];
            U[0] = f[d].rho[side] + S[0];
#pragma unroll
            for (int q = 0; q < 3; ++q)
                U[1 + q] = q == d ? f[d].mn[side] + S[1 + q] : S[1 + q] + f[d].rho[side] * f[d].u[side][q];
            U[4] = f[d].e[side] + S[4];
            ok = ok && physical(U);
        }
    }
    return ok;
}

// Physical flux of a rotated conserved state (normal = component 1), given
// its normal velocity and pressure.
template <typename T>
__device__ __forceinline__ void rot_flux(const T U[NV], T un, T p, T F[NV]) {
#pragma clang fp contract(on)
    F[0] = U[1];
    F[1] = U[1] * un + p;
    F[2] = U[2] * un;
    F[3] = U[3] * un;
    F[4] = (U[4] + p) * un;
}

// HLLE flux (Einfeldt) with signal speeds SL, SR.
template <typename T>
__device__ __forceinline__ void hlle(const T L[NV], const T R[NV], T uL, T pL, T uR, T pR, T SL, T SR,
                                  T F[NV]) {
#pragma clang fp contract(on)
    T FL[NV], FR[NV];
    rot_flux(L, uL, pL, FL);
    rot_flux(R, uR, pR, FR);
    if (SL >= T(0)) {
#pragma unroll
        for (int m = 0; m < NV; ++m) F[m] = FL[m];
    } else if (SR <= T(0)) {
#pragma unroll
        for (int m = 0; m < NV; ++m) F[m] = FR[m];
    } else {
        const T id = rcp(SR - SL);
#pragma unroll
        for (int m = 0; m < NV; ++m) F[m] = (SR * FL[m] - SL * FR[m] + SL * SR * (R[m] - L[m])) * id;
    }
}

// Roe flux between rotated conserved states (component 1 = normal momentum).
// Harten-Hyman entropy fix on the acoustic waves, HLLE when a2 <= 0 or an
// intermediate state is unphysical.  Returns true when HLLE was used.
// Arithmetic layout: one reciprocal square root per side gives sqrt(rho) and 1/rho
// (one of the product rho_L rho_R would give both sides' with an instruction or two
// less, but leaves the double range at densities of 1e-154 and 1e154, and gives two
// negative densities a root); one of a2 gives a and 1/a; the intermediate states'
// positivity and rho c come from Q = 2 rho E - |m|^2 (p > 0 <=> Q > 0, (rho c)^2 =
// gq Q), so they need no reciprocal unless the entropy fix is active on that lane.
// In double, where a square root is a refined estimate of about fifteen
// instructions, the entropy fix is tested on squared speeds (c^2 = gamma p /
// rho, (rho* c*)^2 = gq Q*), and the square roots are taken only on lanes where
// the fix is active or HLLE is used; in float the square root is one hardware
// instruction and the speeds are formed directly.
// The dissipation sum_k |lambda_k| alpha_k K_k is taken as |u| (U_R - U_L), which
// is |u| times all five waves, plus (|lambda_k| - |u|) alpha_k K_k of the two
// acoustic waves: the three waves of speed u then need no strengths, and with
// dp = (gamma-1)(dE - u.dm + |u|^2/2 drho) and dm_n - u drho, the acoustic ones
// are (dp -+ a (dm_n - u drho)) / (2 a2).
// Rounding: what the dissipation and the pressures are made of is added up before it
// meets the far larger sums of the two physical fluxes, one rounding at their size.
// Subtracted from them term by term, the momentum fluxes' error grew by a fifth in
// smooth flow (rms against 64-bit significands, both types; as here 0.97 to 1.01 of
// the plain form's, which subtracts the fluxes of two formed wave sums).
//
// TWICE: return 2F instead of F.  Every component of F is half of a sum, and
// halving is exact, so a caller that scales its use of the flux by 1/2 (the
// update's dt/dh, the flux planes it stores) gets the same values bitwise
// without the five multiplications.
template <typename T, bool TWICE = false>
__device__ __forceinline__ bool roe(const T L[NV], const T R[NV], const Consts<T> &c, T F[NV]) {
#pragma clang fp contract(on)
    const T h = c.half;
    const T hf = TWICE ? T(1) : h;  // the flux sums' factor
    const T qL = rsq(L[0]), qR = rsq(R[0]);
    const T irL = qL * qL, irR = qR * qR;
    const T uL = L[1] * irL, vL = L[2] * irL, wL = L[3] * irL;
    const T uR = R[1] * irR, vR = R[2] * irR, wR = R[3] * irR;
    const T kL = L[1] * uL, kR = R[1] * uR;
    const T iL = L[4] - h * (kL + L[2] * vL + L[3] * wL);  // internal energies
    const T iR = R[4] - h * (kR + R[2] * vR + R[3] * wR);
    const T pL = c.gm1 * iL, pR = c.gm1 * iR;
    // HLLE's pressures: in float formed again there, so that only the internal energies
    // stay in registers for the flux sums (256^3 periodic 603 -> 595 us; in double the
    // other way round, CTU 9 x 8 x 7 groups 376 -> 364 us)
    auto hlle_p = [&](T i, T p) { return sizeof(T) == 4 ? c.gm1 * fresh(i) : p; };
    const T c2L = c.g * pL * irL, c2R = c.g * pR * irR;  // squared sound speeds
    const T eL = L[4] + pL, eR = R[4] + pR;

    // Roe averages with weights sqrt(rho): sqrt(rho) u = m / sqrt(rho)
    const T is = rcp(L[0] * qL + R[0] * qR);
    const T u = (L[1] * qL + R[1] * qR) * is;
    const T v = (L[2] * qL + R[2] * qR) * is;
    const T w = (L[3] * qL + R[3] * qR) * is;
    const T H = (eL * qL + eR * qR) * is;
    const T hq2 = h * (u * u + v * v + w * w);
    const T a2 = c.gm1 * (H - hq2);
    if (!(a2 > T(0))) {
        hlle(L, R, uL, hlle_p(iL, pL), uR, hlle_p(iR, pR), uL - sqrt_(c2L), uR + sqrt_(c2R), F);
        if (TWICE) {
#pragma unroll
            for (int m = 0; m < NV; ++m) F[m] *= T(2);
        }
        return true;
    }
    const T ia = rsq(a2);
    const T a = a2 * ia;
    const T D0 = R[0] - L[0], D1 = R[1] - L[1], D2 = R[2] - L[2], D3 = R[3] - L[3],
            D4 = R[4] - L[4];
    const T dp = D4 - u * D1 - v * D2 - w * D3 + hq2 * D0;  // over gamma - 1
    const T X = a * (D1 - u * D0);
    const T k = h * (ia * ia);
    const T al1 = (c.gm1 * dp - X) * k, al5 = (c.gm1 * dp + X) * k;
    const T lam1 = u - a, lam5 = u + a;

    // states on the inner sides of the two acoustic waves
    const T Ls[NV] = {L[0] + al1, L[1] + al1 * lam1, L[2] + al1 * v, L[3] + al1 * w,
                      L[4] + al1 * (H - u * a)};
    const T Rs[NV] = {R[0] - al5, R[1] - al5 * lam5, R[2] - al5 * v, R[3] - al5 * w,
                      R[4] - al5 * (H + u * a)};
    const T QL = (Ls[0] + Ls[0]) * Ls[4] - (Ls[1] * Ls[1] + Ls[2] * Ls[2] + Ls[3] * Ls[3]);
    const T QR = (Rs[0] + Rs[0]) * Rs[4] - (Rs[1] * Rs[1] + Rs[2] * Rs[2] + Rs[3] * Rs[3]);
    if (!(Ls[0] > T(0) && QL > T(0) && Rs[0] > T(0) && QR > T(0))) {
        hlle(L, R, uL, hlle_p(iL, pL), uR, hlle_p(iR, pR), fmin(uL - sqrt_(c2L), lam1), fmax(uR + sqrt_(c2R), lam5), F);
        if (TWICE) {
#pragma unroll
            for (int m = 0; m < NV; ++m) F[m] *= T(2);
        }
        return true;
    }
    // Harten-Hyman: wave 1 between L (speed uL - cL) and L* (speed (m* - rho* c*)/rho*),
    // wave 5 between R* (speed (m* + rho* c*)/rho*) and R (speed uR + cR).  The fix is
    // active when |lambda| < lambda - lambda_left or |lambda| < lambda_right - lambda.
    T ab1 = fabs(lam1), ab5 = fabs(lam5);
    if constexpr (sizeof(T) == 4) {
        const T cL = sqrt_(c2L), cR = sqrt_(c2R);
        const T rcLs = sqrt_(c.gq * QL), rcRs = sqrt_(c.gq * QR);  // rho* c*
        const T t1a = lam1 - (uL - cL);
        const T t1b_r = (Ls[1] - rcLs) - lam1 * Ls[0];  // (lambda_right - lambda) rho*
        const T t5b = (uR + cR) - lam5;
        const T t5a_r = lam5 * Rs[0] - (Rs[1] + rcRs);  // (lambda - lambda_left) rho*
        if (ab1 < t1a || ab1 * Ls[0] < t1b_r) {
            const T e = fmax(t1a, t1b_r * rcp(Ls[0]));
            ab1 = (lam1 * lam1 + e * e) * (h * rcp(e));
        }
        if (ab5 < t5b || ab5 * Rs[0] < t5a_r) {
            const T e = fmax(t5b, t5a_r * rcp(Rs[0]));
            ab5 = (lam5 * lam5 + e * e) * (h * rcp(e));
        }
    } else {
        // with the speeds' square roots isolated the tests read, for wave 1,
        //   cL > |lam1| - (lam1 - uL)     and   rho* c* < m* - (lam1 + |lam1|) rho*,
        // and for wave 5
        //   cR > |lam5| + (lam5 - uR)     and   rho* c* < (lam5 - |lam5|) rho* - m*,
        // each compared through the squares when its right-hand side is positive
        const T A1 = ab1 - (lam1 - uL), B1 = Ls[1] - (lam1 + ab1) * Ls[0];
        const T A5 = ab5 + (lam5 - uR), B5 = (lam5 - ab5) * Rs[0] - Rs[1];
        const bool fix1 = A1 < T(0) || c2L > A1 * A1 || (B1 > T(0) && c.gq * QL < B1 * B1);
        const bool fix5 = A5 < T(0) || c2R > A5 * A5 || (B5 > T(0) && c.gq * QR < B5 * B5);
        // Faces with either fix take its two square roots and two reciprocals (one
        // of rho*^2 e would do, over half the range) together, wave 5 as the mirror
        // image of wave 1; hardly any face has both.
        // In a flow of strong contrasts a seventh of the faces has one of them, so
        // that most waves hold both kinds: 1,009 groups with flux planes 338 ->
        // 329 us, and fewer registers (256^3 periodic, smooth, 1,055 -> 1,037 us);
        // 333 and 1,042 us with the second reciprocal and a root per side.
        if (fix1 || fix5) {
            const T s1 = sqrt_(fix1 ? c2L : c2R), s2 = sqrt_(c.gq * (fix1 ? QL : QR));
            const T lam = fix1 ? lam1 : -lam5, us = fix1 ? uL : -uR;
            const T ms = fix1 ? Ls[1] : -Rs[1], rs = fix1 ? Ls[0] : Rs[0];
            const T e = fmax(lam - (us - s1), ((ms - s2) - lam * rs) * rcp(rs));  // the larger gap
            const T ab = (lam * lam + e * e) * (h * rcp(e));
            // The gap has to exceed |lambda| itself: the squares above may pass a face
            // whose gap comes out as |lambda| or less, down to zero at a uniform flow
            // of exactly the speed of sound (where the quotient would be 0 / 0).
            const bool wide = e > fabs(lam);
            ab1 = fix1 && wide ? ab : ab1;
            ab5 = !fix1 && wide ? ab : ab5;
            if (fix1 && fix5) {
                const T e5 = fmax((uR + sqrt_(c2R)) - lam5, (lam5 * Rs[0] - (Rs[1] + sqrt_(c.gq * QR))) * rcp(Rs[0]));
                if (e5 > fabs(lam5)) ab5 = (lam5 * lam5 + e5 * e5) * (h * rcp(e5));
            }
        }
    }

    const T ab2 = fabs(u);
    const T d5 = ab5 - ab2, e1 = al1 * (ab1 - ab2);
    const T es = e1 + al5 * d5, et = a * (al5 * d5 - e1);
    F[0] = hf * ((L[1] + R[1]) - (es + ab2 * D0));
    F[1] = hf * (((kL + c.gm1 * iL) + (kR + c.gm1 * iR)) - (et + es * u + ab2 * D1));
    F[2] = hf * ((L[2] * uL + R[2] * uR) - (es * v + ab2 * D2));
    F[3] = hf * ((L[3] * uL + R[3] * uR) - (es * w + ab2 * D3));
    F[4] = hf * ((eL * uL + eR * uR) - (es * H + et * u + ab2 * D4));
    return false;
}

// Roe flux along direction D for unrotated conserved states (2F with TWICE).
template <int D, bool TWICE = false, typename T>
__device__ __forceinline__ bool roe_dir(const T UL[NV], const T UR[NV], const Consts<T> &c,
                                        T F[NV]) {
    constexpr int n = 1 + D, t1 = 1 + (D + 1) % 3, t2 = 1 + (D + 2) % 3;
    const T L[NV] = {UL[0], UL[n], UL[t1], UL[t2], UL[4]};
    const T R[NV] = {UR[0], UR[n], UR[t1], UR[t2], UR[4]};
    T Fr[NV];
    const bool fb = roe<T, TWICE>(L, R, c, Fr);
    F[0] = Fr[0];
    F[n] = Fr[1];
    F[t1] = Fr[2];
    F[t2] = Fr[3];
    F[4] = Fr[4];
    return fb;
}

// The arithmetic above as one argument of a kernel (the FP64-state, FP32-arithmetic
// path takes MixedArith of euler_mixed.h instead).
template <typename T>
struct Arith {
    static __device__ __forceinline__ T limiter(T a, T b, const Consts<T> &c) { return gamer::limiter(a, b, c.k1); }
    template <int D>
    static __device__ __forceinline__ void char_slope(const T a[NV], const T b[NV], T h, T q, T cr, T c2,
                                                      const Consts<T> &c, T dw[NV]) {
        gamer::char_slope<D>(a, b, h, q, cr, c2, c.k1, dw);
    }
    static __device__ __forceinline__ bool predict(const T W0[NV], const T dW[3][NV], T hdt, const Consts<T> &c,
                                                   T Ub[3][2][NV]) {
        return gamer::predict(W0, dW, hdt, c, Ub);
    }
    // Roe's flux doubled
    static __device__ __forceinline__ bool roe2(const T L[NV], const T R[NV], const Consts<T> &c, T F[NV]) {
        return gamer::roe<T, true>(L, R, c, F);
    }
};

// Fixed-order reduction of NSTAT doubles per thread over NTHREADS threads
// (thread index t, 0 .. NTHREADS - 1, NTHREADS a multiple of 64 when the
// work-group holds several such sets): stats 0..4 and 6..7 are summed, stat 5
// is a maximum that keeps NaN.  Thread 0 writes the result to dst (if not
// null).  The values go through LDS PART at a time; `red` must hold
// NTHREADS * PART doubles.  Each value is folded in the same order whatever
// PART is: thread t takes the values of threads t, t + 64, ..., then the 64
// partial results are folded by halving.
template <int NTHREADS, int PART = NSTAT>
__device__ __forceinline__ void block_reduce_stats(double st[NSTAT], double *red, double *dst,
                                                   int t = threadIdx.x) {
    static_assert(NSTAT % PART == 0, "whole passes");
#pragma unroll
    for (int q0 = 0; q0 < NSTAT; q0 += PART) {
#pragma unroll
        for (int q = 0; q < PART; ++q) red[q * NTHREADS + t] = st[q0 + q];
        __syncthreads();
        if (t < 64) {
            double acc[PART];
#pragma unroll
            for (int q = 0; q < PART; ++q) {
                double a = red[q * NTHREADS + t];
                for (int s = t + 64; s < NTHREADS; s += 64) {
                    const double b = red[q * NTHREADS + s];
                    a = (q0 + q == 5) ? max_nan(a, b) : a + b;
                }
                acc[q] = a;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
                for (int q = 0; q < PART; ++q) {
                    const double b = __shfl_down(acc[q], off, 64);
                    acc[q] = (q0 + q == 5) ? max_nan(acc[q], b) : acc[q] + b;
                }
            }
            if (t == 0 && dst) {
#pragma unroll
                for (int q = 0; q < PART; ++q) dst[q0 + q] = acc[q];
            }
        }
        __syncthreads();
    }
}

}  // namespace
}  // namespace gamer
