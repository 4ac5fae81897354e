// euler_mixed.h -- the float arithmetic of the FP64-state, FP32-arithmetic path:
// limiters, Hancock predictor and Roe's flux in the order of operations that they
// had before euler.h's shorter forms.  That path stores its result in double, where
// a float operation taken in another order shows in the ninth digit.  With periodic
// input its values are those of the earlier kernels bitwise.  With padded input the
// default variant now gives the same bits as with periodic input, which it did not
// before: up to 2e-8 of the state's norm in a flow of strong contrasts, half the
// step's own error.  The predictor's and the fluxes' multiply-adds are the
// compiler's choice (unlike those of euler.h, and of the limiters here): to fix them
// by the source would move those values again.
#pragma once

#include "euler.h"

namespace gamer {
namespace {

struct MixedArith {
    static __device__ __forceinline__ bool physical(const float u[NV]) {
        // rho > 0 and p > 0  <=>  rho > 0 and 2 rho E > |m|^2
        return u[0] > float(0) && float(2) * u[0] * u[4] > u[1] * u[1] + u[2] * u[2] + u[3] * u[3];
    }

    // Generalised minmod: 0 at extrema (a b <= 0), else sign(a) min(theta|a|,
    // theta|b|, |a+b|/2).  In float it is evaluated as med3(theta a,
    // med3(theta b, (a+b)/2, 0), 0): the median with 0 is the two-argument minmod,
    // and nesting it gives the same value bitwise whenever a and b share a sign
    // (and 0 otherwise); only an a b that underflows to 0 would differ.
    static __device__ __forceinline__ float limiter(float a, float b, const Consts<float> &c) {
#pragma clang fp contract(on)
        const float theta = c.theta;
        const float inner = __builtin_amdgcn_fmed3f(theta * b, 0.5f * (a + b), 0.0f);
        return __builtin_amdgcn_fmed3f(theta * a, inner, 0.0f);
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
    // h = rho/(2c), q = 1/(2c^2), cr = c/rho, c2 = c^2 of the cell.
    template <int D>
    static __device__ __forceinline__ void char_slope(const float a[NV], const float b[NV], float h, float q, float cr, float c2,
                                               const Consts<float> &c, float dw[NV]) {
#pragma clang fp contract(on)
        constexpr int N = 1 + D, T1 = D == 0 ? 2 : 1, T2 = D == 2 ? 2 : 3;
        const float m0 = limiter(q * a[4] - h * a[N], q * b[4] - h * b[N], c);
        const float m1 = limiter(a[0] - float(2) * q * a[4], b[0] - float(2) * q * b[4], c);
        const float m4 = limiter(q * a[4] + h * a[N], q * b[4] + h * b[N], c);
        dw[0] = m0 + m1 + m4;
        dw[N] = cr * (m4 - m0);
        dw[T1] = limiter(a[T1], b[T1], c);
        dw[T2] = limiter(a[T2], b[T2], c);
        dw[4] = c2 * (m0 + m4);
    }

    // Physical flux along direction D of a primitive state (rho, u_x, u_y, u_z, p).
    template <int D>
    static __device__ __forceinline__ void flux_prim(const float w[NV], const Consts<float> &c, float f[NV]) {
        const float un = w[1 + D];
        const float e = w[4] * c.igm1 + c.half * w[0] * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
        const float mn = w[0] * un;
        f[0] = mn;
        f[1] = mn * w[1];
        f[2] = mn * w[2];
        f[3] = mn * w[3];
        f[1 + D] += w[4];
        f[4] = (e + w[4]) * un;
    }

    // Conserved variables of a primitive state.
    static __device__ __forceinline__ void cons_prim(const float w[NV], const Consts<float> &c, float u[NV]) {
        u[0] = w[0];
        u[1] = w[0] * w[1];
        u[2] = w[0] * w[2];
        u[3] = w[0] * w[3];
        u[4] = w[4] * c.igm1 + c.half * w[0] * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
    }

    // S += F_D(W0 - dW/2) - F_D(W0 + dW/2)
    template <int D>
    static __device__ __forceinline__ void flux_difference(const float W0[NV], const float dw[NV], const Consts<float> &c,
                                                    float Sv[NV]) {
        float wm[NV], wp[NV], fm[NV], fp[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            wm[v] = W0[v] - c.half * dw[v];
            wp[v] = W0[v] + c.half * dw[v];
        }
        flux_prim<D>(wm, c, fm);
        flux_prim<D>(wp, c, fp);
#pragma unroll
        for (int v = 0; v < NV; ++v) Sv[v] += fm[v] - fp[v];
    }

    // Half-step prediction of one cell (conservative Hancock step, all three
    // directions): face values W0 -+ dW_d/2, the common increment
    //   S = dt/(2dh) sum_d [F_d(W0 - dW_d/2) - F_d(W0 + dW_d/2)],
    // and Ub[d][0] (minus face), Ub[d][1] (plus face) = cons(W0 -+ dW_d/2) + S.
    // Returns false if any of the six has rho <= 0 or p <= 0.
    static __device__ __forceinline__ bool predict(const float W0[NV], const float dW[3][NV], float hdt,
                                            const Consts<float> &c, float Ub[3][2][NV]) {
        float Sv[NV] = {float(0), float(0), float(0), float(0), float(0)};
        flux_difference<0>(W0, dW[0], c, Sv);
        flux_difference<1>(W0, dW[1], c, Sv);
        flux_difference<2>(W0, dW[2], c, Sv);
#pragma unroll
        for (int v = 0; v < NV; ++v) Sv[v] *= hdt;
        bool ok = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                float wf[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) wf[v] = W0[v] + float(side ? 1 : -1) * (c.half * dW[d][v]);
                cons_prim(wf, c, Ub[d][side]);
#pragma unroll
                for (int v = 0; v < NV; ++v) Ub[d][side][v] += Sv[v];
                ok = ok && physical(Ub[d][side]);
            }
        }
        return ok;
    }

    // Physical flux of a rotated conserved state (normal = component 1), given
    // its normal velocity and pressure.
    static __device__ __forceinline__ void rot_flux(const float U[NV], float un, float p, float F[NV]) {
        F[0] = U[1];
        F[1] = U[1] * un + p;
        F[2] = U[2] * un;
        F[3] = U[3] * un;
        F[4] = (U[4] + p) * un;
    }

    // HLLE flux (Einfeldt) with signal speeds SL, SR.
    static __device__ __forceinline__ void hlle(const float L[NV], const float R[NV], float uL, float pL, float uR, float pR, float SL, float SR,
                                      float F[NV]) {
        float FL[NV], FR[NV];
        rot_flux(L, uL, pL, FL);
        rot_flux(R, uR, pR, FR);
        if (SL >= float(0)) {
#pragma unroll
            for (int m = 0; m < NV; ++m) F[m] = FL[m];
        } else if (SR <= float(0)) {
#pragma unroll
            for (int m = 0; m < NV; ++m) F[m] = FR[m];
        } else {
            const float id = rcp(SR - SL);
#pragma unroll
            for (int m = 0; m < NV; ++m) F[m] = (SR * FL[m] - SL * FR[m] + SL * SR * (R[m] - L[m])) * id;
        }
    }

    // Roe flux between rotated conserved states (component 1 = normal momentum).
    // Harten-Hyman entropy fix on the acoustic waves, HLLE when a2 <= 0 or an
    // intermediate state is unphysical.  Returns true when HLLE was used.
    // Arithmetic layout: one reciprocal square root per side gives sqrt(rho) and
    // 1/rho; one of a2 gives a and 1/a; the intermediate states' positivity and
    // rho c come from Q = 2 rho E - |m|^2 (p > 0 <=> Q > 0, (rho c)^2 = gq Q), so
    // they need no reciprocal unless the entropy fix is active on that lane.
    //
    // TWICE: return 2F instead of F.  Every component of F is half of a sum, and
    // halving is exact, so a caller that scales its use of the flux by 1/2 (the
    // update's dt/dh, the flux planes it stores) gets the same values bitwise
    // without the five multiplications.
    template <bool TWICE = false>
    static __device__ __forceinline__ bool roe(const float L[NV], const float R[NV], const Consts<float> &c, float F[NV]) {
        const float h = c.half;
        const float hf = TWICE ? float(1) : h;  // the flux sums' factor
        const float qL = rsq(L[0]), qR = rsq(R[0]);
        const float irL = qL * qL, irR = qR * qR;
        const float uL = L[1] * irL, vL = L[2] * irL, wL = L[3] * irL;
        const float uR = R[1] * irR, vR = R[2] * irR, wR = R[3] * irR;
        const float pL = c.gm1 * (L[4] - h * (L[1] * uL + L[2] * vL + L[3] * wL));
        const float pR = c.gm1 * (R[4] - h * (R[1] * uR + R[2] * vR + R[3] * wR));
        const float c2L = c.g * pL * irL, c2R = c.g * pR * irR;  // squared sound speeds

        // Roe averages with weights sqrt(rho): sqrt(rho) u = m / sqrt(rho)
        const float is = rcp(L[0] * qL + R[0] * qR);
        const float u = (L[1] * qL + R[1] * qR) * is;
        const float v = (L[2] * qL + R[2] * qR) * is;
        const float w = (L[3] * qL + R[3] * qR) * is;
        const float H = ((L[4] + pL) * qL + (R[4] + pR) * qR) * is;
        const float q2 = u * u + v * v + w * w;
        const float a2 = c.gm1 * (H - h * q2);
        if (!(a2 > float(0))) {
            hlle(L, R, uL, pL, uR, pR, uL - sqrt_(c2L), uR + sqrt_(c2R), F);
            if (TWICE) {
#pragma unroll
                for (int m = 0; m < NV; ++m) F[m] *= float(2);
            }
            return true;
        }
        const float ia = rsq(a2);
        const float a = a2 * ia;
        const float D0 = R[0] - L[0], D1 = R[1] - L[1], D2 = R[2] - L[2], D3 = R[3] - L[3],
                D4 = R[4] - L[4];
        const float al3 = D2 - v * D0;
        const float al4 = D3 - w * D0;
        const float d5 = D4 - al3 * v - al4 * w;
        const float al2 = c.gm1 * (ia * ia) * (D0 * (H - u * u) + u * D1 - d5);
        const float al1 = (D0 * (u + a) - D1 - a * al2) * (h * ia);
        const float al5 = D0 - (al1 + al2);
        const float ua = u * a;

        // states on the inner sides of the two acoustic waves
        const float Ls[NV] = {L[0] + al1, L[1] + al1 * (u - a), L[2] + al1 * v, L[3] + al1 * w,
                          L[4] + al1 * (H - ua)};
        const float Rs[NV] = {R[0] - al5, R[1] - al5 * (u + a), R[2] - al5 * v, R[3] - al5 * w,
                          R[4] - al5 * (H + ua)};
        const float QL = float(2) * Ls[0] * Ls[4] - (Ls[1] * Ls[1] + Ls[2] * Ls[2] + Ls[3] * Ls[3]);
        const float QR = float(2) * Rs[0] * Rs[4] - (Rs[1] * Rs[1] + Rs[2] * Rs[2] + Rs[3] * Rs[3]);
        if (!(Ls[0] > float(0) && QL > float(0) && Rs[0] > float(0) && QR > float(0))) {
            hlle(L, R, uL, pL, uR, pR, fmin(uL - sqrt_(c2L), u - a), fmax(uR + sqrt_(c2R), u + a), F);
            if (TWICE) {
#pragma unroll
                for (int m = 0; m < NV; ++m) F[m] *= float(2);
            }
            return true;
        }
        // Harten-Hyman: wave 1 between L (speed uL - cL) and L* (speed (m* - rho* c*)/rho*),
        // wave 5 between R* (speed (m* + rho* c*)/rho*) and R (speed uR + cR).  The fix is
        // active when |lambda| < lambda - lambda_left or |lambda| < lambda_right - lambda.
        const float lam1 = u - a, lam5 = u + a;
        float ab1 = fabs(lam1), ab5 = fabs(lam5);
        const float cL = sqrt_(c2L), cR = sqrt_(c2R);
        const float rcLs = sqrt_(c.gq * QL), rcRs = sqrt_(c.gq * QR);  // rho* c*
        const float t1a = lam1 - (uL - cL);
        const float t1b_r = (Ls[1] - rcLs) - lam1 * Ls[0];  // (lambda_right - lambda) rho*
        const float t5b = (uR + cR) - lam5;
        const float t5a_r = lam5 * Rs[0] - (Rs[1] + rcRs);  // (lambda - lambda_left) rho*
        if (ab1 < t1a || ab1 * Ls[0] < t1b_r) {
            const float e = fmax(t1a, t1b_r * rcp(Ls[0]));
            ab1 = (lam1 * lam1 + e * e) * (h * rcp(e));
        }
        if (ab5 < t5b || ab5 * Rs[0] < t5a_r) {
            const float e = fmax(t5b, t5a_r * rcp(Rs[0]));
            ab5 = (lam5 * lam5 + e * e) * (h * rcp(e));
        }
        const float ab2 = fabs(u);

        // dissipation sum_k |lambda_k| alpha_k K_k: waves 1, 2 and 5 share the
        // transverse components v and w of their eigenvectors, so those rows take
        // the sum of the three amplitudes once
        const float c1 = al1 * ab1, c2 = al2 * ab2, c3 = al3 * ab2, c4 = al4 * ab2, c5 = al5 * ab5;
        const float s125 = (c1 + c2) + c5;
        F[0] = hf * ((L[1] + R[1]) - s125);
        F[1] = hf * ((L[1] * uL + pL + R[1] * uR + pR) - ((c1 * (u - a) + c2 * u) + c5 * (u + a)));
        F[2] = hf * ((L[2] * uL + R[2] * uR) - (s125 * v + c3));
        F[3] = hf * ((L[3] * uL + R[3] * uR) - (s125 * w + c4));
        F[4] = hf * (((L[4] + pL) * uL + (R[4] + pR) * uR) -
                     ((((c1 * (H - ua) + c2 * (h * q2)) + c3 * v) + c4 * w) + c5 * (H + ua)));
        return false;
    }

    // Roe's flux doubled
    static __device__ __forceinline__ bool roe2(const float L[NV], const float R[NV], const Consts<float> &c,
                                                float F[NV]) {
        return roe<true>(L, R, c, F);
    }
};

}  // namespace
}  // namespace gamer
