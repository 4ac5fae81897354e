// device_math.h -- arithmetic and addressing helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace gamer {

template <typename T>
struct Consts {
    T g, gm1, igm1, theta, half;
    T ht, k1;  // theta / 2 and 1 / (2 theta)
    T gq;  // gamma (gamma - 1) / 2: (rho c)^2 = gq (2 rho E - |m|^2)
};

// Reciprocal and square root.  float: the hardware instructions (about 1 ulp,
// well inside the FP32 path's tolerance).  double: the hardware estimate (within
// 5.2e-8) refined by one cubic step, without the range scaling of the IEEE
// expansions (operands here are normal numbers).  Against 64-bit significands
// over 4 M values in 2^+-30: reciprocal worst 1.00 and rms 0.44, reciprocal root
// 1.24 and 0.48, root 1.00 and 0.42 in units of 2^-53, the same as two Newton
// steps give with one, two and four instructions more.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double rcp(double x) {
    // r (1 + e + e^2) with e = 1 - x r, whose error is e^3
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq(double x) {
    // y (1 + e/2 + 3 e^2 / 8) with e = 1 - x y^2
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double sqrt_(double x) {
    // two Newton steps g <- g + (x - g^2) h on g = x y, with h = y / 2 of the
    // estimate throughout: its own error only scales the last correction
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-g, h, 0.5), g);
    g = fma(fma(-g, g, x), h, g);
    return x > 0.0 ? g : (x == 0.0 ? 0.0 : __builtin_nan(""));
}

// |u| + |v| + |w| + 3 c_s of a conserved state in the working precision, or NaN
// when the state is not physical (rho <= 0 or p <= 0) or not finite: such a
// state has no sound speed, and the NaN carries through the maxima below to
// the time step instead of being dropped.  The solver epilogue and the
// stand-alone stats kernel both use this function, whose multiply-adds contract
// within one expression only, so their per-group maxima agree bitwise.
template <typename T>
__device__ __forceinline__ T signal_speed(T r, T mx, T my, T mz, T e, const Consts<T> &c) {
#pragma clang fp contract(on)
    const T ir = rcp(r);
    const T u = mx * ir, v = my * ir, w = mz * ir;
    const T p = c.gm1 * (e - c.half * (mx * u + my * v + mz * w));
    const T cs = sqrt_(c.g * p * ir);
    const T s = fabs(u) + fabs(v) + fabs(w) + T(3) * cs;
    return (r > T(0) && p > T(0) && isfinite(s)) ? s : T(__builtin_nan(""));
}

// Maximum that keeps a NaN of either operand (fmax drops it).
__device__ __forceinline__ double max_nan(double a, double b) { return (a > b || a != a) ? a : b; }

template <typename T>
__device__ __forceinline__ Consts<T> make_consts(double gamma, double theta) {
    return Consts<T>{T(gamma), T(gamma - 1.0), T(1.0 / (gamma - 1.0)), T(theta), T(0.5), T(0.5 * theta), T(0.5 / theta),
                     T(0.5 * gamma * (gamma - 1.0))};
}

// An index taken afresh at this place: what is derived from it (addresses of
// rarely executed accesses above all) is computed here and not kept in registers
// across the sweep, where every register is in use.
template <typename T>
__device__ __forceinline__ T fresh(T x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The value at byte offset `off` of a wave-uniform base pointer.  The base is
// pinned to scalar registers, so that each access takes it as it is: with a 32-bit
// lane offset (itself taken afresh in the same place) the access needs no vector
// instruction for its address, with a 64-bit one a single add.  Left alone, the
// compiler keeps one vector pointer for the five variables and adds their strides
// to it, two instructions and a wait state per access: 45 of the float sweep's
// 1,000 vector instructions per wave and plane.
template <typename P, typename Off>
__device__ __forceinline__ auto &at(P *base, Off off) {
    using G = __attribute__((address_space(1))) P;
    using C = __attribute__((address_space(1))) std::conditional_t<std::is_const_v<P>, const char, char>;
    C *b = (C *)base;  // global memory, which the pinning would hide
    asm volatile("" : "+s"(b));
    return *(G *)(b + off);
}

}  // namespace gamer
