// aux_kernels.hip -- periodic ghost fill, per-group stats and the fixed-order
// reduction of group stats to per-level time steps and conserved totals.
#include "device_math.h"
#include "internal.h"

namespace gamer {
namespace {

// ---- same-level periodic ghost fill --------------------------------------
// One work-group per (group, variable) pair: the pair's padded block of 20^3
// values is one contiguous run of the output, written as 2,000 pieces of four
// values (padded x = 4k - 2 .. 4k + 1 of one padded row), consecutive threads
// on consecutive pieces.  A piece takes two pairs of source values: from the
// left x neighbour (x = 14, 15) and the group's own row for k = 0, from the own
// row and the right x neighbour (x = 0, 1) for k = 4, and from the own row
// otherwise.  The group's position and its periodic neighbours are worked out
// once per work-group; per piece, the padded y and z indices pick the source
// group (own, or the neighbour below or above) and the row within it with
// compares, shifts and masks.  Each thread loads all its pieces before it
// stores any, so that eight pieces' loads are in flight at once.
//
// Work-groups go to the 8 XCDs round-robin by flat index; they are numbered so
// that each XCD takes a contiguous run of (group, variable) pairs, which puts a
// group and its x neighbours (5 pairs apart) under one L2.  The other order
// sent them to different L2s, and the x ghost cells were fetched again from
// memory: reads of 3.8 (256^3) and 4.7 (1024^3) times the field, against 1.5
// and 1.7 with this numbering.
template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
    using type = float4;
};
template <>
struct Vec4<double> {
    using type = double4;
};
template <typename T>
struct Vec2;
template <>
struct Vec2<float> {
    using type = float2;
};
template <>
struct Vec2<double> {
    using type = double2;
};

constexpr int PIECES = NP * NP * 5;  // 4-value pieces in one padded block of one variable

template <typename T>
__global__ __launch_bounds__(256) void pack_block_kernel(const T *__restrict__ state, int gx, int gy,
                                                         int gz, T *__restrict__ padded, int64_t n_blocks) {
    using V = typename Vec4<T>::type;
    using V2 = typename Vec2<T>::type;
    static_assert(NI == 16 && NG == 2, "the masks below assume 16 interior cells and 2 ghost cells");
    unsigned xb = blockIdx.x;
    if ((gridDim.x & 7) == 0) xb = (xb & 7) * (gridDim.x >> 3) + (xb >> 3);
    for (int64_t gv = xb; gv < n_blocks; gv += gridDim.x) {
        const int64_t g = gv / NV;
        const int v = int(gv - g * NV);
        const int bx = int(g % gx);
        const int64_t g1 = g / gx;
        const int by = int(g1 % gy), bz = int(g1 / gy);
        const int ym = by == 0 ? gy - 1 : by - 1, yp = by == gy - 1 ? 0 : by + 1;
        const int zm = bz == 0 ? gz - 1 : bz - 1, zp = bz == gz - 1 ? 0 : bz + 1;
        const int xm = bx == 0 ? gx - 1 : bx - 1, xp = bx == gx - 1 ? 0 : bx + 1;
        const T *src = state + int64_t(v) * (NI * NI * NI);
        V *dst = reinterpret_cast<V *>(padded + gv * (NP * NP * NP));
        constexpr int PER = (PIECES + 255) / 256;
        V2 a[PER], b[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int o = int(threadIdx.x) + 256 * q;
            if (o < PIECES) {
                const int row = o / 5, k = o - row * 5;  // row = kp * 20 + jp
                const int kp = row / NP, jp = row - kp * NP;
                const int yb = jp < NG ? ym : (jp >= NG + NI ? yp : by);
                const int zb = kp < NG ? zm : (kp >= NG + NI ? zp : bz);
                const int yo = (jp - NG) & (NI - 1), zo = (kp - NG) & (NI - 1);
                const int64_t grow = int64_t(gx) * (yb + int64_t(gy) * zb);  // group of x block 0
                const int off = zo * (NI * NI) + yo * NI;
                const int xa = k == 0 ? xm : bx, xc = k == 4 ? xp : bx;  // groups of the two pairs
                const int x0 = k == 0 ? NI - 2 : 4 * k - 2, x1 = k == 4 ? 0 : 4 * k;
                a[q] = *reinterpret_cast<const V2 *>(src + (grow + xa) * GOUT + off + x0);
                b[q] = *reinterpret_cast<const V2 *>(src + (grow + xc) * GOUT + off + x1);
            }
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int o = int(threadIdx.x) + 256 * q;
            if (o < PIECES) dst[o] = V{a[q].x, a[q].y, b[q].x, b[q].y};
        }
    }
}

// ---- per-group stats of interior groups -----------------------------------
// 256 threads per group, thread (i, j) walks its z column in order; the block
// reduction matches the solver epilogue's order, so stats of the same cells
// agree bitwise with the ones the solver writes.
template <typename T>
__global__ __launch_bounds__(256) void group_stats_kernel(const T *__restrict__ groups, int64_t n,
                                                          double gamma, double *__restrict__ stats) {
    __shared__ double red[320 * NSTAT];
    const int t = threadIdx.x;
    const Consts<T> c = make_consts<T>(gamma, 1.5);
    for (int64_t g = blockIdx.x; g < n; g += gridDim.x) {
        const T *src = groups + g * GOUT + t;
        double st[NSTAT] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int k = 0; k < NI; ++k) {
            T u[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                u[v] = src[v * NI * NI * NI + k * NI * NI];
                st[v] += double(u[v]);
            }
            st[5] = max_nan(st[5], double(signal_speed(u[0], u[1], u[2], u[3], u[4], c)));
        }
        // same layout and order as the solver's 320-thread reduction, with
        // the 64 entries of its ghost-cell threads equal to zero
#pragma unroll
        for (int q = 0; q < NSTAT; ++q) {
            red[q * 320 + t] = st[q];
            if (t < 64) red[q * 320 + 256 + t] = 0.0;
        }
        __syncthreads();
        if (t < 64) {
            double acc[NSTAT];
#pragma unroll
            for (int q = 0; q < NSTAT; ++q) {
                double a = red[q * 320 + t];
                for (int s = t + 64; s < 320; s += 64) {
                    const double b = red[q * 320 + s];
                    a = (q == 5) ? max_nan(a, b) : a + b;
                }
                acc[q] = a;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
                for (int q = 0; q < NSTAT; ++q) {
                    const double b = __shfl_down(acc[q], off, 64);
                    acc[q] = (q == 5) ? max_nan(acc[q], b) : acc[q] + b;
                }
            }
            if (t == 0) {
#pragma unroll
                for (int q = 0; q < NSTAT; ++q) stats[g * NSTAT + q] = acc[q];
            }
        }
        __syncthreads();
    }
}

// ---- fixed-order reduction of group stats ----------------------------------
// One work-group of RT threads.  Each thread folds its groups in a fixed order, each
// wave its lanes by a fixed shuffle tree, and one thread per value the waves in order;
// the result does not depend on timing.  Maxima keep NaN, so a level holding a
// non-physical cell gets a NaN time step.
//
// One level (a uniform grid): thread t takes pair r = t mod 4 (stats 2r, 2r + 1) of
// groups t / 4, t / 4 + RT / 4, ..., so that a wave reads 1 KiB of consecutive stats
// per load.  Several levels: a thread takes whole groups t, t + RT, ..., since the
// weights and maxima by level would cost the pairs' four threads each.  Bound by the
// one CU that reads them: 262,144 groups of one level 259 -> 159 us, 24,608 29 -> 15
// (of three levels 31 -> 30); the kernel alone takes 4 us for a few groups, 12 us with
// one thread folding the waves of every value.
constexpr int RT = 1024;
constexpr int RW = RT / 64;
constexpr int RP1 = 8;  // groups per thread whose loads are in flight together, one level
constexpr int RU = 4;   // and several levels
constexpr int RL = 4;   // levels whose maxima are taken in the totals' pass

struct alignas(8) StatPair {  // read as one 16-byte load; the array is 8-byte aligned
    double a, b;
};

template <bool ONE>  // ONE: n_levels is 1 and level is null
__global__ __launch_bounds__(RT) void reduce_kernel(const double *__restrict__ stats, int64_t n,
                                                    const int8_t *__restrict__ level,
                                                    const double *__restrict__ dh_dev, double dh,
                                                    int n_levels, double cfl,
                                                    double *__restrict__ dt_out,
                                                    double *__restrict__ totals_out) {
    // sums of stats 0..7, 0..4 weighted by dh^3 ([5] not used), then the signal-speed
    // maxima of levels 0..RL-1
    constexpr int NR = NSTAT + RL;
    __shared__ double red[NR][RW];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int folded = n_levels <= RL ? n_levels : 0;  // levels whose maxima are taken here
    if constexpr (ONE) {
        const int r = t & 3;
        const StatPair *pairs = reinterpret_cast<const StatPair *>(stats) + r;
        const double h = dh_dev ? dh_dev[0] : dh;
        const double w = r == 3 ? 1.0 : h * h * h;
        double a = 0.0, b = 0.0, m = 0.0;
        int64_t g = t >> 2;
        // RP1 groups at once, summed pair by pair: with RT / 4 threads per value, adding
        // them one by one would put four times as many roundings in a row as a thread
        // per group does, and this puts no more of them for any n
        auto fold = [&](auto whole) {
            StatPair s[RP1];
            bool ok[RP1];
#pragma unroll
            for (int u = 0; u < RP1; ++u) {
                const int64_t gu = g + int64_t(u) * (RT / 4);
                ok[u] = decltype(whole)::value || gu < n;
                s[u] = pairs[(ok[u] ? gu : g) * (NSTAT / 2)];
            }
            __builtin_amdgcn_sched_barrier(0);  // every load issued before the first is used
#pragma unroll
            for (int u = 0; u < RP1; ++u) {
                if (!ok[u]) s[u] = StatPair{0.0, 0.0};
                m = max_nan(m, s[u].b);  // stat 5 where r is 2
            }
#pragma unroll
            for (int d = 1; d < RP1; d *= 2) {
#pragma unroll
                for (int u = 0; u < RP1; u += 2 * d) {
                    s[u].a += s[u + d].a;
                    s[u].b += s[u + d].b;
                }
            }
            a += w * s[0].a;
            b += w * s[0].b;
        };
        for (; g + int64_t(RT / 4) * (RP1 - 1) < n; g += int64_t(RT / 4) * RP1) fold(std::true_type());
        if (g < n) fold(std::false_type());
#pragma unroll
        for (int off = 32; off >= 4; off >>= 1) {
            a += __shfl_down(a, off, 64);
            b += __shfl_down(b, off, 64);
            m = max_nan(m, __shfl_down(m, off, 64));
        }
        if (lane < 4) {
            red[2 * r][wave] = a;
            red[2 * r + 1][wave] = b;
            if (r == 2) red[NSTAT][wave] = m;
        }
    } else {
        double x[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) x[q] = 0.0;
        const int64_t end = totals_out || folded > 0 ? n : 0;  // nothing to take in this pass
        for (int64_t g0 = t; g0 < end; g0 += int64_t(RT) * RU) {
            double s[RU][NSTAT], w[RU];
            int lv[RU];
            bool ok[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const int64_t g1 = g0 + int64_t(u) * RT;
                ok[u] = g1 < n;
                const int64_t g = ok[u] ? g1 : g0;  // a valid group to read; its values are not used
                lv[u] = level ? int(level[g]) : 0;
                double h = dh;
                if (dh_dev) {
                    // a level out of range is never used as an index; it makes the totals NaN
                    h = (lv[u] >= 0 && lv[u] < n_levels) ? dh_dev[lv[u]] : __builtin_nan("");
                }
                w[u] = h * h * h;
                const double *st = stats + g * NSTAT;
#pragma unroll
                for (int q = 0; q < NSTAT; ++q) s[u][q] = st[q];
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (!ok[u]) continue;
#pragma unroll
                for (int q = 0; q < NSTAT; ++q)
                    if (q != 5) x[q] += q < 5 ? w[u] * s[u][q] : s[u][q];
#pragma unroll
                for (int L = 0; L < RL; ++L)
                    if (L < folded && lv[u] == L) x[NSTAT + L] = max_nan(x[NSTAT + L], s[u][5]);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const double y = __shfl_down(x[q], off, 64);
                x[q] = q >= NSTAT ? max_nan(x[q], y) : x[q] + y;
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < NR; ++q) red[q][wave] = x[q];
        }
    }
    __syncthreads();
    auto write_dt = [&](int L, double top) {
        const double hL = dh_dev ? dh_dev[L] : dh;
        // NaN when a group of the level has a non-physical cell
        dt_out[L] = top > 0.0 ? cfl * hL / top : (top != top ? top : INFINITY);
    };
    if (t < NSTAT + folded) {
        double x = red[t][0];
        for (int w = 1; w < RW; ++w) x = t < NSTAT ? x + red[t][w] : max_nan(x, red[t][w]);
        if (t < NSTAT) {
            if (totals_out && t != 5) totals_out[t < 5 ? t : t - 1] = x;
        } else if (dt_out) {
            write_dt(t - NSTAT, x);
        }
    }
    // more levels: one pass over the stats for the maximum of each
    if (dt_out && n_levels > RL) {
        for (int L = 0; L < n_levels; ++L) {
            double x = 0.0;
#pragma unroll 4
            for (int64_t g = t; g < n; g += RT) {
                const double sp = stats[g * NSTAT + 5];
                if ((level ? int(level[g]) : 0) == L) x = max_nan(x, sp);
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) x = max_nan(x, __shfl_down(x, off, 64));
            __syncthreads();  // the last values read from red[0]
            if (lane == 0) red[0][wave] = x;
            __syncthreads();
            if (t == 0) {
                for (int w = 1; w < RW; ++w) x = max_nan(x, red[0][w]);
                write_dt(L, x);
            }
        }
    }
}

}  // namespace

template <typename T>
hipError_t launch_pack_periodic(const T *state, int gx, int gy, int gz, T *padded, hipStream_t s) {
    const int64_t n_blocks = int64_t(gx) * gy * gz * NV;  // (group, variable) pairs
    if (n_blocks == 0) return hipSuccess;
    const int64_t cap = int64_t(256) * 2048;  // a multiple of 8, as the XCD numbering wants
    hipLaunchKernelGGL(pack_block_kernel<T>, dim3(unsigned(n_blocks < cap ? n_blocks : cap)), dim3(256), 0, s,
                       state, gx, gy, gz, padded, n_blocks);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_group_stats(const T *groups, int64_t n, double gamma, double *stats,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t cap = int64_t(1) << 30;
    hipLaunchKernelGGL(group_stats_kernel<T>, dim3(unsigned(n < cap ? n : cap)), dim3(256), 0, s,
                       groups, n, gamma, stats);
    return hipGetLastError();
}

hipError_t launch_reduce(const double *stats, int64_t n, const int8_t *level, const double *dh_dev,
                         double dh, int n_levels, double cfl, double *dt_out, double *totals_out,
                         hipStream_t s) {
    const auto kernel = n_levels == 1 && !level ? reduce_kernel<true> : reduce_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(RT), 0, s, stats, n, level, dh_dev, dh, n_levels, cfl, dt_out, totals_out);
    return hipGetLastError();
}

template hipError_t launch_pack_periodic<float>(const float *, int, int, int, float *, hipStream_t);
template hipError_t launch_pack_periodic<double>(const double *, int, int, int, double *,
                                                 hipStream_t);
template hipError_t launch_group_stats<float>(const float *, int64_t, double, double *,
                                              hipStream_t);
template hipError_t launch_group_stats<double>(const double *, int64_t, double, double *,
                                               hipStream_t);

}  // namespace gamer
