// rtvd.hip -- the relaxing TVD scheme (the solver the paper compares
// MUSCL-Hancock with): three dimensionally split sweeps per step, each advancing
// every pencil along the sweep direction by the relaxing scheme's half step and
// full step.  The z sweep is a launch of its own; x and y take one launch together
// on large inputs and one each on small ones (rtvd_xy, together()).
//
// Padded groups: the block shrinks by three cells per side along the sweep
// direction only, so the three sweeps go 22^3 -> 16 x 22 x 22 -> 16 x 16 x 22 ->
// 16^3 (x, y, z order) through two workspace arrays.
//
// A periodic grid: every sweep takes whole groups (16^3) to whole groups, with the
// three ghost cells at a pencil's ends read from the neighbouring groups, since a
// neighbour's swept cells are the values that sweeping them again as ghost cells
// gives.  No cell is swept twice: the padded form sweeps 22^2 / 16^2 and 22 / 16
// times the pencils in its first two sweeps, and writes and reads as many more
// cells between them (256^3 step: 839 -> 393 us in float, 1,592 -> 724 in double).
//
// x sweeps hold one cell per lane and take their neighbours by lane shifts; y and z
// sweeps march a thread along each pencil, with consecutive threads on
// consecutive x.  Both run the same functions on the same values, whose rounding
// is fixed by the source (multiply-adds contract within one expression only), so
// that the two kinds of input give the same bits and a uniform state stays so.
#include "device_math.h"
#include "internal.h"

namespace gamer {
namespace {

constexpr int RP = 22;      // padded cells per axis (three ghost cells per side)
constexpr int RG = 3;

template <typename T>
struct SweepArgs {
    const T *in;      // blocks [n][5][ez][ey][ex], or a periodic grid of groups [n][5][16][16][16]
    int gx, gy, gz;   // periodic grid: groups per axis
    int ex, ey, ez;   // padded input: block extents
    int tiles, width; // periodic x sweep: tiles per row of cells, and output cells of each
    int seg;          // periodic y and z sweeps: cells that one thread marches through
    T *out;           // [n][5][..] with extent e[d] - 6 along d, or groups
    const int8_t *level;
    const double *dt_dev, *dh_dev;
    int n_levels;     // a level byte outside [0, n_levels) gives the group NaN dt and dh
    double gamma;
    int64_t n_groups;
};

template <typename T>
struct Step {
    T g, gm1;
    T hdt2;        // half of dt/(2 dx): the first-order fluxes are kept doubled
    double hdtdx;  // dt/(2 dx): the second-order fluxes are too
};
template <typename T>
__device__ __forceinline__ Step<T> make_step(const SweepArgs<T> &P, int64_t g) {
    double dt, dh;
    level_dt(P.level, g, P.n_levels, P.dt_dev, P.dh_dev, dt, dh);
    const double dtdx = dt / dh;
    return Step<T>{T(P.gamma), T(P.gamma - 1.0), T(0.25 * dtdx), 0.5 * dtdx};
}

// The right- and left-moving fluxes r = c u + F_D(u) and l = c u - F_D(u), with the
// freezing speed c = |v_D| + c_s: ten multiply-adds on the five fluxes.
template <int D, typename T>
__device__ __forceinline__ void relax(const T u[NV], const Step<T> &c, T r[NV], T l[NV]) {
#pragma clang fp contract(on)
    const T ir = rcp(u[0]);
    const T vx = u[1] * ir, vy = u[2] * ir, vz = u[3] * ir;
    const T vd = D == 0 ? vx : (D == 1 ? vy : vz);
    const T p = c.gm1 * (u[4] - T(0.5) * (u[1] * vx + u[2] * vy + u[3] * vz));
    const T s = fabs(vd) + sqrt_(c.g * p * ir);
    T F[NV];
#pragma unroll
    for (int v = 1; v < 4; ++v) F[v] = v == 1 + D ? u[v] * vd + p : u[v] * vd;
    F[0] = u[1 + D];
    F[4] = (u[4] + p) * vd;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        r[v] = s * u[v] + F[v];
        l[v] = s * u[v] - F[v];
    }
}

// q + VL(x/2, y/2) with van Leer's limiter of the half differences, VL(x/2, y/2) =
// 2 (x/2)(y/2) / (x/2 + y/2) if their product is positive, else 0, written as
// x y / (x + y).
template <typename T>
__device__ __forceinline__ T extrapolate(T q, T x, T y) {
#pragma clang fp contract(on)
    const T xy = x * y;
    return xy > T(0) ? q + xy * rcp(x + y) : q;
}

// the half-step state from twice the first-order fluxes above and below the cell
template <typename T>
__device__ __forceinline__ T half_state(T u, T Fp, T Fm, const Step<T> &c) {
#pragma clang fp contract(on)
    return u - c.hdt2 * (Fp - Fm);
}

// the new value from twice the second-order fluxes above and below the cell
template <typename T>
__device__ __forceinline__ T full_state(T u, T Fp, T Fm, const Step<T> &c) {
#pragma clang fp contract(on)
    return T(double(u) - c.hdtdx * (double(Fp) - double(Fm)));
}

// ---- x sweeps: one cell per lane -----------------------------------------------

// The value of the lane below / above (0 at the wave's ends, which hold no output).
template <int CTRL>
__device__ __forceinline__ int lane_shift(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float x) {
    return __int_as_float(lane_shift<CTRL>(__float_as_int(x)));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
    return __hiloint2double(lane_shift<CTRL>(__double2hiint(x)), lane_shift<CTRL>(__double2loint(x)));
}
template <typename T>
__device__ __forceinline__ T below(T x) { return lane_shift<0x138>(x); }  // wave_shr:1
template <typename T>
__device__ __forceinline__ T above(T x) { return lane_shift<0x130>(x); }  // wave_shl:1

// The sweep of a run of cells along x held by consecutive lanes: every lane's new
// value, meaningful where three cells of the run lie on either side.
template <typename T>
__device__ __forceinline__ void sweep_lanes(const T u[NV], const Step<T> &c, T o[NV]) {
    T fr[NV], fl[NV], h[NV], r[NV], l[NV];
    relax<0>(u, c, fr, fl);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const T Fp = fr[v] - above(fl[v]);
        h[v] = half_state(u[v], Fp, below(Fp), c);
    }
    relax<0>(h, c, r, l);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const T dr = r[v] - below(r[v]), dl = below(l[v]) - l[v];
        const T R = extrapolate(r[v], dr, above(dr)), L = extrapolate(l[v], dl, above(dl));
        const T F = R - above(L);
        o[v] = full_state(u[v], F, below(F), c);
    }
}

// The same with two neighbouring cells a, b per lane, which halves the lane shifts.
template <typename T>
__device__ __forceinline__ void sweep_lanes2(const T ua[NV], const T ub[NV], const Step<T> &c, T oa[NV], T ob[NV]) {
    T fra[NV], fla[NV], frb[NV], flb[NV], ha[NV], hb[NV], ra[NV], la[NV], rb[NV], lb[NV];
    relax<0>(ua, c, fra, fla);
    relax<0>(ub, c, frb, flb);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const T Fa = fra[v] - flb[v], Fb = frb[v] - above(fla[v]);
        ha[v] = half_state(ua[v], Fa, below(Fb), c);
        hb[v] = half_state(ub[v], Fb, Fa, c);
    }
    relax<0>(ha, c, ra, la);
    relax<0>(hb, c, rb, lb);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const T dra = ra[v] - below(rb[v]), drb = rb[v] - ra[v];
        const T dla = below(lb[v]) - la[v], dlb = la[v] - lb[v];
        const T Ra = extrapolate(ra[v], dra, drb), Rb = extrapolate(rb[v], drb, above(dra));
        const T La = extrapolate(la[v], dla, dlb), Lb = extrapolate(lb[v], dlb, above(dla));
        const T Fa = Ra - Lb, Fb = Rb - above(La);
        oa[v] = full_state(ua[v], Fa, below(Fb), c);
        ob[v] = full_state(ub[v], Fb, Fa, c);
    }
}

// x pencils of padded blocks of E x E pencils of 22 cells, two cells per lane: a
// wave takes five pencils (lanes 0..54).  Bound by vector issue, so what counts is
// that 110 of 128 places hold cells (a cell per lane: two pencils, 44 of 64) and
// that nothing goes through LDS (a lane per position with a barrier per phase took
// 2.4 times the instructions).  Step of 1,000 padded groups against that form: float
// 197 -> 183 us, double 394 -> 325; with one cell per lane 205 and 368.
constexpr int XROWS = 5, XLANES = RP / 2;
template <int E>
constexpr int x_waves() { return (E * E + XROWS - 1) / XROWS; }
template <typename T, int E>
__global__ __launch_bounds__(256) void rtvd_x_padded(SweepArgs<T> P) {
    constexpr int VIN = RP * E * E, VOUT = NI * E * E, WAVES = x_waves<E>();
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
    const int64_t w = (int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * 4 + wave;
    const int64_t g = w / WAVES;
    if (g >= P.n_groups) return;
    const int q = lane / XLANES, i = lane - q * XLANES;  // pencil of the wave, pair of cells
    const int row = int(w - g * WAVES) * XROWS + q;
    const bool live = q < XROWS && row < E * E;
    const Step<T> c = make_step(P, g);
    const T *src = P.in + g * (NV * VIN);
    const int at = live ? row * RP + 2 * i : 0;
    T ua[NV], ub[NV], oa[NV], ob[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        ua[v] = src[v * VIN + at];
        ub[v] = src[v * VIN + at + 1];
    }
    sweep_lanes2(ua, ub, c, oa, ob);
    // cells 2 i and 2 i + 1: output positions 2 i - 3 and 2 i - 2
    T *dst = P.out + g * (NV * VOUT);
    const int to = row * NI + 2 * i - RG;
    if (live && i >= 2 && i <= 9) {
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[v * VOUT + to] = oa[v];
    }
    if (live && i >= 1 && i <= 8) {
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[v * VOUT + to + 1] = ob[v];
    }
}

// Work-groups are dispatched to the 8 XCDs round-robin, each with its own L2;
// numbered so that each XCD takes a contiguous run, neighbours share an L2.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned n) {
    const unsigned x = b % 8, q = n / 8, r = n % 8;
    return x * q + (x < r ? x : r) + b / 8;
}

// x pencils of a periodic grid: a row of cells across all groups of the grid is cut
// into tiles of `width` <= 58 output cells, one wave each with the three cells on
// either side.  A work-group's waves take four consecutive rows, which share the
// cache lines of a group's 16-cell rows.
template <typename T>
__global__ __launch_bounds__(256) void rtvd_x_periodic(SweepArgs<T> P) {
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
    // blocks: rows of a group row fastest (64 blocks of four), then tiles, then (by, bz)
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    const unsigned rest = b / 64, tile = rest % unsigned(P.tiles), col = rest / unsigned(P.tiles);
    const int row = int(b % 64) * 4 + wave;  // z * 16 + y within the groups
    const int NX = P.gx * NI, x0 = int(tile) * P.width;
    const int width = NX - x0 < P.width ? NX - x0 : P.width;
    const Step<T> c = make_step(P, 0);
    int x = x0 + lane - RG;
    if (x < 0) x += NX;
    while (x >= NX) x -= NX;
    const int64_t at = int64_t(x / NI) * GOUT + row * NI + x % NI;
    const T *src = P.in + int64_t(col) * P.gx * GOUT;
    T u[NV], o[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = src[v * (NI * NI * NI) + at];
    sweep_lanes(u, c, o);
    if (lane >= RG && lane < RG + width) {
        T *dst = P.out + int64_t(col) * P.gx * GOUT;
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[v * (NI * NI * NI) + at] = o[v];
    }
}

// ---- y and z sweeps: one thread per pencil -------------------------------------

// A pencil's state between two cells: everything is formed once, in registers.
// After cell n was pushed: the input of cells n, n-1, n-2; twice the first-order
// flux above cell n-1; the moving fluxes of the half-step state of cell n-1 with
// their differences from cell n-2; the extrapolated right-moving flux of cell n-2
// and twice the second-order flux above cell n-3.
template <typename T, int D>
struct March {
    T u0[NV], u1[NV], u2[NV], fr[NV], Fp[NV], r[NV], l[NV], dr[NV], dl[NV], R[NV], F[NV];

    // Push cell n of the pencil (n capped at 6: the count of cells before it); from
    // n = 6 on, o is the new value of cell n - 3.
    template <int N>
    __device__ __forceinline__ void push(const T u[NV], const Step<T> &c, T o[NV]) {
        T a[NV], b[NV], h[NV], rn[NV], ln[NV];
        relax<D>(u, c, a, b);
        if constexpr (N >= 1) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const T Fn = fr[v] - b[v];
                if constexpr (N >= 2) h[v] = half_state(u0[v], Fn, Fp[v], c);
                Fp[v] = Fn;
            }
        }
        if constexpr (N >= 2) {
            relax<D>(h, c, rn, ln);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                if constexpr (N >= 3) {
                    const T drn = rn[v] - r[v], dln = l[v] - ln[v];
                    if constexpr (N >= 4) {
                        const T Rn = extrapolate(r[v], dr[v], drn);
                        if constexpr (N >= 5) {
                            const T Fn = R[v] - extrapolate(l[v], dl[v], dln);
                            if constexpr (N >= 6) o[v] = full_state(u2[v], Fn, F[v], c);
                            F[v] = Fn;
                        }
                        R[v] = Rn;
                    }
                    dr[v] = drn;
                    dl[v] = dln;
                }
                r[v] = rn[v];
                l[v] = ln[v];
            }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            u2[v] = u1[v];
            u1[v] = u0[v];
            u0[v] = u[v];
            fr[v] = a[v];
        }
    }
};

constexpr int PREFETCH = 2;  // cells between a load's issue and its use (segments are whole multiples)

// Pencils of padded blocks (22 cells along D), consecutive threads on consecutive
// pencils along the fastest transverse axis.
template <typename T, int D>
__global__ __launch_bounds__(256) void rtvd_march_padded(SweepArgs<T> P) {
    static_assert(D == 1 || D == 2, "y and z sweeps");
    constexpr int A = 0, B = D == 2 ? 1 : 2;  // transverse axes, A fastest
    const int e[3] = {P.ex, P.ey, P.ez};
    int eo[3] = {P.ex, P.ey, P.ez};
    eo[D] -= 2 * RG;
    const int ea = e[A], npen = e[A] * e[B];
    // 32-bit index arithmetic: the host caps n_groups * pencils below 2^31
    const int tid = int(blockIdx.x) * 256 + int(threadIdx.x);
    if (int64_t(tid) >= P.n_groups * npen) return;
    const int gi = tid / npen;
    const int p = tid - gi * npen;
    const int64_t g = gi;
    const int ia = p % ea, ib = p / ea;
    const int64_t vin = int64_t(e[0]) * e[1] * e[2], vout = int64_t(eo[0]) * eo[1] * eo[2];
    const int si[3] = {1, e[0], e[0] * e[1]}, so[3] = {1, eo[0], eo[0] * eo[1]};
    const T *src = P.in + g * NV * vin + int64_t(ia) * si[A] + int64_t(ib) * si[B];
    T *dst = P.out + g * NV * vout + int64_t(ia) * so[A] + int64_t(ib) * so[B];
    const Step<T> c = make_step(P, g);

    March<T, D> m;
    T u[RP][NV], o[NV];
    auto load = [&](int s) {
#pragma unroll
        for (int v = 0; v < NV; ++v) u[s][v] = src[v * vin + s * si[D]];
    };
#pragma unroll
    for (int s = 0; s < PREFETCH; ++s) load(s);
#pragma unroll
    for (int s = 0; s < RP; ++s) {
        if (s + PREFETCH < RP) load(s + PREFETCH);
        if (s == 0) m.template push<0>(u[s], c, o);
        else if (s == 1) m.template push<1>(u[s], c, o);
        else if (s == 2) m.template push<2>(u[s], c, o);
        else if (s == 3) m.template push<3>(u[s], c, o);
        else if (s == 4) m.template push<4>(u[s], c, o);
        else if (s == 5) m.template push<5>(u[s], c, o);
        else {
            m.template push<6>(u[s], c, o);
#pragma unroll
            for (int v = 0; v < NV; ++v) dst[v * vout + int64_t(s - 2 * RG) * so[D]] = o[v];
        }
    }
}

// Pencils of a periodic grid: one work-group per (group column along D, segment of
// P.seg cells), thread t on the pencil of its 16 x 16 transverse cells (x fastest).
// A thread marches through its segment without a restart, so only the six cells
// around a segment's ends are read and relaxed twice.
template <typename T, int D>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
void rtvd_march_periodic(SweepArgs<T> P) {
    static_assert(D == 1 || D == 2, "y and z sweeps");
    constexpr int STR = D == 1 ? NI : NI * NI;  // stride of a pencil within a group
    constexpr int VS = NI * NI * NI;
    const int n = (D == 1 ? P.gy : P.gz) * NI;  // cells along the pencil
    const unsigned nseg = unsigned((n + P.seg - 1) / P.seg);
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    const unsigned col = b / nseg;
    const int y0 = int(b % nseg) * P.seg, end = n - y0 < P.seg ? n : y0 + P.seg;
    // first group of the column, and the group stride along the pencil
    const unsigned cx = col % unsigned(P.gx), co = col / unsigned(P.gx);
    const int64_t g0 = D == 1 ? int64_t(cx) + int64_t(P.gx) * P.gy * co : int64_t(cx) + int64_t(P.gx) * co;
    const int64_t gs = D == 1 ? P.gx : int64_t(P.gx) * P.gy;
    const int t = threadIdx.x;
    const unsigned off = (D == 1 ? unsigned((t >> 4) * (NI * NI) + (t & 15)) : unsigned(t)) * unsigned(sizeof(T));
    auto cell = [&](int y) -> int64_t {  // values before cell y (-3 .. n + 4, wrapped) of the column's pencils
        y = y < 0 ? y + n : (y >= n ? y - n : y);
        return (g0 + gs * (y >> 4)) * GOUT + (y & 15) * STR;
    };
    auto load = [&](T u[NV], int y) {
        const T *src = P.in + cell(y);
        const unsigned ob = unsigned(fresh(int(off)));
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = at(src + v * VS, ob);
    };
    const Step<T> c = make_step(P, 0);
    March<T, D> m;
    T pre[PREFETCH][NV], o[NV];
    {
        T u[2 * RG][NV];
#pragma unroll
        for (int s = 0; s < 2 * RG; ++s) load(u[s], y0 + s - RG);
#pragma unroll
        for (int s = 0; s < PREFETCH; ++s) load(pre[s], y0 + RG + s);
        m.template push<0>(u[0], c, o);
        m.template push<1>(u[1], c, o);
        m.template push<2>(u[2], c, o);
        m.template push<3>(u[3], c, o);
        m.template push<4>(u[4], c, o);
        m.template push<5>(u[5], c, o);
    }
    for (int y = y0; y < end; y += PREFETCH) {
#pragma unroll
        for (int q = 0; q < PREFETCH; ++q) {  // push cell y + q + 3, update cell y + q
            T u[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = pre[q][v];
            load(pre[q], y + q + RG + PREFETCH);
            m.template push<6>(u, c, o);
            T *dst = P.out + cell(y + q);
            const unsigned ob = unsigned(fresh(int(off)));
#pragma unroll
            for (int v = 0; v < NV; ++v) at(dst + v * VS, ob) = o[v];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// ---- x and y sweeps in one launch -------------------------------------------------

// Lanes hold a run of cells along x and march along y.  ORDER 0 (x, then y) pushes
// each row it has swept along x into the march; ORDER 1 (y, then x) sweeps along x
// each row that the march gives.  Nothing goes to memory between the two.
//   periodic: a wave takes 64 cells of a row of the grid, `width` of them output, and
//     marches through P.seg cells; a work-group's waves take four z planes.
//   padded: a wave takes the 22-cell rows of two z planes of a group (lanes 0..21 and
//     22..43) and marches over the 22 rows.
// A pass over the grid costs 160 us at 256^3 in float (671 MB), and the two sweeps'
// arithmetic overlaps what is left: x and y took 409 us as two launches and 262 us
// as one, the step 545 and 392 us (double 853 and 722).
template <typename T, int ORDER, bool PERIODIC>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
void rtvd_xy(SweepArgs<T> P) {
    // z planes and cells per variable of a padded block, before and after
    constexpr int EZ = ORDER == 0 ? RP : NI;
    constexpr int VIN = PERIODIC ? NI * NI * NI : RP * RP * EZ, VOUT = PERIODIC ? NI * NI * NI : NI * NI * EZ;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
    int64_t g = 0;            // the padded group
    const T *in = P.in;
    T *out = P.out;
    unsigned off, to;         // byte offsets of this lane's cell within a row, input and output
    bool live;                // whether the lane holds an output cell
    int y0, end;              // output rows of the wave
    int64_t plane = 0;        // periodic: values before the wave's z plane in group row 0
    const int NY = P.gy * NI;
    if constexpr (PERIODIC) {
        const unsigned nseg = unsigned((NY + P.seg - 1) / P.seg);
        const unsigned b = xcd_block(blockIdx.x, gridDim.x), rest = b / nseg;
        const unsigned tile = rest % unsigned(P.tiles), z = rest / unsigned(P.tiles) * 4 + unsigned(wave);
        const int NX = P.gx * NI, x0 = int(tile) * P.width;
        const int width = NX - x0 < P.width ? NX - x0 : P.width;
        int x = x0 + lane - RG;
        if (x < 0) x += NX;
        while (x >= NX) x -= NX;
        off = to = (unsigned(x / NI) * unsigned(GOUT) + unsigned(x % NI)) * unsigned(sizeof(T));
        live = lane >= RG && lane < RG + width;
        plane = int64_t(z / NI) * P.gy * P.gx * GOUT + int64_t(z % NI) * (NI * NI);
        y0 = int(b % nseg) * P.seg;
        end = NY - y0 < P.seg ? NY : y0 + P.seg;
    } else {
        const int64_t w = (int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * 4 + wave;
        g = w / (EZ / 2);
        if (g >= P.n_groups) return;
        const int z = 2 * int(w - g * (EZ / 2));
        const bool two = lane >= RP, mine = lane < 2 * RP;
        const int l = mine ? (two ? lane - RP : lane) : 0;
        const int zl = z + (mine && two);
        in += g * (NV * VIN);
        out += g * (NV * VOUT);
        live = mine && l >= RG && l < RG + NI;
        off = unsigned(zl * (RP * RP) + l) * unsigned(sizeof(T));
        to = unsigned(zl * (NI * NI) + (live ? l - RG : 0)) * unsigned(sizeof(T));
        y0 = 0;
        end = NI;
    }
    const Step<T> c = make_step(P, g);
    // values before input row y (-3 .. the row after next behind the end) and output row y
    auto row = [&](int y) -> int64_t {
        if constexpr (PERIODIC) {
            y = y < 0 ? y + NY : (y >= NY ? y - NY : y);
            return plane + int64_t(y >> 4) * P.gx * GOUT + (y & 15) * NI;
        } else {
            y = y + RG < RP ? y + RG : RP - 1;  // the prefetch behind the last row reads it again
            return y * RP;
        }
    };
    March<T, 1> m;
    T pre[PREFETCH][NV], o[NV];
    auto load = [&](T u[NV], int y) {
        const T *src = in + row(y);
        const unsigned ob = unsigned(fresh(int(off)));
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = at(src + v * VIN, ob);
    };
    auto swept = [&](const T u[NV], T w[NV]) {
        if constexpr (ORDER == 0) {
            sweep_lanes(u, c, w);
        } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) w[v] = u[v];
        }
    };
    {
        T u[2 * RG][NV], w[NV];
#pragma unroll
        for (int s = 0; s < 2 * RG; ++s) load(u[s], y0 + s - RG);
#pragma unroll
        for (int s = 0; s < PREFETCH; ++s) load(pre[s], y0 + RG + s);
        swept(u[0], w);
        m.template push<0>(w, c, o);
        swept(u[1], w);
        m.template push<1>(w, c, o);
        swept(u[2], w);
        m.template push<2>(w, c, o);
        swept(u[3], w);
        m.template push<3>(w, c, o);
        swept(u[4], w);
        m.template push<4>(w, c, o);
        swept(u[5], w);
        m.template push<5>(w, c, o);
    }
    static_assert(NI % PREFETCH == 0, "whole rounds of the prefetch ring");
    for (int y = y0; y < end; y += PREFETCH) {
#pragma unroll
        for (int q = 0; q < PREFETCH; ++q) {  // push row y + q + 3, update row y + q
            T u[NV], w[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = pre[q][v];
            load(pre[q], y + q + RG + PREFETCH);
            swept(u, w);
            m.template push<6>(w, c, o);
            if constexpr (ORDER == 1) {
#pragma unroll
                for (int v = 0; v < NV; ++v) w[v] = o[v];
                sweep_lanes(w, c, o);
            }
            if (live) {
                T *dst = out + (PERIODIC ? row(y + q) : int64_t(y + q) * NI);
                const unsigned ob = unsigned(fresh(int(to)));
#pragma unroll
                for (int v = 0; v < NV; ++v) at(dst + v * VOUT, ob) = o[v];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

constexpr int XWIDTH = 64 - 2 * RG;  // most output cells of a wave's run

// Cells that a thread of the periodic y and z sweeps marches through: longer
// segments read and relax fewer cells twice (six per segment), shorter ones fill the
// chip, which holds 1,024 float work-groups (four per CU), and on grids too small
// for that shorten the chain of cells that one thread takes in series.  Measured per
// step: 256^3 float 430, 402, 393 and 424 us with segments of 16, 32, 64 and 128
// cells (x and y together: 1,280 work-groups at 64), double 843, 772, 732 and 773;
// 128^3 float 62, 63 and 88 us with 16, 32 and 64; 32^3 double 37, 25, 18 and 16 us
// with 16, 8, 4 and 2 (12 to 96 work-groups), but 64^3 28 us with 4 and 30 with 2
// (256 and 512).
int march_segment(int64_t columns, int gd) {
    const int n = gd * NI;
    auto blocks = [&](int seg) { return columns * ((n + seg - 1) / seg); };
    int seg = NI;
    while (2 * seg <= 8 * NI && 2 * seg <= n && blocks(2 * seg) >= 1024) seg *= 2;
    while (seg > PREFETCH && blocks(seg / 2) <= 256) seg /= 2;
    return seg;
}

// Whether the x and y sweeps go together.  A periodic grid: where a thread still has
// two groups to march through (at 128^3, where it has one, two launches take 62 us
// and one 64; at 64^3 29 and 33).  Padded groups, x then y: float batches of 1,024
// groups and more (1,000 groups 179 against 183 us, 2,744 469 against 488, but 512
// 97 against 86), no double ones (the march leaves two waves per SIMD and a wave
// fills 44 of its lanes: 1,000 groups 351 against 325).  Padded groups, y then x,
// where the ghost rows of the march are not swept along x: from 128 groups on, eight
// waves each (1,000 groups float 161 against 213 us, double 328 against 367, 512
// groups double 161 against 194; 27 groups double 40 against 36).
template <typename T>
bool together(bool periodic, int order, int seg, int64_t n) {
    if (periodic) return seg > NI;
    return n >= (order == 1 ? 128 : 1024) && (order == 1 || sizeof(T) == 4);
}

}  // namespace

template <typename T>
size_t rtvd_workspace_elems(int64_t n_groups) {
    // two intermediate blocks: 16 x 22 x 22 and 16 x 16 x 22 cells per group (the
    // periodic sweeps need 16^3 of each)
    return size_t(n_groups) * NV * (NI * RP * RP + NI * NI * RP);
}

template <typename T>
hipError_t launch_rtvd(const T *in, int gx, int gy, int gz, int64_t n, const int8_t *level,
                       int n_levels, const double *dt_dev, const double *dh_dev, double gamma,
                       int order, T *work, T *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const bool periodic = gx > 0;
    const int dirs[2][3] = {{0, 1, 2}, {2, 1, 0}};
    T *b1 = work;
    T *b2 = work + size_t(n) * NV * NI * RP * RP;
    int e[3] = {RP, RP, RP};
    const T *src = in;
    for (int k = 0; k < 3; ++k) {
        const int d = dirs[order][k];
        SweepArgs<T> P = {};
        P.in = src;
        P.gx = gx;
        P.gy = gy;
        P.gz = gz;
        P.ex = e[0];
        P.ey = e[1];
        P.ez = e[2];
        P.out = k == 0 ? b1 : (k == 1 ? b2 : out);
        P.level = level;
        P.dt_dev = dt_dev;
        P.dh_dev = dh_dev;
        P.n_levels = n_levels;
        P.gamma = gamma;
        P.n_groups = n;
        const dim3 bl(256);
        const bool pair = k == order;  // the x and y sweeps: the first two, or the last two
        if (periodic && pair) {
            P.tiles = (gx * NI + XWIDTH - 1) / XWIDTH;
            P.width = (gx * NI + P.tiles - 1) / P.tiles;
            P.seg = march_segment(int64_t(P.tiles) * gz * 4, gy);
        }
        if (periodic && pair && together<T>(true, order, P.seg, n) && int64_t(gx) * int64_t(GOUT * sizeof(T)) <= int64_t(1) << 32) {
            const int64_t blocks = int64_t(P.tiles) * gz * 4 * ((gy * NI + P.seg - 1) / P.seg);
            if (blocks > INT32_MAX) return hipErrorInvalidValue;
            if (k == 1) P.out = out;
            if (order == 0) hipLaunchKernelGGL((rtvd_xy<T, 0, true>), dim3(unsigned(blocks)), bl, 0, s, P);
            else hipLaunchKernelGGL((rtvd_xy<T, 1, true>), dim3(unsigned(blocks)), bl, 0, s, P);
            ++k;
        } else if (!periodic && pair && together<T>(false, order, 0, n)) {
            // two z planes per wave, four waves per work-group; rows of 2^20 work-groups
            const int64_t blocks = (n * (e[2] / 2) + 3) / 4;
            const int64_t cols = blocks < (1 << 20) ? blocks : (1 << 20);
            const dim3 gr(unsigned(cols), unsigned((blocks + cols - 1) / cols));
            P.out = k == 1 ? out : b2;
            if (order == 0) hipLaunchKernelGGL((rtvd_xy<T, 0, false>), gr, bl, 0, s, P);
            else hipLaunchKernelGGL((rtvd_xy<T, 1, false>), gr, bl, 0, s, P);
            e[0] -= 2 * RG;
            e[1] -= 2 * RG;
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
            src = P.out;
            ++k;
            continue;
        } else if (periodic && d == 0) {
            P.tiles = (gx * NI + XWIDTH - 1) / XWIDTH;
            P.width = (gx * NI + P.tiles - 1) / P.tiles;
            const int64_t blocks = int64_t(gy) * gz * P.tiles * 64;
            if (blocks > INT32_MAX) return hipErrorInvalidValue;
            hipLaunchKernelGGL((rtvd_x_periodic<T>), dim3(unsigned(blocks)), bl, 0, s, P);
        } else if (periodic) {
            const int gd = d == 1 ? gy : gz;
            const int64_t columns = n / gd;
            P.seg = march_segment(columns, gd);
            const int64_t blocks = columns * ((gd * NI + P.seg - 1) / P.seg);
            if (d == 1) hipLaunchKernelGGL((rtvd_march_periodic<T, 1>), dim3(unsigned(blocks)), bl, 0, s, P);
            else hipLaunchKernelGGL((rtvd_march_periodic<T, 2>), dim3(unsigned(blocks)), bl, 0, s, P);
        } else if (d == 0) {
            // five pencils per wave, four waves per work-group; rows of 2^20 work-groups
            const int64_t blocks = (n * (e[1] == RP ? x_waves<RP>() : x_waves<NI>()) + 3) / 4;
            const int64_t cols = blocks < (1 << 20) ? blocks : (1 << 20);
            const dim3 gr(unsigned(cols), unsigned((blocks + cols - 1) / cols));
            if (e[1] == RP) hipLaunchKernelGGL((rtvd_x_padded<T, RP>), gr, bl, 0, s, P);
            else hipLaunchKernelGGL((rtvd_x_padded<T, NI>), gr, bl, 0, s, P);
        } else {
            // one thread per pencil (contiguous across the wave)
            const int64_t pencils = n * (d == 1 ? int64_t(e[0]) * e[2] : int64_t(e[0]) * e[1]);
            if (pencils >= int64_t(1) << 31) return hipErrorInvalidValue;
            const dim3 gr(unsigned((pencils + 255) / 256));
            if (d == 1) hipLaunchKernelGGL((rtvd_march_padded<T, 1>), gr, bl, 0, s, P);
            else hipLaunchKernelGGL((rtvd_march_padded<T, 2>), gr, bl, 0, s, P);
        }
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        src = P.out;
        e[d] -= 2 * RG;
    }
    return hipSuccess;
}

template size_t rtvd_workspace_elems<float>(int64_t);
template size_t rtvd_workspace_elems<double>(int64_t);
template hipError_t launch_rtvd<float>(const float *, int, int, int, int64_t, const int8_t *, int,
                                       const double *, const double *, double, int, float *, float *,
                                       hipStream_t);
template hipError_t launch_rtvd<double>(const double *, int, int, int, int64_t, const int8_t *, int,
                                        const double *, const double *, double, int, double *,
                                        double *, hipStream_t);

}  // namespace gamer
