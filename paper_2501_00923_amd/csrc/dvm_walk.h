// A wave's walk over one cell's velocities, and the sums over a wave: shared by
// the sweeps and the kernels that read whole rows as they do.
#pragma once

#include "dvm_device.h"

namespace dvm {

typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));

// Velocities per lane and step: two adjacent ones of a velocity-grid row in
// FP32 with an even n1, so that a lane moves 16 bytes as in FP64.
template <typename T>
__device__ __forceinline__ bool pair_velocities(int n1)
{
    return sizeof(T) == 4 && (n1 & 1) == 0;
}

// ---------------------------------------------------------------------------
// a wave's walk over one cell's velocities
//
// A lane stays on one column of the velocity grid (V adjacent ones) for a
// whole walk down its rows (LaneMap of dvm_internal.h), so every factor of
// v1 is a per-lane constant of the inner loop, and the sums over the rows
// carry only the v2 factors (from LDS); the v1 factors join once per walk.
// Vector instructions per 64 velocities, 256x128 cells with 48x48 velocities,
// set-up and sums included, a column that changes every step against this: FP64
// primal 107 -> 89, FP32 primal 108 -> 77, adjoint with the residual's sums 165
// -> 114 and 130 -> 101, without (all but a call's last sweep) 95 and 89.
// (Where a walk has one step only, lane_map, nothing is shared between steps.)
// Lanes outside the grid run along on padded table entries (v = 1, weight 0)
// and buffer accesses that the row's range check drops.
// ---------------------------------------------------------------------------
constexpr int kOutside = 0x40000000;            // byte offset past any row (rows have at most 256 KB)

struct Walk {
    int a, b, off;           // column, first row, byte offset there
    bool in;                 // in the grid's columns
};

template <typename T, int V>
__device__ __forceinline__ Walk make_walk(const DevSolve &d, int lane, int i)
{
    Walk w;
    const int k = i * d.lm.ks + lane;
    const int r = (int)(((float)k + 0.5f) * d.lm.inv_width), m = k - r * d.lm.width;
    const bool idle = r >= d.lm.rows;
    w.a = idle ? d.lm.n1p - V : V * (m + i * d.lm.as);
    w.b = idle ? 0 : r;
    w.in = !idle && w.a < d.n1;
    w.off = w.in ? (r * d.n1 + w.a) * 2 * (int)sizeof(T) : kOutside;
    return w;
}

// V velocities' two components
template <typename T, int V>
struct Vals {
    T x[V], y[V];
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}

// NT: non-temporal
template <typename T, int V, bool NT>
__device__ __forceinline__ Vals<T, V> row_load(__amdgpu_buffer_rsrc_t r, int off)
{
    Vals<T, V> o;
    if constexpr (V * sizeof(T) == 8) {
        const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, NT ? 2 : 0);
        if constexpr (sizeof(T) == 8) {
            o.x[0] = __longlong_as_double(((unsigned long long)v.y << 32) | v.x);
            o.y[0] = __longlong_as_double(((unsigned long long)v.w << 32) | v.z);
        } else {
            o.x[0] = __uint_as_float(v.x);
            o.y[0] = __uint_as_float(v.y);
            o.x[1] = __uint_as_float(v.z);
            o.y[1] = __uint_as_float(v.w);
        }
    } else {
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, NT ? 2 : 0);
        o.x[0] = __uint_as_float(v.x);
        o.y[0] = __uint_as_float(v.y);
    }
    return o;
}

template <typename T, int V, bool NT>
__device__ __forceinline__ void row_store(__amdgpu_buffer_rsrc_t r, int off, const Vals<T, V> &o)
{
    if constexpr (V * sizeof(T) == 8) {
        u4 v;
        if constexpr (sizeof(T) == 8) {
            const unsigned long long a = __double_as_longlong(o.x[0]), b = __double_as_longlong(o.y[0]);
            v = u4{(unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32)};
        } else {
            v = u4{__float_as_uint(o.x[0]), __float_as_uint(o.y[0]), __float_as_uint(o.x[1]), __float_as_uint(o.y[1])};
        }
        __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, NT ? 2 : 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint(o.x[0]), __float_as_uint(o.y[0])}, r, off, 0, NT ? 2 : 0);
    }
}

// Reciprocal: hardware estimate and Newton steps, two in FP64 (error about
// one ulp) and one in FP32, where a run over every mantissa of one binade gave
// the correctly rounded 1 / x, at a third of the division's instructions.  (x
// and 1 / x normal and finite; 0 and infinity give NaN.)
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float recip(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// c + a b: fused in FP64, rounded twice in FP32, where the stored values
// carry the rounding: FP32 results stay those of the plain expressions to the
// last bit, so that a derivative's FP32 noise does not depend on the kernel
__device__ __forceinline__ double madd(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float madd(float a, float b, float c) { return c + a * b; }
// keeps a per-lane constant in its register (the compiler would recompute the
// product in every step)
__device__ __forceinline__ void keep(double &x) { asm("" : "+v"(x)); }
__device__ __forceinline__ void keep(float &x) { asm("" : "+v"(x)); }
// the loads above are issued before any LDS read below (table entries read
// late do not hold registers while the loads are in flight)
__device__ __forceinline__ void loads_first() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ double min0(double x) { return fmin(x, 0.0); }
__device__ __forceinline__ float min0(float x) { return fminf(x, 0.0f); }
__device__ __forceinline__ double max0(double x) { return fmax(x, 0.0); }
__device__ __forceinline__ float max0(float x) { return fmaxf(x, 0.0f); }

// v2 factors of a grid row b, shared by a workgroup's cells: v2, w, w v2, w v2^2 / 2
struct alignas(16) RowFactor {
    double v, w, wv, wh;
};
// v1 factors of a column a: v1, w
struct alignas(16) ColFactor {
    double v, w;
};
// weighted Maxwellian factors of a grid row in one cell (adjoint moments):
// e = w Y, e c2, e c2^2
struct alignas(16) AdjRow {
    double e, ec, ecc, pad;
};

// the workgroup's dynamic LDS (launch bytes: primal_lds, adjoint_lds)
extern __shared__ __align__(16) unsigned char sweep_smem[];

// The adjoint's sums of a thread over the walks before the current one, parked
// in LDS so that the inner loop does not hold 12 registers for them (sum k of
// a thread is a block's stride from the next: no bank conflicts).  256x128
// cells with 256 velocities, FP64 / FP32: 108 / 70 -> 99 / 60 us.  The primal
// keeps its four in registers: with fewer, more waves run at once and push
// each other's neighbour rows out of L2 (128x64 cells with 4096 velocities in
// FP64 234 -> 244 us).
struct WalkSums {
    double *p;
    __device__ __forceinline__ WalkSums() : p(reinterpret_cast<double *>(sweep_smem) + threadIdx.x) {}
    __device__ __forceinline__ double &operator[](int k) const { return p[k * kPatchCells * kWave]; }
};

// The velocity grid's values for the LDS tables, whose entries are numbered
// columns (n1p) first, then rows (n2p), padded past the grid with v = 1 and
// weight 0.  The kernels load a thread's first entries before anything else
// (their addresses need nothing but the arguments), so that these loads, the
// cell's and the neighbour list's wait for memory together.  Sweeps, us,
// primal / adjoint, against loading each where it is used: 256x128 cells with
// 16x16 velocities in FP64 58 / 92 -> 57 / 83, in FP32 41 / 60 -> 38 / 54,
// 128x64 with 32x32 in FP32 27.1 / 37.5 -> 26.2 / 36.3, 256x128 with 48x48 in
// FP64 468 / 659 -> 464 / 650.
struct GridEntry {
    int k;
    bool col, in;            // a column; inside the grid
    double v, w;
};
struct GridTables {
    int n1, n2, n1p, n;
    GlobalDoubles vx, vy, wx, wy;
    // (in registers: a choice between two arguments would be loaded per lane)
    __device__ __forceinline__ explicit GridTables(const DevSolve &d)
        : n1(uni(d.n1)), n2(uni(d.n2)), n1p(d.lm.n1p), n(d.lm.n1p + d.lm.n2p), vx(uni(d.vx)), vy(uni(d.vy)), wx(uni(d.wx)),
          wy(uni(d.wy))
    {
    }
    __device__ __forceinline__ GridEntry at(int i) const
    {
        GridEntry e;
        e.col = i < n1p;
        e.k = e.col ? i : i - n1p;
        const int m = e.col ? n1 : n2, k = min(e.k, m - 1);
        e.in = e.k < m;
        e.v = (e.col ? vx : vy)[k];
        e.w = (e.col ? wx : wy)[k];
        return e;
    }
    // put(i, entry i) for i = i0, i0 + step, ...; e: entry i0
    template <typename Put>
    __device__ __forceinline__ void each(int i0, int step, GridEntry e, Put put) const
    {
        for (int i = i0; i < n; i += step) {
            GridEntry next = e;
            if (i + step < n) next = at(i + step);
            put(i, e);
            e = next;
        }
    }
};

// The workgroup's shared tables from byte `at` of its LDS.
struct Factors {
    RowFactor *row;
    ColFactor *col;
    void *end;
    __device__ __forceinline__ Factors(const DevSolve &d, int at)
    {
        row = reinterpret_cast<RowFactor *>(sweep_smem + at);
        col = reinterpret_cast<ColFactor *>(row + d.lm.n2p);
        end = col + d.lm.n1p;
    }
    __device__ __forceinline__ void put(const GridEntry &e) const
    {
        const double v = e.in ? e.v : 1.0, w = e.in ? e.w : 0.0;
        if (e.col) {
            col[e.k] = {v, w};
        } else {
            const double wv = w * v;
            row[e.k] = {v, w, wv, 0.5 * (wv * v)};
        }
    }
    // e: entry threadIdx.x; all threads of the workgroup, no barrier
    __device__ __forceinline__ void fill(const GridTables &g, const GridEntry &e) const
    {
        g.each(threadIdx.x, kPatchCells * kWave, e, [&](int, const GridEntry &x) { put(x); });
    }
};

// ---------------------------------------------------------------------------
// sums over the wave: lane l ends with the total of v[l / 8], by pairwise
// exchanges that halve the number of values carried (34 vector instructions
// for 8 values; a butterfly of each value takes 12 LDS exchanges per value).
// The order is fixed and the same in every kernel that sums moments.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x)
{
    const unsigned long long u = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

template <int HALF>
__device__ __forceinline__ double swap_add(double a, double b)
{
    const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    u2 lo, hi;
    if constexpr (HALF == 32) {
        lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
        hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
        hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    }
    return __longlong_as_double(((unsigned long long)hi.x << 32) | lo.x) +
           __longlong_as_double(((unsigned long long)hi.y << 32) | lo.y);
}

__device__ __forceinline__ double wave_scatter8(const double (&v)[8])
{
    double q[4], p[2];
#pragma unroll
    for (int i = 0; i < 4; i++) q[i] = swap_add<32>(v[i], v[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; i++) p[i] = swap_add<16>(q[i], q[i + 2]);
    const bool up = (threadIdx.x & 8) != 0;
    double s = (up ? p[1] : p[0]) + dpp_move<0x128>(up ? p[0] : p[1]);     // lane ^ 8
    s += dpp_move<0x141>(s);                                               // lane ^ 7
    s += dpp_move<0x4e>(s);                                                // lane ^ 2
    s += dpp_move<0xb1>(s);                                                // lane ^ 1
    return s;
}

// value of a lane, the same in every lane
__device__ __forceinline__ double lane_value(double x, int lane)
{
    const unsigned long long u = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// LDS tables of the adjoint kernels: the shared factors, then per cell the
// weighted Maxwellian factors (adj, gx) and the source's v2 part (qb)
template <typename T>
struct AdjLds {
    Factors fac;
    AdjRow *adj;
    double *gx;
    T *qb;
    __device__ __forceinline__ AdjLds(const DevSolve &d, int w) : fac(d, kWalkSums * (int)sizeof(double) * kPatchCells * kWave)
    {
        AdjRow *a0 = static_cast<AdjRow *>(fac.end);
        double *g0 = reinterpret_cast<double *>(a0 + kPatchCells * d.lm.n2p);
        T *q0 = reinterpret_cast<T *>(g0 + kPatchCells * d.lm.n1p);
        adj = a0 + w * d.lm.n2p;
        gx = g0 + w * d.lm.n1p;
        qb = q0 + w * d.lm.n2p;
    }
    // this wave's Maxwellian factors of the frozen state from entry i0 in steps
    // of `step` (e0: entry i0); row(k, v2): anything else per row; no
    // barrier
    template <typename Row>
    __device__ __forceinline__ void fill(const GridTables &g, const GridEntry &e0, const double *ac, int i0, int step,
                                         Row row) const
    {
        const double u1 = uni(ac[1]), u2 = uni(ac[2]), h = 0.5 * recip(uni(ac[3])), gc = uni(ac[5]);
        g.each(i0, step, e0, [&](int, const GridEntry &e) {
            const double c = e.in ? e.v - (e.col ? u1 : u2) : 0.0, w = e.in ? e.w : 0.0;
            const double x = w * exp(-c * c * h);
            if (e.col) {
                gx[e.k] = gc * x;
            } else {
                adj[e.k] = {x, x * c, x * c * c, 0.0};
                row(e.k, e.in ? e.v : 1.0);
            }
        });
    }
    __device__ __forceinline__ void fill(const GridTables &g, const double *ac, int lane) const
    {
        fill(g, g.at(lane), ac, lane, kWave, [](int, double) {});
    }
};

// What a wave of a sweep works on.  A row's steps are summed in `parts` equal
// parts (sweep_parts), each reduced over the wave and added in order, so that a
// cell's sums do not depend on whether one wave walks all parts or `parts`
// waves one each.
struct SweepUnit {
    int c;                   // cell
    bool act;                // exists (idle waves of a partial patch run along on the first cell without storing)
    int slot;                // the cell's LDS tables
    int fill0, fill_step;    // table entries this lane fills
    int p0, p1, parts;       // parts p0 .. p1 - 1 of parts
};

// wave w of a workgroup that takes patch p, one cell a wave
__device__ __forceinline__ SweepUnit patch_unit(const DevSolve &d, int p, int parts)
{
    const int w = uni((int)(threadIdx.x / kWave));
    const int c0 = uni(d.patch[p]), cnt = uni(d.patch[p + 1]) - c0;
    SweepUnit u;
    u.act = w < cnt;
    u.c = c0 + (u.act ? w : 0);
    u.slot = w;
    u.fill0 = threadIdx.x % kWave;
    u.fill_step = kWave;
    u.p0 = 0;
    u.p1 = u.parts = parts;
    return u;
}

// wave w of the k-th of `parts` (2 or 4) workgroups that share patch p, `parts`
// waves a cell
__device__ __forceinline__ SweepUnit part_unit(const DevSolve &d, int p, int k, int parts)
{
    const int w = uni((int)(threadIdx.x / kWave)), cells = kPatchCells >> (parts >> 1);
    const int c0 = uni(d.patch[p]), cnt = uni(d.patch[p + 1]) - c0;
    SweepUnit u;
    u.slot = w >> (parts >> 1);
    const int i = k * cells + u.slot;
    u.act = i < cnt;
    u.c = c0 + (u.act ? i : 0);
    u.fill0 = (w & (parts - 1)) * kWave + threadIdx.x % kWave;
    u.fill_step = parts * kWave;
    u.p0 = w & (parts - 1);
    u.p1 = u.p0 + 1;
    u.parts = parts;
    return u;
}

// The pieces of parts p0 .. p1 - 1 in walk order: go(i, t0, n) takes steps t0 ..
// t0 + n - 1 of walk i, done() ends a part.  PARTS: there is more than one (the
// plain walk costs a launch of few short rows up to 9 % less).
template <bool PARTS, typename Go, typename Done>
__device__ __forceinline__ void walk_parts(const LaneMap &m, int p0, int p1, int parts, Go go, Done done)
{
    if constexpr (!PARTS) {
        for (int i = 0; i < m.isteps; i++) go(i, 0, m.tq + (i < m.tr ? 1 : 0));
        done();
        return;
    }
    int i = 0, start = 0;
    for (int p = p0; p < p1; p++) {
        int g = m.total * p >> (parts >> 1);
        const int ge = m.total * (p + 1) >> (parts >> 1);
        while (g < ge) {
            int steps = m.tq + (i < m.tr ? 1 : 0);
            while (g >= start + steps) {
                start += steps;
                i++;
                steps = m.tq + (i < m.tr ? 1 : 0);
            }
            const int n = min(start + steps, ge) - g;
            go(i, g - start, n);
            g += n;
        }
        done();
    }
}

// the wave's cell of patch p: its number, whether it exists (idle waves of a
// partial patch run along on the first cell without storing)
__device__ __forceinline__ int patch_wave(const DevSolve &d, int p, int &w, bool &act)
{
    w = uni((int)(threadIdx.x / kWave));
    const int c0 = uni(d.patch[p]), cnt = uni(d.patch[p + 1]) - c0;
    act = w < cnt;
    return c0 + (act ? w : 0);
}

}  // namespace dvm
