// Second-order reconstruction kernels of libdvm (Sec. 3.1 states
// second-order accuracy in physical space for the primal and the adjoint
// balance and leaves the scheme to its references).  The scheme: cell
// values at the cell centroids, Green-Gauss slopes with the face mean of
// the two cell values (the cell value on a boundary face), the
// Venkatakrishnan limiter (smoothing relative to the cell value), and face
// values reconstructed on the upwind side
// (far-field and wall inflow are not reconstructed; the wall flux F_l sums
// the reconstructed outgoing values).
//
// It is applied by defect correction: every K sweeps
//   k_so_slope  limited slopes G of f and the wall-flux correction dF,
//   k_so_corr   c = sum_q (v.S_q) (second- minus first-order face value),
// and the first-order sweep subtracts the held c and uses F + dF.  The
// adjoint linearises with the limiter factors of the converged f frozen
// (k_so_slope in its psi mode) and holds, every K sweeps,
//   k_so_adj_b  B_u = psi_u sum_{outflow q} (v.S_q)(phi_u - phi_down)(m_q - x_u),
//   k_so_adj_e  E_m, the transpose of the Green-Gauss sum applied to B,
// which the adjoint sweep subtracts.
//
// Layout and launch as in the sweeps: one workgroup per patch (XCD-aware
// order), one wave per cell, a lane per velocity; per-cell constants in
// scalar registers.  Each kernel reads its cell's row and its interior
// neighbours' rows (in L2 for the same reasons as in the sweeps) and writes
// one row.  All are bound by memory; 256x128 cells with 48x48 velocities in
// FP64, us: slopes 806 (1045 when the limiter took four fractions and bound
// them), psi 611 (867), c 799 (868), B 939 (1084), E 894 (1004).  Rows go
// through buffer accesses whose range check drops what is not wanted (a
// boundary face's neighbour, a face that the velocity does not cross that
// way), so a step issues its loads together without a branch.  FP32
// expressions keep their order and roundings.

#include "dvm_walk.h"

namespace dvm {

namespace {

constexpr int kSoBlock = kPatchCells * kWave;

// Per-cell constants of one wave's cell c: neighbour codes, face vectors,
// the face-midpoint offsets from c's centroid (r) and from the neighbours'
// centroids (rn), 1 / V.
template <typename T>
struct Cell {
    int c, nb[4];
    T Sx[4], Sy[4], rx[4], ry[4], nx[4], ny[4];
    T iV, iVn[4];
};

template <typename T>
__device__ __forceinline__ Cell<T> load_cell(const DevSolve &d, int c, bool want_rn)
{
    Cell<T> g;
    g.c = c;
    g.iV = uni((T)(1.0 / d.vol[c]));
#pragma unroll
    for (int q = 0; q < 4; q++) {
        g.nb[q] = uni(d.nbr[4 * c + q]);
        g.Sx[q] = uni((T)d.S[8 * c + 2 * q]);
        g.Sy[q] = uni((T)d.S[8 * c + 2 * q + 1]);
        g.rx[q] = uni((T)d.rf[8 * c + 2 * q]);
        g.ry[q] = uni((T)d.rf[8 * c + 2 * q + 1]);
        if (want_rn) {
            g.nx[q] = uni((T)d.rn[8 * c + 2 * q]);
            g.ny[q] = uni((T)d.rn[8 * c + 2 * q + 1]);
            g.iVn[q] = uni((T)(g.nb[q] >= 0 ? 1.0 / d.vol[g.nb[q]] : 0.0));
        } else {
            g.nx[q] = g.ny[q] = g.iVn[q] = 0;
        }
    }
    return g;
}

// Venkatakrishnan smoothing relative to the cell value: e = kVkKappa |f_c|
constexpr double kVkKappa = 1e-3;

__device__ __forceinline__ double max2(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float max2(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double min2(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float min2(float a, float b) { return fminf(a, b); }

// Row of a cell in an array of `bytes` a cell, and those of its neighbours:
// without bytes (all loads zero) behind boundary faces.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t cell_row(const void *p, int c, int bytes)
{
    return row_rsrc(static_cast<const char *>(p) + (size_t)c * bytes, bytes);
}
template <typename T>
__device__ __forceinline__ void neighbour_rows(const void *p, const Cell<T> &g, int bytes, __amdgpu_buffer_rsrc_t (&r)[4])
{
#pragma unroll
    for (int q = 0; q < 4; q++)
        r[q] = row_rsrc(static_cast<const char *>(p) + (size_t)(g.nb[q] >= 0 ? g.nb[q] : g.c) * bytes,
                        g.nb[q] >= 0 ? bytes : 0);
}

// Slopes of velocity k (layout: Slopes); nothing if !want.
template <typename T>
__device__ __forceinline__ Slopes<T> slope_load(__amdgpu_buffer_rsrc_t r, int k, int nv, bool want)
{
    const int off = want ? 16 * k : kOutside;
    if constexpr (sizeof(T) == 8) {
        const Vals<T, 1> a = row_load<T, 1, false>(r, off), b = row_load<T, 1, false>(r, off + 16 * nv);
        return {{a.x[0], b.x[0]}, {a.y[0], b.y[0]}};
    } else {
        const Vals<T, 2> a = row_load<T, 2, false>(r, off);
        return {{a.x[0], a.x[1]}, {a.y[0], a.y[1]}};
    }
}
template <typename T>
__device__ __forceinline__ void slope_store(__amdgpu_buffer_rsrc_t r, int k, int nv, const Slopes<T> &o)
{
    if constexpr (sizeof(T) == 8) {
        row_store<T, 1, true>(r, 16 * k, Vals<T, 1>{{o.x[0]}, {o.y[0]}});
        row_store<T, 1, true>(r, 16 * (k + nv), Vals<T, 1>{{o.x[1]}, {o.y[1]}});
    } else {
        row_store<T, 2, true>(r, 16 * k, Vals<T, 2>{{o.x[0], o.x[1]}, {o.y[0], o.y[1]}});
    }
}

// Limited slope of one component: Green-Gauss gradient from the cell value
// fc and the interior neighbours' values fn (fc at a boundary face), then the
// Venkatakrishnan factor p = min(1, min_q (D^2 + e^2 + 2 d D) / (D^2 + 2 d^2 +
// d D + e^2)) with d the face's unlimited increment grad . r_q and D the room
// to the neighbourhood's max (d > 0) or min.  For D > 0 the fraction is at
// least 1 up to d = D / 2 and falls from there on (the sign of its derivative
// is that of D^3 - 4 d D (d + D) + e^2 (D - 4 d)), so the smallest one of a
// side is that of its largest |d|, or above 1: two fractions instead of four.
// The smaller is found by comparing cross products, then divided once (IEEE).
// The limiter arithmetic is FP64 for both storage types, on d, D and e
// rescaled by the power of two nearest 1 / |f_c| (exact, and the fractions are
// homogeneous of degree 0): squares of values near the Maxwellian's tail
// (f ~ 1e-22 and below on common grids) underflow in FP32, and the adjoint
// uses p on its own, not only p grad f.
template <typename T>
__device__ __forceinline__ void slope1(const Cell<T> &g, T fc, const T (&fn)[4], int lim, T &gx, T &gy, T &p)
{
    // FP64 from the differences (the face vectors of a cell add up to zero),
    // with g.Sx, g.Sy as they are; FP32 from the values, so that D is taken in
    // FP64 without a rounding to FP32 before
    constexpr bool kDiff = sizeof(T) == 8;
    T hi = kDiff ? (T)0 : fc, lo = hi;
    gx = 0;
    gy = 0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const T x = kDiff ? fn[q] - fc : fn[q];
        const T b = kDiff ? x : (T)0.5 * (fc + fn[q]);
        hi = max2(hi, x);
        lo = min2(lo, x);
        gx = madd(b, g.Sx[q], gx);
        gy = madd(b, g.Sy[q], gy);
    }
    const T h = kDiff ? (T)0.5 * g.iV : g.iV;
    gx *= h;
    gy *= h;
    p = 1;
    if (lim) {
        int ex = 0;
        (void)frexp((double)fc, &ex);
        const double sc = ldexp(1.0, -ex);
        const double e = kVkKappa * ((double)fc * sc), e2 = e * e;
        const double f0 = kDiff ? 0.0 : (double)fc;
        const double Dh = ((double)hi - f0) * sc, Dl = ((double)lo - f0) * sc, gxd = (double)gx * sc, gyd = (double)gy * sc;
        double dh = 0, dl = 0;       // largest increment of either sign
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const double t = fma(gxd, (double)g.rx[q], gyd * (double)g.ry[q]);
            dh = max2(dh, t);
            dl = min2(dl, t);
        }
        const double ph = fma(Dh, Dh, e2), pl = fma(Dl, Dl, e2);
        const double nh = fma(2.0 * dh, Dh, ph), mh = fma(dh, fma(2.0, dh, Dh), ph);
        const double nl = fma(2.0 * dl, Dl, pl), ml = fma(dl, fma(2.0, dl, Dl), pl);
        const bool low = !(mh > 0) || nl * mh < nh * ml;
        const double n = low ? nl : nh, m = low ? ml : mh;
        p = n < m ? (T)(n / m) : (T)1;   // 0 / 0: no increment, no limit
    }
}

// the wave's cell of patch p, or -1 for an idle wave of a partial patch
__device__ __forceinline__ int patch_cell(const DevSolve &d, int p)
{
    const int w = uni((int)(threadIdx.x / kWave));
    const int c0 = uni(d.patch[p]), cnt = uni(d.patch[p + 1]) - c0;
    return w < cnt ? c0 + w : -1;
}

// A launch takes the rows in slabs of kSlab velocities, one after the other:
// each XCD all its patches for the first slab, then all for the second, so
// that a row of patches and its neighbours fit the XCD's L2 together.  With
// whole rows the neighbours came from memory again (256x128 cells with 48x48
// velocities in FP64, reads over the arrays' size: slopes 2.0, E 2.3).  us
// there, with slabs of 128 / 256 / 512 / all velocities: slopes 793 / 806 /
// 829 / 884, c 802 / 799 / 801 / 837, psi 590 / 611 / 625 / 670, B 960 / 939 /
// 948 / 965, E 888 / 894 / 920 / 1000.
constexpr int kSlab = 256;
__device__ __forceinline__ int slab_cell(const DevSolve &d, int b, int &k0, int &k1)
{
    const int per = (d.np + 7) >> 3, i = b >> 3, slab = i / per, p = (b & 7) * per + i - slab * per;
    k0 = slab * kSlab;
    k1 = min(k0 + kSlab, d.nv);
    return p < d.np ? patch_cell(d, p) : -1;
}
static int slab_grid(const DevSolve &d) { return 8 * ((d.np + 7) / 8) * ((d.nv + kSlab - 1) / kSlab); }

// dF_l: what the limited slopes of the wall cell add to the wall flux F_l; a
// workgroup per element, from f itself so that it needs not wait for G
template <typename T>
__device__ __forceinline__ void wall_flux(const DevSolve &d, int par, int l)
{
    __shared__ double red[kSoBlock / kWave];
    const int c = uni(d.wall_cell[l]), rowb = d.nv * 2 * (int)sizeof(T);
    const Cell<T> g = load_cell<T>(d, c, false);
    const double S0x = d.S[8 * c], S0y = d.S[8 * c + 1];
    const __amdgpu_buffer_rsrc_t own = cell_row(d.f[par], c, rowb);
    __amdgpu_buffer_rsrc_t nbr[4];
#pragma unroll
    for (int q = 0; q < 4; q++) nbr[q] = cell_row(d.f[par], g.nb[q] >= 0 ? g.nb[q] : c, rowb);
    double acc[1] = {0};
    for (int k = threadIdx.x; k < d.nv; k += kSoBlock) {
        const int a = k % d.n1, b = k / d.n1, off = k * 2 * (int)sizeof(T);
        const double s0 = d.vx[a] * S0x + d.vy[b] * S0y;
        const T fc = row_load<T, 1, false>(own, off).x[0];
        T fn[4], gx, gy, p;
#pragma unroll
        for (int q = 0; q < 4; q++) fn[q] = row_load<T, 1, false>(nbr[q], off).x[0];
        slope1(g, fc, fn, d.limiter, gx, gy, p);
        if (s0 > 0) acc[0] += d.wx[a] * d.wy[b] * s0 * (double)(p * gx * g.rx[0] + p * gy * g.ry[0]);
    }
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) d.dF[l] = acc[0] / d.wall_A[l];
}

// Limited slopes of f[par] into G and the wall elements' dF (PSI = false), or
// the limiter factors into psi (PSI = true).  The first `walls` workgroups (a
// multiple of 8: the others' XCDs stay) take a wall element each: as a launch of
// its own dF cost 2 us on small meshes (24x10 cells with 8x8 velocities, sweep and
// correction 16.0 -> 13.6 us), 12 on 256x128 cells with 48x48.
template <typename T, bool PSI>
__global__ __launch_bounds__(kSoBlock) void k_so_slope(DevSolve d, int par, int walls)
{
    if constexpr (!PSI) {
        if ((int)blockIdx.x < walls) {
            if ((int)blockIdx.x < d.nw) wall_flux<T>(d, par, blockIdx.x);
            return;
        }
    }
    int k0, k1;
    const int c = slab_cell(d, (int)blockIdx.x - walls, k0, k1);
    if (c < 0) return;
    const int lane = threadIdx.x % kWave, nv = d.nv, lim = d.limiter, rowb = nv * 2 * (int)sizeof(T);
    const Cell<T> g = load_cell<T>(d, c, false);
    const __amdgpu_buffer_rsrc_t own = cell_row(d.f[par], c, rowb);
    const __amdgpu_buffer_rsrc_t dst = PSI ? cell_row(d.psi, c, rowb) : cell_row(d.G, c, 2 * rowb);
    __amdgpu_buffer_rsrc_t nbr[4];
#pragma unroll
    for (int q = 0; q < 4; q++) nbr[q] = cell_row(d.f[par], g.nb[q] >= 0 ? g.nb[q] : c, rowb);
    for (int k = k0 + lane; k < k1; k += kWave) {
        const int off = k * 2 * (int)sizeof(T);
        const Vals<T, 1> fc = row_load<T, 1, false>(own, off);
        Vals<T, 1> fn[4];
#pragma unroll
        for (int q = 0; q < 4; q++) fn[q] = row_load<T, 1, false>(nbr[q], off);
        const T f1[4] = {fn[0].x[0], fn[1].x[0], fn[2].x[0], fn[3].x[0]};
        const T f2[4] = {fn[0].y[0], fn[1].y[0], fn[2].y[0], fn[3].y[0]};
        T g1x, g1y, p1, g2x, g2y, p2;
        slope1(g, fc.x[0], f1, lim, g1x, g1y, p1);
        slope1(g, fc.y[0], f2, lim, g2x, g2y, p2);
        if constexpr (PSI) {
            row_store<T, 1, true>(dst, off, Vals<T, 1>{{p1}, {p2}});
        } else {
            const Slopes<T> o = {{p1 * g1x, p2 * g2x}, {p1 * g1y, p2 * g2y}};
            slope_store(dst, k, nv, o);
        }
    }
}

// c = sum_q (v.S_q) G_u . (m_q - x_u) with u the upwind cell of face q
// (nothing for inflow through a boundary)
template <typename T>
__global__ __launch_bounds__(kSoBlock) void k_so_corr(DevSolve d)
{
    int k0, k1;
    const int c = slab_cell(d, blockIdx.x, k0, k1);
    if (c < 0) return;
    const int lane = threadIdx.x % kWave, nv = d.nv, n1 = d.n1, rowb = nv * 2 * (int)sizeof(T);
    const Cell<T> g = load_cell<T>(d, c, true);
    const __amdgpu_buffer_rsrc_t own = cell_row(d.G, c, 2 * rowb), dst = cell_row(d.corr, c, rowb);
    __amdgpu_buffer_rsrc_t nbr[4];
    neighbour_rows(d.G, g, 2 * rowb, nbr);
    int a = (k0 + lane) % n1, b = (k0 + lane) / n1;
    const int da = kWave % n1, db = kWave / n1;
    for (int k = k0 + lane; k < k1; k += kWave) {
        const T v1 = (T)d.vx[a], v2 = (T)d.vy[b];
        const Slopes<T> o = slope_load<T>(own, k, nv, true);
        // a neighbour's slopes are needed only where it is upwind
        T sq[4];
        Slopes<T> n[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            sq[q] = madd(v2, g.Sy[q], v1 * g.Sx[q]);
            n[q] = slope_load<T>(nbr[q], k, nv, !(sq[q] > 0));
        }
        Vals<T, 1> r = {{0}, {0}};
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const T sp = max0(sq[q]), sm = min0(sq[q]);
            r.x[0] = madd(sp, madd(o.y[0], g.ry[q], o.x[0] * g.rx[q]), r.x[0]);
            r.y[0] = madd(sp, madd(o.y[1], g.ry[q], o.x[1] * g.rx[q]), r.y[0]);
            r.x[0] = madd(sm, madd(n[q].y[0], g.ny[q], n[q].x[0] * g.nx[q]), r.x[0]);
            r.y[0] = madd(sm, madd(n[q].y[1], g.ny[q], n[q].x[1] * g.nx[q]), r.y[0]);
        }
        row_store<T, 1, true>(dst, k * 2 * (int)sizeof(T), r);
        a += da;
        b += db;
        if (a >= n1) {
            a -= n1;
            b++;
        }
    }
}

// B_u = psi_u sum_{q: v.S_q > 0} (v.S_q)(phi_u - phi_down,q)(m_q - x_u), with
// phi_down the neighbour's phi, 0 at the far field, (Phi_l - m_J, 0) at the wall
template <typename T>
__global__ __launch_bounds__(kSoBlock) void k_so_adj_b(DevSolve d, int par)
{
    int k0, k1;
    const int c = slab_cell(d, blockIdx.x, k0, k1);
    if (c < 0) return;
    const int lane = threadIdx.x % kWave, nv = d.nv, n1 = d.n1, obj = d.objective, rowb = nv * 2 * (int)sizeof(T);
    const Cell<T> g = load_cell<T>(d, c, false);
    const __amdgpu_buffer_rsrc_t own = cell_row(d.phi[par], c, rowb), lim = cell_row(d.psi, c, rowb);
    const __amdgpu_buffer_rsrc_t dst = cell_row(d.G, c, 2 * rowb);
    __amdgpu_buffer_rsrc_t nbr[4];
    neighbour_rows(d.phi[par], g, rowb, nbr);
    const int wl = g.nb[0] <= -2 ? -2 - g.nb[0] : -1;
    const T Phi_w = wl >= 0 ? uni((T)d.Phi[par][wl]) : (T)0;
    int a = (k0 + lane) % n1, b = (k0 + lane) / n1;
    const int da = kWave % n1, db = kWave / n1;
    for (int k = k0 + lane; k < k1; k += kWave) {
        const int off = k * 2 * (int)sizeof(T);
        const double v1d = d.vx[a], v2d = d.vy[b];
        const T v1 = (T)v1d, v2 = (T)v2d;
        const Vals<T, 1> pu = row_load<T, 1, false>(own, off), ps = row_load<T, 1, false>(lim, off);
        // a neighbour's phi is needed only where it is downwind
        T sq[4];
        Vals<T, 1> pd[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            sq[q] = madd(v2, g.Sy[q], v1 * g.Sx[q]);
            pd[q] = row_load<T, 1, false>(nbr[q], sq[q] > 0 ? off : kOutside);
        }
        if (wl >= 0) pd[0].x[0] = Phi_w - (T)mJ_of(obj, v1d, v2d);
        Slopes<T> o = {{0, 0}, {0, 0}};
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const T s = max0(sq[q]);
            const T a1 = s * (pu.x[0] - pd[q].x[0]), a2 = s * (pu.y[0] - pd[q].y[0]);
            o.x[0] = madd(a1, g.rx[q], o.x[0]);
            o.y[0] = madd(a1, g.ry[q], o.y[0]);
            o.x[1] = madd(a2, g.rx[q], o.x[1]);
            o.y[1] = madd(a2, g.ry[q], o.y[1]);
        }
        slope_store(dst, k, nv,
                    Slopes<T>{{o.x[0] * ps.x[0], o.x[1] * ps.y[0]}, {o.y[0] * ps.x[0], o.y[1] * ps.y[0]}});
        a += da;
        b += db;
        if (a >= n1) {
            a -= n1;
            b++;
        }
    }
}

// E_m = d/df_m of sum_u B_u . grad f_u with grad f_u = (1/V_u) sum_q fbar_q S_uq:
// the own part (1/2 on interior faces, 1 on boundary faces) and, through each
// interior face q, the neighbour's part with its face vector -S_q.
template <typename T>
__global__ __launch_bounds__(kSoBlock) void k_so_adj_e(DevSolve d)
{
    int k0, k1;
    const int c = slab_cell(d, blockIdx.x, k0, k1);
    if (c < 0) return;
    const int lane = threadIdx.x % kWave, nv = d.nv, rowb = nv * 2 * (int)sizeof(T);
    const Cell<T> g = load_cell<T>(d, c, true);
    const __amdgpu_buffer_rsrc_t own = cell_row(d.G, c, 2 * rowb), dst = cell_row(d.corr, c, rowb);
    __amdgpu_buffer_rsrc_t nbr[4];
    neighbour_rows(d.G, g, 2 * rowb, nbr);
    for (int k = k0 + lane; k < k1; k += kWave) {
        const Slopes<T> o = slope_load<T>(own, k, nv, true);
        Slopes<T> n[4];
#pragma unroll
        for (int q = 0; q < 4; q++) n[q] = slope_load<T>(nbr[q], k, nv, true);
        T e[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < 4; q++) {
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const T t = madd(o.y[i], g.Sy[q], o.x[i] * g.Sx[q]) * g.iV;
                const T u = madd(n[q].y[i], g.Sy[q], n[q].x[i] * g.Sx[q]) * g.iVn[q];
                e[i] += g.nb[q] >= 0 ? (T)0.5 * (t - u) : t;
            }
        }
        row_store<T, 1, true>(dst, k * 2 * (int)sizeof(T), Vals<T, 1>{{e[0]}, {e[1]}});
    }
}

// J_l = A_l sum_k w m_J (v.n) f1_{l,k} with the outgoing wall values
// reconstructed from f[par] and the incoming ones (F_l + dF_l) gbar1, dF_l
// of the same f: one block per element.  With H = sum_{Xi^-} w m_J (v.n)
// gbar1, J_l = A_l (sum_{Xi^+} w m_J (v.n) f1 + (F_l + dF_l) H).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_so_objective_elem(DevSolve d, int par)
{
    using T2 = typename Vec2<T>::type;
    __shared__ double red[4 * 3];
    const int l = blockIdx.x;
    const int c = d.wall_cell[l];
    const T2 *f = static_cast<const T2 *>(d.f[par]);
    const T *gM = static_cast<const T *>(d.gM);
    const Cell<T> g = load_cell<T>(d, c, false);
    const double n1 = d.wall_n[2 * l], n2 = d.wall_n[2 * l + 1], iD = 1.0 / d.D[l];
    double jp = 0, dF = 0, H = 0;
    for (int k = threadIdx.x; k < d.nv; k += kBlock) {
        const int a = k % d.n1, b = k / d.n1;
        const double v1 = d.vx[a], v2 = d.vy[b];
        const double vn = v1 * n1 + v2 * n2;
        const double wm = d.wx[a] * d.wy[b] * mJ_of(d.objective, v1, v2);
        if (vn > 0) {
            const T2 fc = f[(size_t)c * d.nv + k];
            T f1[4];
#pragma unroll
            for (int q = 0; q < 4; q++) f1[q] = f[(size_t)(g.nb[q] >= 0 ? g.nb[q] : c) * d.nv + k].x;
            T gx, gy, p1;
            slope1(g, fc.x, f1, d.limiter, gx, gy, p1);
            const double delta = (double)((p1 * gx) * g.rx[0] + (p1 * gy) * g.ry[0]);
            jp += wm * vn * ((double)fc.x + delta);
            dF += d.wx[a] * d.wy[b] * vn * delta;
        } else {
            H += wm * vn * (double)gM[k] * iD;
        }
    }
    double acc[3] = {jp, dF, H};
    block_sum<3>(acc, red);
    if (threadIdx.x == 0) d.Jl[l] = d.wall_A[l] * (acc[0] + (d.F[par][l] + acc[1]) * acc[2]);
}

}  // namespace

hipError_t launch_so_slopes(const DevSolve &d, int par, hipStream_t st)
{
    const int walls = xcd_grid(d.nw);
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_so_slope<T, false>), dim3(walls + slab_grid(d)), dim3(kSoBlock), 0, st, d,
                                             par, walls));
    return hipGetLastError();
}

hipError_t launch_so_correction(const DevSolve &d, int par, hipStream_t st)
{
    if (hipError_t e = launch_so_slopes(d, par, st)) return e;
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_so_corr<T>, dim3(slab_grid(d)), dim3(kSoBlock), 0, st, d));
    return hipGetLastError();
}

hipError_t launch_so_freeze(const DevSolve &d, int fpar, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_so_slope<T, true>), dim3(slab_grid(d)), dim3(kSoBlock), 0, st, d, fpar, 0));
    return hipGetLastError();
}

hipError_t launch_so_adjoint_term(const DevSolve &d, int par, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_so_adj_b<T>, dim3(slab_grid(d)), dim3(kSoBlock), 0, st, d, par));
    if (hipError_t e = hipGetLastError()) return e;
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_so_adj_e<T>, dim3(slab_grid(d)), dim3(kSoBlock), 0, st, d));
    return hipGetLastError();
}

hipError_t launch_so_objective_elem(const DevSolve &d, int par, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_so_objective_elem<T>, dim3(d.nw), dim3(kBlock), 0, st, d, par));
    return hipGetLastError();
}

}  // namespace dvm
