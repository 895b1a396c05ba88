// HIP kernels of libdvm for gfx950 (CDNA4).
//
// Layout: f and phi are [cell][velocity][2] (the two reduced distributions
// of Sec. 2.2 interleaved), so one cell's row of 2*nv values is contiguous
// and a wave64 reading consecutive velocities streams whole cache lines.
// Cells are numbered on the device in sweep order (see dvm_internal.h).
//
// Sweeps: a workgroup takes a patch of up to kPatchCells cells, one wave per
// cell, or, where rows are summed in parts (sweep_parts), one or two of its
// cells, one wave per part.  A wave walks its cell's velocities 64 or 128 at a
// time (dvm_walk.h) and reads the neighbour rows it needs from L2 (the
// neighbouring patch ran shortly before or runs alongside on the same XCD; a
// neighbour in the same patch is in L1), far-field and wall rows from tables.  The FP64 velocity
// moments of the new row are summed in registers and reduced across the wave
// in a fixed order, so the next sweep finds W^{n+1} ready and f is streamed
// once per sweep.  The Maxwellian is evaluated as rho/(2 pi theta) * ex[a] *
// ey[b] with the per-cell 1-D factors in LDS (tensor-product velocity grid),
// i.e. n1 + n2 exponentials per cell instead of n1*n2.
//
// What bounds them, 256x128 C-grid with 2304 velocities: memory (FP64 primal
// 469 us, adjoint 653 us: 5.2 and 5.5 TB/s of the rows' own bytes, against
// 5.75 and 5.82 for a stream of that mix; FP32 257 and 356 us).  States that
// fit the MALL are bound by instruction issue and, below some ten thousand
// cells, by the latency of a patch's prologue and steps (64x32 cells with 256
// velocities: 7.2 and 8.2 us; 9.7 and 12.8 us with a walk in storage order,
// FP64 neighbour rows exchanged through LDS and butterflies for the sums).  A
// software-pipelined loop (the next step's loads issued before this step's
// arithmetic) and tighter register limits measured within 1% at large sizes
// and up to 20% slower at small.

#include <math.h>

#include <algorithm>
#include <mutex>

#include "dvm_walk.h"

namespace dvm {

// ---------------------------------------------------------------------------
// FP64 moments of one cell: W (4) and the wall flux sum.  Per walk the
// sums over the grid rows of f1 w, f1 w v2, f1 w v2^2/2 + f2 w.  The same
// additions in the sweep and in k_moments, so a state loaded from a
// checkpoint continues bit for bit.
// ---------------------------------------------------------------------------
template <int V>
struct Moments {
    double A[V], B[V], C[V], F; // of this walk; wall flux sum
    double m[4];                // of the part's walks before
    double s;                   // wave totals of the parts before, moment lane / 8

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int i = 0; i < 4; i++) m[i] = 0;
        F = s = 0;
        clear();
    }
    __device__ __forceinline__ void end_part()
    {
        const double in[8] = {m[0], m[1], m[2], m[3], F, 0, 0, 0};
        s += wave_scatter8(in);
#pragma unroll
        for (int i = 0; i < 4; i++) m[i] = 0;
        F = 0;
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int v = 0; v < V; v++) A[v] = B[v] = C[v] = 0;
    }
    template <typename T>
    __device__ __forceinline__ void add(const RowFactor &rf, const Vals<T, V> &r)
    {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double f1 = (double)r.x[v], f2 = (double)r.y[v];
            A[v] = fma(rf.w, f1, A[v]);
            B[v] = fma(rf.wv, f1, B[v]);
            C[v] = fma(rf.w, f2, fma(rf.wh, f1, C[v]));
        }
    }
    // outgoing flux through the wall face (S0x, S0y)
    template <typename T>
    __device__ __forceinline__ void add_wall(const RowFactor &rf, const ColFactor *col, double S0x, double S0y,
                                             const Vals<T, V> &r)
    {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double s0 = col[v].v * S0x + rf.v * S0y;
            if (s0 > 0) F = fma(col[v].w * rf.w * (double)r.x[v], s0, F);
        }
    }
    // joins the v1 factors of this walk
    __device__ __forceinline__ void fold(const ColFactor *col)
    {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double v1 = col[v].v, w = col[v].w;
            const double wA = w * A[v];
            m[0] += wA;
            m[1] = fma(wA, v1, m[1]);
            m[2] = fma(w, B[v], m[2]);
            m[3] = fma(0.5 * v1 * v1, wA, fma(w, C[v], m[3]));
        }
        clear();
    }
    // totals over the wave, in every lane
    __device__ __forceinline__ void total(double (&o)[5])
    {
#pragma unroll
        for (int i = 0; i < 5; i++) o[i] = lane_value(s, 8 * i);
    }
};

// Part sums s of the waves that share a cell, added in part order: s of the
// first one (true) becomes the cell's.  All waves of the workgroup.
__device__ __forceinline__ bool join_parts(const DevSolve &d, const SweepUnit &u, int lane, double &s)
{
    double *x = reinterpret_cast<double *>(sweep_smem) + u.slot * u.parts * kWave + lane;
    __syncthreads();                            // the tables are done with
    x[u.p0 * kWave] = s;
    __syncthreads();
    if (u.p0 == 0)
        for (int p = 1; p < u.parts; p++) s += x[p * kWave];
    return u.p0 == 0;
}

// ---------------------------------------------------------------------------
// primal sweep of one patch: eq. (numerpr_gov), first-order upwind, Jacobi
// point-implicit: f^{n+1} = (sum_in |v.S| f_up + V g/tau) / (sum_out v.S + V/tau)
// SO (second-order scheme, defect correction): the held correction c is
// subtracted from the numerator and the wall flux is F + dF.
// NT: rows are stored (and the held correction loaded) non-temporally.
// ---------------------------------------------------------------------------
template <typename T, int V, bool SO, bool NT, bool PARTS>
__device__ __forceinline__ void primal_cell(const DevSolve &d, int par, const SweepUnit &u, bool split, int lane)
{
    const int c = u.c;
    const bool act = u.act;
    const Factors fac(d, 0);
    const GridTables gt(d);
    const GridEntry ge = gt.at(threadIdx.x), ge0 = gt.at(u.fill0);
    T *ex = static_cast<T *>(fac.end) + u.slot * (d.lm.n1p + d.lm.n2p), *ey = ex + d.lm.n1p;

    int nb[4];
    T Sx[4], Sy[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        nb[q] = uni(d.nbr[4 * c + q]);
        Sx[q] = uni((T)d.S[8 * c + 2 * q]);
        Sy[q] = uni((T)d.S[8 * c + 2 * q + 1]);
    }
    const double *Win = d.W[par] + 4 * c;
    const double W0 = uni(Win[0]), W1 = uni(Win[1]), W2 = uni(Win[2]), W3 = uni(Win[3]);
    const double ir = recip(W0), u1 = W1 * ir, u2 = W2 * ir;
    const double th = (2.0 / 3.0) * (W3 * ir - 0.5 * (u1 * u1 + u2 * u2));
    const double itau = d.inv_tau_inf * W0 * sqrt(2.0 * th);
    const double Vt = d.vol[c] * itau;
    // the equilibrium's parameters: the primitive variables, or those whose
    // grid moments equal W (found by k_eq_params before the sweep; tau keeps
    // the cell's own rho and theta)
    double Pe[4] = {W0, u1, u2, th};
    if (d.equil) {
        const double *pe = d.mstate + kEqState * c;
#pragma unroll
        for (int a = 0; a < 4; a++) Pe[a] = uni(pe[a]);
    }
    const double ith = recip(Pe[3]), h = 0.5 * ith;
    fac.fill(gt, ge);
    // Maxwellian factors: g1 = gc ex[a] ey[b]
    gt.each(u.fill0, u.fill_step, ge0, [&](int i, const GridEntry &e) {
        const double x = e.v - (e.col ? Pe[1] : Pe[2]);
        ex[i] = e.in ? (T)exp(-x * x * h) : (T)0;
    });

    const int nv = d.nv, rowb = nv * 2 * (int)sizeof(T);
    const char *fin = static_cast<const char *>(d.f[par]);
    char *fout = static_cast<char *>(d.f[par ^ 1]);
    const int wl = nb[0] <= -2 ? -2 - nb[0] : -1;
    T wcoef = 1;
    double S0x = 0, S0y = 0;
    if (wl >= 0) {
        wcoef = uni((T)((SO ? d.F[par][wl] + d.dF[wl] : d.F[par][wl]) / d.D[wl]));
        S0x = uni(d.S[8 * c]);
        S0y = uni(d.S[8 * c + 1]);
    }
    // one source row per face: the neighbour's row (a neighbour in the same
    // patch was read moments before by its own wave on this CU and is in
    // L1), the far-field table, or the wall table (g_M1, theta_w/2 g_M1)
    // scaled by F_l / D_l
    __amdgpu_buffer_rsrc_t src[4];
#pragma unroll
    for (int q = 0; q < 4; q++)
        src[q] = row_rsrc(nb[q] >= 0 ? fin + (size_t)nb[q] * rowb : static_cast<const char *>(nb[q] == -1 ? d.fd : d.gw2),
                          rowb);
    const __amdgpu_buffer_rsrc_t dst = row_rsrc(fout + (size_t)c * rowb, act ? rowb : 0);
    const __amdgpu_buffer_rsrc_t crow =
        row_rsrc(SO ? static_cast<const char *>(d.corr) + (size_t)c * rowb : nullptr, SO ? rowb : 0);
    const T th2 = uni((T)(0.5 * Pe[3])), VtT = uni((T)Vt), gc = uni((T)(Pe[0] * ith * (0.5 / kPi)));
    const int bstep = d.lm.brow * d.n1 * 2 * (int)sizeof(T);
    __syncthreads();

    Moments<V> mom;
    mom.init();
    walk_parts<PARTS>(d.lm, u.p0, u.p1, u.parts, [&](int i, int t0, int steps) {
        const Walk wk = make_walk<T, V>(d, lane, i);
        const int a = wk.a;
        const ColFactor *col = fac.col + a;
        T sx[4][V], e1[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            const T v1 = (T)col[v].v;
            e1[v] = gc * ex[a + v];
            keep(e1[v]);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                sx[q][v] = v1 * Sx[q];
                keep(sx[q][v]);
            }
        }
        int off = wk.off + t0 * bstep, b = wk.b + t0 * d.lm.brow;
        for (int t = 0; t < steps; t++, b += d.lm.brow, off += bstep) {
            const T v2 = (T)fac.row[b].v;
            T s[4][V];
            Vals<T, V> up[4], cr;
            // a face's source row only where the face is upwind (the lanes
            // of a wave split by the sign of v.S): about half the L2
            // requests of loading all four
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const T sy = v2 * Sy[q];
                bool out = true;
#pragma unroll
                for (int v = 0; v < V; v++) {
                    s[q][v] = sx[q][v] + sy;
                    out = out && s[q][v] > 0;
                }
                up[q] = row_load<T, V, false>(src[q], out ? kOutside : off);
            }
            if constexpr (SO) cr = row_load<T, V, NT>(crow, off);
            loads_first();
            const T eyb = ey[b];
            Vals<T, V> r;
#pragma unroll
            for (int v = 0; v < V; v++) {
                T out = 0, in1 = 0, in2 = 0;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    out += max0(s[q][v]);
                    const T m = min0(s[q][v]);
                    T u1 = up[q].x[v], u2 = up[q].y[v];
                    if (q == 0 && wl >= 0) {
                        u1 *= wcoef;
                        u2 *= wcoef;
                    }
                    in1 = madd(-m, u1, in1);
                    in2 = madd(-m, u2, in2);
                }
                if constexpr (SO) {
                    in1 -= cr.x[v];
                    in2 -= cr.y[v];
                }
                const T g1 = e1[v] * eyb, g2 = th2 * g1;
                const T rden = recip(out + VtT);
                r.x[v] = madd(VtT, g1, in1) * rden;
                r.y[v] = madd(VtT, g2, in2) * rden;
            }
            row_store<T, V, NT>(dst, off, r);
            const RowFactor rf = fac.row[b];
            mom.add(rf, r);
            if (wl >= 0) mom.add_wall(rf, col, S0x, S0y, r);
        }
        mom.fold(col);
    }, [&] { mom.end_part(); });
    if (PARTS && split && !join_parts(d, u, lane, mom.s)) return;
    double acc[5];
    mom.total(acc);
    if (act && lane == 0) {
        double *Wo = d.W[par ^ 1] + 4 * c;
        Wo[0] = acc[0];
        Wo[1] = acc[1];
        Wo[2] = acc[2];
        Wo[3] = acc[3];
        if (wl >= 0) d.F[par ^ 1][wl] = acc[4] / d.wall_A[wl];
        const double e0 = acc[0] - W0, e1 = acc[1] - W1, e2 = acc[2] - W2, e3 = acc[3] - W3;
        d.red[2 * c] = e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
        d.red[2 * c + 1] = W0 * W0 + W1 * W1 + W2 * W2 + W3 * W3;
    }
}

template <typename T, bool SO, bool NT, bool PARTS>
__device__ __forceinline__ void primal_unit(const DevSolve &d, int par, const SweepUnit &u, bool split)
{
    const int lane = threadIdx.x % kWave;
    if (sizeof(T) == 4 && pair_velocities<T>(d.n1))
        primal_cell<T, sizeof(T) == 4 ? 2 : 1, SO, NT, PARTS>(d, par, u, split, lane);
    else
        primal_cell<T, 1, SO, NT, PARTS>(d, par, u, split, lane);
}

// moments W and wall flux F of f[par] of a cell (no update): the walk,
// expressions and summation order of the primal sweep.  FILL: f is first set
// to the far-field Maxwellian, so only the writes touch memory (256x128 cells
// with 64x64 velocities in FP64: fill and moments 837 us as two passes, 416
// as one).
template <typename T, int V, bool FILL, bool NT>
__device__ __forceinline__ void moments_cell(const DevSolve &d, int par, int c, bool act, int lane)
{
    const Factors fac(d, 0);
    const GridTables gt(d);
    fac.fill(gt, gt.at(threadIdx.x));
    const int rowb = d.nv * 2 * (int)sizeof(T);
    const int l0 = uni(d.nbr[4 * c]);
    const int wl = l0 <= -2 ? -2 - l0 : -1;
    const double S0x = uni(d.S[8 * c]), S0y = uni(d.S[8 * c + 1]);
    char *row = static_cast<char *>(d.f[par]) + (size_t)c * rowb;
    const __amdgpu_buffer_rsrc_t src = row_rsrc(FILL ? d.fd : row, rowb), dst = row_rsrc(row, FILL && act ? rowb : 0);
    const int bstep = d.lm.brow * d.n1 * 2 * (int)sizeof(T);
    __syncthreads();
    Moments<V> mom;
    mom.init();
    walk_parts<true>(d.lm, 0, d.parts[0], d.parts[0], [&](int i, int t0, int steps) {
        const Walk wk = make_walk<T, V>(d, lane, i);
        const int a = wk.a;
        const ColFactor *col = fac.col + a;
        int off = wk.off + t0 * bstep, b = wk.b + t0 * d.lm.brow;
        for (int t = 0; t < steps; t++, b += d.lm.brow, off += bstep) {
            const RowFactor rf = fac.row[b];
            const Vals<T, V> r = row_load<T, V, false>(src, off);
            if constexpr (FILL) row_store<T, V, NT>(dst, off, r);
            mom.add(rf, r);
            if (wl >= 0) mom.add_wall(rf, col, S0x, S0y, r);
        }
        mom.fold(col);
    }, [&] { mom.end_part(); });
    double acc[5];
    mom.total(acc);
    if (act && lane == 0) {
        double *Wo = d.W[par] + 4 * c;
        Wo[0] = acc[0];
        Wo[1] = acc[1];
        Wo[2] = acc[2];
        Wo[3] = acc[3];
        if (wl >= 0) d.F[par][wl] = acc[4] / d.wall_A[wl];
    }
}

// ---------------------------------------------------------------------------
// FP64 adjoint moments of phi (eqs. adjoint_macdefines, formula_adjointbgk)
// of one cell: phi . dg/dP for P = (rho, u1, u2, theta) from
// A0 = sum w g1 qq, A1 = sum w g1 c1 qq, A2, A3 = sum w g1 |c|^2 qq and
// A4 = sum w g1 phi2 (qq = phi1 + theta/2 phi2, c = v - u); the rho_tau sum
// T = sum w (phi . (g - f)); the wall multiplier sum Pw over the wall face's
// incoming velocities.  Per walk the sums over the grid rows carry w Y c2^p
// (AdjRow) and R = sum w phi . f; the factors w gc X(v1), c1 join once per
// walk.  T takes the difference of A0 and R there, lane by lane: g and f nearly
// cancel near the continuum, and the cells' totals subtracted at the end lose
// twice the rounding (relative to A0 1.4e-16 against 0.8e-16).  Shared by the
// adjoint sweep's epilogue and k_adjoint_moments, so both give the same bits.
// ---------------------------------------------------------------------------
// Per-cell constants: the frozen velocity u1, theta/2, theta_w/2, the wall
// face vector and wall element (-1: none), objective.
struct AdjCell {
    double u1, hth, thw2, S0x, S0y;
    int wl, obj;
};

template <int V>
struct AdjMoments {
    double Q[V], Qc[V], Qcc[V], E[V], R[V], Pw; // of this walk; wall multiplier sum
    WalkSums m;                                 // of the part's walks before (6)
    double s;                                   // wave totals of the parts before, sum lane / 8

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int i = 0; i < 6; i++) m[i] = 0;
        Pw = s = 0;
        clear();
    }
    __device__ __forceinline__ void end_part()
    {
        const double in[8] = {m[0], m[1], m[2], m[3], m[4], m[5], Pw, 0};
        s += wave_scatter8(in);
#pragma unroll
        for (int i = 0; i < 6; i++) m[i] = 0;
        Pw = 0;
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int v = 0; v < V; v++) Q[v] = Qc[v] = Qcc[v] = E[v] = R[v] = 0;
    }
    template <typename T>
    __device__ __forceinline__ void add(const AdjCell &q, const AdjRow &ar, double w, const Vals<T, V> &r,
                                        const Vals<T, V> &fs)
    {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double p1 = (double)r.x[v], p2 = (double)r.y[v];
            const double qq = fma(q.hth, p2, p1);
            Q[v] = fma(ar.e, qq, Q[v]);
            Qc[v] = fma(ar.ec, qq, Qc[v]);
            Qcc[v] = fma(ar.ecc, qq, Qcc[v]);
            E[v] = fma(ar.e, p2, E[v]);
            R[v] = fma(w, fma(p1, (double)fs.x[v], p2 * (double)fs.y[v]), R[v]);
        }
    }
    // incoming velocities of the wall face; gM: g_M1(1, 0, theta_w) of the V velocities
    template <typename T>
    __device__ __forceinline__ void add_wall(const AdjCell &q, const RowFactor &rf, const ColFactor *col,
                                             const Vals<T, V> &r, const T *__restrict__ gM, bool in)
    {
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double s0 = col[v].v * q.S0x + rf.v * q.S0y;
            if (in && s0 <= 0)
                Pw += col[v].w * rf.w * s0 * (double)gM[v] *
                      (((double)r.x[v] + mJ_of(q.obj, col[v].v, rf.v)) + q.thw2 * (double)r.y[v]);
        }
    }
    // joins the v1 factors of this walk (gx: w gc X of the V columns)
    __device__ __forceinline__ void fold(const AdjCell &q, const ColFactor *col, const double *gx)
    {
        double t[6];
#pragma unroll
        for (int i = 0; i < 6; i++) t[i] = m[i];
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double g = gx[v], c1 = col[v].v - q.u1;
            const double gQ = g * Q[v];
            t[0] += gQ;
            t[1] = fma(gQ, c1, t[1]);
            t[2] = fma(g, Qc[v], t[2]);
            t[3] = fma(gQ, c1 * c1, fma(g, Qcc[v], t[3]));
            t[4] = fma(g, E[v], t[4]);
            t[5] += fma(-col[v].w, R[v], gQ);
        }
#pragma unroll
        for (int i = 0; i < 6; i++) m[i] = t[i];
        clear();
    }
    // totals: A0..A4, T, Pw
    __device__ __forceinline__ void total(double (&o)[7])
    {
#pragma unroll
        for (int i = 0; i < 7; i++) o[i] = lane_value(s, 8 * i);
    }
};

// dP/dW of the cell (P = the equilibrium's (rho, u1, u2, theta)) for
// adjoint_store: entry `lane` of the row-major 4x4 in lanes 0 .. 15, loaded
// ahead of the sums
__device__ __forceinline__ double adjoint_jacobian(const double *ac, int lane) { return ac[16 + (lane & 15)]; }

// The wave's totals -> What (4) and rho_tau of the cell (ao[0..4]) and the
// wall multiplier Phi_l of its wall element.
__device__ __forceinline__ void adjoint_store(const DevSolve &d, double rho, double th, double itau, double M, bool act,
                                              int lane, int wl, const double (&acc)[7], double *ao, double *Phi)
{
    const double ith = recip(th);
    // phi . dg/dP
    const double P0 = acc[0] * recip(rho), P1 = acc[1] * ith, P2 = acc[2] * ith;
    const double P3 = 0.5 * acc[3] * (ith * ith) - acc[0] * ith + 0.5 * acc[4];
    // What_m = sum_q (phi . dg/dP_q) dP_q/dW_m: lane 4 q + m, summed over q
    const int q = (lane >> 2) & 3;
    double s = (q < 2 ? (q == 0 ? P0 : P1) : (q == 2 ? P2 : P3)) * M;
    s += dpp_move<0x128>(s);                                    // lane ^ 8
    s += dpp_move<0x124>(s);                                    // lane - 4 in the row of 16
    if (lane == 4) s = acc[5] * itau;
    if (act && lane < 5) ao[lane] = s;
    if (act && wl >= 0 && lane == 0) Phi[wl] = -acc[6] / (d.wall_A[wl] * d.D[wl]);
}

// ---------------------------------------------------------------------------
// adjoint sweep of one patch: eq. (numerad_gov) with the wall and far-field
// conditions of eq. (formula_adjointbgk), Jacobi point-implicit:
// phi^{n+1} = (sum_out v.S phi_down + V (phi_eq/tau + phi_tau)) / (sum_out v.S + V/tau)
// Epilogue: What (eq. adjoint_macdefines, via primitive variables),
// rho_tau, the wall multiplier Phi_l and (RES) the residual partials of
// phi^{n+1}.  SO (second-order scheme): the held reconstruction term E is
// subtracted from the numerator.  NT: rows only this cell touches are loaded
// and stored non-temporally.
// ---------------------------------------------------------------------------
template <typename T, int V, bool SO, bool NT, bool RES, bool PARTS>
__device__ __forceinline__ void adjoint_cell(const DevSolve &d, int par, const SweepUnit &u, bool split, int lane)
{
    const int c = u.c;
    const bool act = u.act;
    const AdjLds<T> sm(d, u.slot);
    const GridTables gt(d);
    const GridEntry ge = gt.at(threadIdx.x), ge0 = gt.at(u.fill0);
    int nb[4];
    T Sx[4], Sy[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        nb[q] = uni(d.nbr[4 * c + q]);
        Sx[q] = uni((T)d.S[8 * c + 2 * q]);
        Sy[q] = uni((T)d.S[8 * c + 2 * q + 1]);
    }
    const double *ac = d.acoef + kAcoef * c;
    const double rho = uni(ac[0]), th = uni(ac[3]), itau = uni(ac[4]), Vv = uni(d.vol[c]);
    const double M = adjoint_jacobian(ac, lane);
    const double *aw = d.aW[par] + 8 * c;
    const double rt = uni(aw[4]);
    // source V (phi_eq / tau + phi_tau) = V (C0 + C1 v1 + C2 v2 + C3 |v|^2/2)
    // (first), V C3 (second): in FP64 with V folded in, as a part in v1 and a
    // part in v2 (qb); in FP32 qb = C2 v2
    constexpr bool kFold = sizeof(T) == 8;
    double C[4];
#pragma unroll
    for (int m = 0; m < 4; m++) C[m] = uni(aw[m]) * itau - rt * uni(ac[6 + m]);
    const T VT = uni((T)Vv), Ct1 = uni((T)C[1]), Ct2 = uni((T)C[2]), Ct3 = uni((T)C[3]);
    sm.fac.fill(gt, ge);
    sm.fill(gt, ge0, ac, u.fill0, u.fill_step, [&](int k, double v2) {
        sm.qb[k] = kFold ? (T)(Vv * v2 * fma(0.5 * C[3], v2, C[2])) : Ct2 * (T)v2;
    });

    const int nv = d.nv, rowb = nv * 2 * (int)sizeof(T);
    const char *pin = static_cast<const char *>(d.phi[par]);
    __amdgpu_buffer_rsrc_t src[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        // downstream row; nothing (zero) behind a boundary face
        src[q] = row_rsrc(pin + (size_t)(nb[q] >= 0 ? nb[q] : c) * rowb, nb[q] >= 0 ? rowb : 0);
    }
    const int wl = nb[0] <= -2 ? -2 - nb[0] : -1;
    T Phi_w = 0;
    double S0x = 0, S0y = 0;
    if (wl >= 0) {
        Phi_w = uni((T)d.Phi[par][wl]);
        S0x = uni(d.S[8 * c]);
        S0y = uni(d.S[8 * c + 1]);
    }
    const T *__restrict__ gM = static_cast<const T *>(d.gM);
    const __amdgpu_buffer_rsrc_t own = row_rsrc(pin + (size_t)c * rowb, rowb);
    const __amdgpu_buffer_rsrc_t fst = row_rsrc(static_cast<const char *>(d.fstar) + (size_t)c * rowb, rowb);
    const __amdgpu_buffer_rsrc_t erow =
        row_rsrc(SO ? static_cast<const char *>(d.corr) + (size_t)c * rowb : nullptr, SO ? rowb : 0);
    const __amdgpu_buffer_rsrc_t dst = row_rsrc(static_cast<char *>(d.phi[par ^ 1]) + (size_t)c * rowb, act ? rowb : 0);
    const T den0 = uni((T)(Vv * itau)), src2 = VT * Ct3;
    const AdjCell cq = {uni(ac[1]), 0.5 * uni(ac[3]), 0.5 * d.theta_w, S0x, S0y, wl, d.objective};
    const int bstep = d.lm.brow * d.n1 * 2 * (int)sizeof(T);
    __syncthreads();

    AdjMoments<V> mom;
    mom.init();
    double dn = 0, dd = 0, rs[2] = {0, 0};
    walk_parts<PARTS>(d.lm, u.p0, u.p1, u.parts, [&](int i, int t0, int steps) {
        const Walk wk = make_walk<T, V>(d, lane, i);
        const int a = wk.a;
        const ColFactor *col = sm.fac.col + a;
        T sx[4][V], s1[V], v1h[V];
        double dnb[V], ddb[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double v1 = col[v].v;
            s1[v] = kFold ? (T)(Vv * fma(fma(0.5 * C[3], v1, C[1]), v1, C[0])) : (T)C[0] + Ct1 * (T)v1;
            keep(s1[v]);
            v1h[v] = (T)v1 * (T)v1;
            if (!kFold) keep(v1h[v]);
            dnb[v] = ddb[v] = 0;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                sx[q][v] = (T)v1 * Sx[q];
                keep(sx[q][v]);
            }
        }
        int off = wk.off + t0 * bstep, b = wk.b + t0 * d.lm.brow;
        for (int t = 0; t < steps; t++, b += d.lm.brow, off += bstep) {
            const T v2 = (T)sm.fac.row[b].v;
            T s[4][V];
            Vals<T, V> dwn[4], old, fs, e;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const T sy = v2 * Sy[q];
                bool in = true;
#pragma unroll
                for (int v = 0; v < V; v++) {
                    s[q][v] = sx[q][v] + sy;
                    in = in && !(s[q][v] > 0);
                }
                dwn[q] = row_load<T, V, false>(src[q], in ? kOutside : off);
            }
            fs = row_load<T, V, NT>(fst, off);
            if constexpr (RES) old = row_load<T, V, false>(own, off);
            if constexpr (SO) e = row_load<T, V, NT>(erow, off);
            loads_first();
            const T qb = sm.qb[b], v2h = v2 * v2;
            Vals<T, V> r;
#pragma unroll
            for (int v = 0; v < V; v++) {
                T out = 0, a1 = 0, a2 = 0;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const T m = max0(s[q][v]);
                    out += m;
                    T d1 = dwn[q].x[v];
                    if (q == 0 && wl >= 0) d1 = Phi_w - (T)mJ_of(cq.obj, col[v].v, sm.fac.row[b].v);
                    a1 = madd(m, d1, a1);
                    a2 = madd(m, dwn[q].y[v], a2);
                }
                if constexpr (SO) {
                    a1 -= e.x[v];
                    a2 -= e.y[v];
                }
                T src1;
                if constexpr (sizeof(T) == 8)
                    src1 = s1[v] + qb;                  // V included
                else
                    src1 = VT * ((s1[v] + qb) + Ct3 * (0.5f * (v1h[v] + v2h)));
                const T rden = recip(out + den0);
                r.x[v] = (a1 + src1) * rden;
                r.y[v] = (a2 + src2) * rden;
            }
            row_store<T, V, NT>(dst, off, r);
            const double w = sm.fac.row[b].w;
            mom.add(cq, sm.adj[b], w, r, fs);
            if (wl >= 0) mom.add_wall(cq, sm.fac.row[b], col, r, gM + b * d.n1 + a, wk.in && b < d.n2);
            if constexpr (RES) {
#pragma unroll
                for (int v = 0; v < V; v++) {
                    const double p1 = (double)r.x[v], p2 = (double)r.y[v];
                    const double e1 = p1 - (double)old.x[v], e2 = p2 - (double)old.y[v];
                    dnb[v] = fma(w, fma(e1, e1, e2 * e2), dnb[v]);
                    ddb[v] = fma(w, fma(p1, p1, p2 * p2), ddb[v]);
                }
            }
        }
        mom.fold(cq, col, sm.gx + a);
        if constexpr (RES) {
#pragma unroll
            for (int v = 0; v < V; v++) {
                dn = fma(col[v].w, dnb[v], dn);
                dd = fma(col[v].w, ddb[v], dd);
            }
        }
    }, [&] {
        mom.end_part();
        if constexpr (RES) {
            double x[2] = {dn, dd};
            wave_sum<2>(x);
            rs[0] += x[0];
            rs[1] += x[1];
            dn = dd = 0;
        }
    });
    if (PARTS && split) {
        if constexpr (RES) {
            join_parts(d, u, lane, rs[0]);
            join_parts(d, u, lane, rs[1]);
        }
        if (!join_parts(d, u, lane, mom.s)) return;
    }
    double acc[7];
    mom.total(acc);
    if constexpr (RES) {
        if (act && lane == 0) {
            d.red[2 * c] = rs[0];
            d.red[2 * c + 1] = rs[1];
        }
    }
    adjoint_store(d, rho, th, itau, M, act, lane, wl, acc, d.aW[par ^ 1] + 8 * c, d.Phi[par ^ 1]);
}

template <typename T, bool SO, bool NT, bool RES, bool PARTS>
__device__ __forceinline__ void adjoint_unit(const DevSolve &d, int par, const SweepUnit &u, bool split)
{
    const int lane = threadIdx.x % kWave;
    if (sizeof(T) == 4 && pair_velocities<T>(d.n1))
        adjoint_cell<T, sizeof(T) == 4 ? 2 : 1, SO, NT, RES, PARTS>(d, par, u, split, lane);
    else
        adjoint_cell<T, 1, SO, NT, RES, PARTS>(d, par, u, split, lane);
}

// Adjoint moments What, rho_tau and wall multipliers Phi_l of phi[par] with
// no update (a loaded phi): the walk, expressions and summation order of the
// adjoint sweep's epilogue, so the next sweep sees what a sweep that had
// produced this phi would have left.  CORR: phi is first corrected in place
// by the collision invariant -(z . Psi, z_3) of the adjoint prediction
// (z [nc][4]), and the moments are those of the result; its rows bypass the
// memory-side cache whatever the sweeps' rule (sweep_memory).
template <typename T, int V, bool CORR>
__device__ __forceinline__ void adjoint_moments_cell(const DevSolve &d, int par, const double *z, int c, bool act, int w,
                                                     int lane)
{
    const AdjLds<T> sm(d, w);
    const GridTables gt(d);
    sm.fac.fill(gt, gt.at(threadIdx.x));
    const double *ac = d.acoef + kAcoef * c;
    sm.fill(gt, ac, lane);
    const double rho = uni(ac[0]), th = uni(ac[3]), itau = uni(ac[4]);
    const double M = adjoint_jacobian(ac, lane);
    const T *__restrict__ gM = static_cast<const T *>(d.gM);
    const int l0 = uni(d.nbr[4 * c]);
    const int wl = l0 <= -2 ? -2 - l0 : -1;
    const int rowb = d.nv * 2 * (int)sizeof(T);
    const AdjCell cq = {uni(ac[1]), 0.5 * uni(ac[3]), 0.5 * d.theta_w, uni(d.S[8 * c]), uni(d.S[8 * c + 1]), wl, d.objective};
    const __amdgpu_buffer_rsrc_t prow = row_rsrc(static_cast<const char *>(d.phi[par]) + (size_t)c * rowb, rowb);
    const __amdgpu_buffer_rsrc_t dst = row_rsrc(static_cast<char *>(d.phi[par]) + (size_t)c * rowb, act ? rowb : 0);
    const __amdgpu_buffer_rsrc_t fst = row_rsrc(static_cast<const char *>(d.fstar) + (size_t)c * rowb, rowb);
    const int bstep = d.lm.brow * d.n1 * 2 * (int)sizeof(T);
    double zc[4] = {0, 0, 0, 0};
    if constexpr (CORR) {
#pragma unroll
        for (int i = 0; i < 4; i++) zc[i] = uni(z[4 * c + i]);
    }
    __syncthreads();
    AdjMoments<V> mom;
    mom.init();
    walk_parts<true>(d.lm, 0, d.parts[1], d.parts[1], [&](int i, int t0, int steps) {
        const Walk wk = make_walk<T, V>(d, lane, i);
        const int a = wk.a;
        const ColFactor *col = sm.fac.col + a;
        double z1[V];
#pragma unroll
        for (int v = 0; v < V; v++) z1[v] = fma(fma(0.5 * zc[3], col[v].v, zc[1]), col[v].v, zc[0]);
        int off = wk.off + t0 * bstep, b = wk.b + t0 * d.lm.brow;
        for (int t = 0; t < steps; t++, b += d.lm.brow, off += bstep) {
            const RowFactor rf = sm.fac.row[b];
            Vals<T, V> r = row_load<T, V, false>(prow, off);
            const Vals<T, V> fs = row_load<T, V, true>(fst, off);
            if constexpr (CORR) {
                const double z2 = rf.v * fma(0.5 * zc[3], rf.v, zc[2]);
#pragma unroll
                for (int v = 0; v < V; v++) {
                    r.x[v] = (T)((double)r.x[v] - (z1[v] + z2));
                    r.y[v] = (T)((double)r.y[v] - zc[3]);
                }
                row_store<T, V, true>(dst, off, r);
            }
            mom.add(cq, sm.adj[b], rf.w, r, fs);
            if (wl >= 0) mom.add_wall(cq, rf, col, r, gM + b * d.n1 + a, wk.in && b < d.n2);
        }
        mom.fold(cq, col, sm.gx + a);
    }, [&] { mom.end_part(); });
    double acc[7];
    mom.total(acc);
    adjoint_store(d, rho, th, itau, M, act, lane, wl, acc, d.aW[par] + 8 * c, d.Phi[par]);
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
constexpr int kPatchBlock = kPatchCells * kWave;   // threads of a patch workgroup

// Workgroup b of a sweep (phase 0 primal, 1 adjoint): each XCD takes its
// stretch of patches (from its end: rev), the last `tail` of them in parts.
// Returns the patch, -1 for padding; k: which of the patch's workgroups, -1 for
// the only one.
template <bool PARTS>
__device__ __forceinline__ int sweep_patch(const DevSolve &d, int phase, int b, int rev, int &k)
{
    k = -1;
    if constexpr (!PARTS) return xcd_item(d.np, b, rev);
    const int per = (d.np + 7) >> 3, parts = d.parts[phase], whole = per - d.tail[phase];
    int j = b >> 3;
    if (j >= whole) {
        k = (j - whole) & (parts - 1);
        j = whole + ((j - whole) >> (parts >> 1));   // parts: 2 or 4
    }
    const int p = (b & 7) * per + (rev ? per - 1 - j : j);
    return p < d.np ? p : -1;
}
template <bool PARTS>
__device__ __forceinline__ SweepUnit sweep_unit(const DevSolve &d, int phase, int p, int k)
{
    return !PARTS || k < 0 ? patch_unit(d, p, d.parts[phase]) : part_unit(d, p, k, d.parts[phase]);
}
static inline int sweep_grid(const DevSolve &d, int phase)
{
    return 8 * ((d.np + 7) / 8 + d.tail[phase] * (d.parts[phase] - 1));
}

template <typename T, bool SO, bool NT, bool PARTS>
__global__ __launch_bounds__(kPatchBlock) void k_primal_sweep(DevSolve d, int par, int rev)
{
    int k;
    const int p = sweep_patch<PARTS>(d, 0, blockIdx.x, rev, k);
    if (p < 0) return;
    primal_unit<T, SO, NT, PARTS>(d, par, sweep_unit<PARTS>(d, 0, p, k), k >= 0);
}

template <typename T, bool FILL, bool NT>
__global__ __launch_bounds__(kPatchBlock) void k_moments(DevSolve d, int par)
{
    const int p = xcd_item(d.np, blockIdx.x);
    if (p < 0) return;
    int w;
    bool act;
    const int c = patch_wave(d, p, w, act), lane = threadIdx.x % kWave;
    if (sizeof(T) == 4 && pair_velocities<T>(d.n1))
        moments_cell<T, sizeof(T) == 4 ? 2 : 1, FILL, NT>(d, par, c, act, lane);
    else
        moments_cell<T, 1, FILL, NT>(d, par, c, act, lane);
}

template <typename T, bool SO, bool NT, bool RES, bool PARTS>
__global__ __launch_bounds__(kPatchBlock) void k_adjoint_sweep(DevSolve d, int par, int rev)
{
    int k;
    const int p = sweep_patch<PARTS>(d, 1, blockIdx.x, rev, k);
    if (p < 0) return;
    adjoint_unit<T, SO, NT, RES, PARTS>(d, par, sweep_unit<PARTS>(d, 1, p, k), k >= 0);
}

// adjoint moments of phi[par]; CORR: corrected by z first
template <typename T, bool CORR>
__global__ __launch_bounds__(kPatchBlock) void k_adjoint_moments(DevSolve d, int par, const double *z)
{
    const int p = xcd_item(d.np, blockIdx.x);
    if (p < 0) return;
    int w;
    bool act;
    const int c = patch_wave(d, p, w, act), lane = threadIdx.x % kWave;
    if (sizeof(T) == 4 && pair_velocities<T>(d.n1))
        adjoint_moments_cell<T, sizeof(T) == 4 ? 2 : 1, CORR>(d, par, z, c, act, w, lane);
    else
        adjoint_moments_cell<T, 1, CORR>(d, par, z, c, act, w, lane);
}

// one sweep of the primal-phase (or adjoint-phase) members of a batch that
// run one scheme (SO: second order, the held corrections evaluated before
// the launch); a workgroup owns one (solve, patch).  Phases and schemes are
// separate kernels so that each gets the occupancy of its own registers.
template <typename T, bool SO, bool NT, bool PARTS>
__global__ __launch_bounds__(kPatchBlock) void k_batch_primal(const DevSolve *__restrict__ tab,
                                                              const int32_t *__restrict__ blk_solve,
                                                              const int32_t *__restrict__ blk_patch,
                                                              const int32_t *__restrict__ par0, int step, int rev)
{
    // rev: each XCD's column from its end
    const int b = rev ? (int)(gridDim.x - 8 - blockIdx.x) + 2 * (int)(blockIdx.x & 7) : (int)blockIdx.x;
    const int s = blk_solve[b];
    if (s < 0) return;
    primal_unit<T, SO, NT, PARTS>(tab[s], (par0[s] + step) & 1, patch_unit(tab[s], blk_patch[b], tab[s].parts[0]), false);
}

template <typename T, bool SO, bool NT, bool RES, bool PARTS>
__global__ __launch_bounds__(kPatchBlock) void k_batch_adjoint(const DevSolve *__restrict__ tab,
                                                               const int32_t *__restrict__ blk_solve,
                                                               const int32_t *__restrict__ blk_patch,
                                                               const int32_t *__restrict__ par0, int step, int rev)
{
    // rev: each XCD's column from its end
    const int b = rev ? (int)(gridDim.x - 8 - blockIdx.x) + 2 * (int)(blockIdx.x & 7) : (int)blockIdx.x;
    const int s = blk_solve[b];
    if (s < 0) return;
    adjoint_unit<T, SO, NT, RES, PARTS>(tab[s], (par0[s] + step) & 1, patch_unit(tab[s], blk_patch[b], tab[s].parts[1]), false);
}

// Block tables of a batch on the device (the allocation-free batch): block
// b of group g runs on XCD x = b % 8 and is the (b / 8)-th slot of that
// XCD's column, which holds, member after member of the group in table
// order, the x-th eighth of each member's patches (ceil(np / 8) of them, the
// last eighth possibly shorter); slots past the last member are padding (-1).
// The same map as the host-built one of dvm_batch_create.
struct BatchGroups {
    int nb[4];
};

__global__ __launch_bounds__(kBlock) void k_batch_tables(const DevSolve *__restrict__ tab,
                                                         const int32_t *__restrict__ phase, int n, BatchGroups grp,
                                                         int32_t *__restrict__ blk_solve,
                                                         int32_t *__restrict__ blk_patch)
{
    const int total = grp.nb[0] + grp.nb[1] + grp.nb[2] + grp.nb[3];
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= total) return;
    int g = 0, local = b;
    while (local >= grp.nb[g]) {
        local -= grp.nb[g];
        g++;
    }
    const int x = local & 7;
    int slot = local >> 3, solve = -1, patch = 0;
    for (int i = 0; i < n; i++) {
        if (2 * phase[i] + (tab[i].order == 2 ? 1 : 0) != g) continue;
        const int np = tab[i].np, per = (np + 7) / 8;
        const int p0 = x * per, cnt = max(0, min(np, p0 + per) - p0);
        if (slot < cnt) {
            solve = i;
            patch = p0 + slot;
            break;
        }
        slot -= cnt;
    }
    blk_solve[b] = solve;
    blk_patch[b] = solve >= 0 ? patch : 0;
}

// The fixed device array of the allocation-free batch (one per GPU the
// library runs on; held until the process ends).  Host code reaches it only
// through the address static_batch_scratch looks up for the current device.
static __device__ __align__(256) unsigned char scratch[kStaticBatchBytes];

hipError_t static_batch_scratch(char **out)
{
    constexpr int kMaxDevices = 64;
    static char *addr[kMaxDevices] = {};
    static std::mutex mu;
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) return e;
        addr[dev] = static_cast<char *>(p);
    }
    *out = addr[dev];
    return hipSuccess;
}

template <typename T>
__global__ void k_zero(T *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = (T)0;
}

// per-cell adjoint coefficients from the frozen moments, one thread per cell
// (the conservative equilibrium's parameters and dP'/dW from mstate, where
// k_eq_params has left them):
// ac[0..3] the equilibrium's (rho, u1, u2, theta), ac[4] 1/tau (the cell's
// own rho, theta), ac[5] rho/(2 pi theta) of the equilibrium, ac[6..9]
// (1/tau) dtau/dW, ac[16..31] dP/dW (row = parameter, column = moment)
__global__ __launch_bounds__(kWave) void k_adjoint_coef(DevSolve d, const double *Wst)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= d.nc) return;
    const double *W = Wst + 4 * c;
    const double rho = W[0], u1 = W[1] / rho, u2 = W[2] / rho, E = W[3] / rho;
    const double th = (2.0 / 3.0) * (E - 0.5 * (u1 * u1 + u2 * u2));
    const double itau = d.inv_tau_inf * rho * sqrt(2.0 * th);
    const double ir = 1.0 / rho, k23 = 2.0 / 3.0;
    // d theta / dW of the cell's own primitive variables
    const double dth0 = k23 * (u1 * u1 + u2 * u2 - E) * ir, dth1 = -k23 * u1 * ir, dth2 = -k23 * u2 * ir,
                 dth3 = k23 * ir;
    double P[4] = {rho, u1, u2, th}, M[16];
    if (d.equil) {
        const double *ms = d.mstate + kEqState * c;
#pragma unroll
        for (int q = 0; q < 4; q++) P[q] = ms[q];
#pragma unroll
        for (int q = 0; q < 16; q++) M[q] = ms[4 + q];
    } else {
        const double J[16] = {1.0, 0.0, 0.0, 0.0, -u1 * ir, ir, 0.0, 0.0, -u2 * ir, 0.0, ir, 0.0,
                              dth0, dth1, dth2, dth3};
#pragma unroll
        for (int q = 0; q < 16; q++) M[q] = J[q];
    }
    double *ac = d.acoef + kAcoef * c;
    ac[0] = P[0];
    ac[1] = P[1];
    ac[2] = P[2];
    ac[3] = P[3];
    ac[4] = itau;
    ac[5] = P[0] / (2.0 * kPi * P[3]);
    // (1/tau) dtau/dW, tau ~ 1 / (rho sqrt(theta)) (hard sphere)
    const double h = 0.5 / th;
    ac[6] = -ir - h * dth0;
    ac[7] = -h * dth1;
    ac[8] = -h * dth2;
    ac[9] = -h * dth3;
    ac[10] = E;
    for (int q = 11; q < 16; q++) ac[q] = 0.0;
    for (int q = 0; q < 16; q++) ac[16 + q] = M[q];
}

// Phi_l of phi = 0 (only the objective's m_J term): one block per element
template <typename T>
__global__ __launch_bounds__(kBlock) void k_wall_phi0(DevSolve d, int par)
{
    __shared__ double red[4 * 1];
    const int l = blockIdx.x;
    const T *gM = static_cast<const T *>(d.gM);
    const double n1 = d.wall_n[2 * l], n2 = d.wall_n[2 * l + 1];
    double s = 0;
    for (int k = threadIdx.x; k < d.nv; k += kBlock) {
        const double v1 = d.vx[k % d.n1], v2 = d.vy[k / d.n1];
        const double vn = v1 * n1 + v2 * n2;
        if (vn <= 0) s += d.wx[k % d.n1] * d.wy[k / d.n1] * vn * mJ_of(d.objective, v1, v2) * (double)gM[k];
    }
    double acc[1] = {s};
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) d.Phi[par][l] = -acc[0] / d.D[l];
}

// deterministic sum of the per-cell residual partials: out[0..1].  One
// workgroup reads them all (16 bytes a cell, 0.5 MB at 32768 cells), so what
// counts is how many loads it keeps in flight: 1024 threads with four each
// 57 -> 9 us, 256 threads with one at a time before.
constexpr int kResBlock = 1024;

__device__ __forceinline__ void residual_sum(const double *red, int nc, double *out)
{
    __shared__ double lds[2 * (kResBlock / kWave)];
    const double2 *r = reinterpret_cast<const double2 *>(red);
    double acc[2] = {0, 0};
    for (int c = threadIdx.x; c < nc; c += 4 * kResBlock) {
        double2 v[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int i = c + k * kResBlock;
            v[k] = i < nc ? r[i] : double2{0, 0};
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            acc[0] += v[k].x;
            acc[1] += v[k].y;
        }
    }
    wave_sum<2>(acc);
    const int lane = threadIdx.x % kWave, w = (int)(threadIdx.x / kWave);
    if (lane == 0) {
        lds[2 * w] = acc[0];
        lds[2 * w + 1] = acc[1];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0;
        for (int k = 0; k < kResBlock / kWave; k++) s += lds[2 * k + threadIdx.x];
        out[threadIdx.x] = s;
    }
}

__global__ __launch_bounds__(kResBlock) void k_residual(const double *red, int nc, double *out)
{
    residual_sum(red, nc, out);
}

__global__ __launch_bounds__(kResBlock) void k_batch_residual(const DevSolve *tab, double *out)
{
    const DevSolve &d = tab[blockIdx.x];
    residual_sum(d.red, d.nc, out + 2 * blockIdx.x);
}

// J_l = A_l sum_k w m_J (v.n) f1_{l,k}, eq. (numer_J): one block per element
template <typename T>
__global__ __launch_bounds__(kBlock) void k_objective_elem(DevSolve d, int par)
{
    using T2 = typename Vec2<T>::type;
    __shared__ double red[4];
    const int l = blockIdx.x;
    const int c = d.wall_cell[l];
    const T2 *f = static_cast<const T2 *>(d.f[par]);
    const T *gM = static_cast<const T *>(d.gM);
    const double n1 = d.wall_n[2 * l], n2 = d.wall_n[2 * l + 1];
    const double FD = d.F[par][l] / d.D[l];
    double s = 0;
    for (int k = threadIdx.x; k < d.nv; k += kBlock) {
        const int a = k % d.n1, b = k / d.n1;
        const double v1 = d.vx[a], v2 = d.vy[b];
        const double vn = v1 * n1 + v2 * n2;
        const double f1 = vn > 0 ? (double)f[(size_t)c * d.nv + k].x : FD * (double)gM[k];
        s += d.wx[a] * d.wy[b] * mJ_of(d.objective, v1, v2) * vn * f1;
    }
    double acc[1] = {s};
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) d.Jl[l] = d.wall_A[l] * acc[0];
}

__global__ __launch_bounds__(kBlock) void k_objective_sum(DevSolve d)
{
    __shared__ double red[4];
    double s = 0;
    for (int l = threadIdx.x; l < d.nw; l += kBlock) s += d.Jl[l];
    double acc[1] = {s};
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) {
        d.out[0] = acc[0];
        d.out[1] = acc[0] / d.cd_scale;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline int ew_grid(size_t n) { return (int)std::min<size_t>((n + kBlock - 1) / kBlock, 8192); }

// f = far-field Maxwellian in every cell, with its moments and wall fluxes
hipError_t launch_primal_init(const DevSolve &d, hipStream_t st)
{
    DVM_FLAG(d.mem[0] == kMemStream, NT, DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_moments<T, true, NT>), dim3(xcd_grid(d.np)),
                                                                   dim3(kPatchBlock), factor_lds(d.lm), st, d, 0)));
    return hipGetLastError();
}

hipError_t launch_moments(const DevSolve &d, int par, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_moments<T, false, false>), dim3(xcd_grid(d.np)), dim3(kPatchBlock), factor_lds(d.lm), st,
                                             d, par));
    return hipGetLastError();
}

hipError_t launch_primal_sweep(const DevSolve &d, int par, hipStream_t st)
{
    const int rev = d.mem[0] == kMemTurn ? par & 1 : 0;
    DVM_FLAG(d.order == 2, SO, DVM_FLAG(d.mem[0] == kMemStream, NT, DVM_FLAG(d.parts[0] > 1, PARTS, DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(
        (k_primal_sweep<T, SO, NT, PARTS>), dim3(sweep_grid(d, 0)), dim3(kPatchBlock), primal_lds(d), st, d, par, rev)))));
    return hipGetLastError();
}

hipError_t launch_residual(const DevSolve &d, int adjoint, hipStream_t st)
{
    hipLaunchKernelGGL(k_residual, dim3(1), dim3(kResBlock), 0, st, d.red, d.nc, d.out + (adjoint ? 4 : 2));
    return hipGetLastError();
}

hipError_t launch_objective(const DevSolve &d, int par, hipStream_t st)
{
    if (d.order == 2) {
        if (hipError_t e = launch_so_objective_elem(d, par, st)) return e;
    } else {
        DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_objective_elem<T>, dim3(d.nw), dim3(kBlock), 0, st, d, par));
        if (hipError_t e = hipGetLastError()) return e;
    }
    hipLaunchKernelGGL(k_objective_sum, dim3(1), dim3(kBlock), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_adjoint_init(const DevSolve &d, int fpar, hipStream_t st)
{
    if (d.equil)
        if (hipError_t e = launch_eq_params(d, fpar, 1, st)) return e;
    hipLaunchKernelGGL(k_adjoint_coef, dim3((d.nc + kWave - 1) / kWave), dim3(kWave), 0, st, d, d.W[fpar]);
    if (hipError_t e = hipGetLastError()) return e;
    const size_t n = (size_t)d.nc * d.nv * 2;
    if (d.mixed)
        hipLaunchKernelGGL(k_zero<float>, dim3(ew_grid(n)), dim3(kBlock), 0, st, static_cast<float *>(d.phi[0]), n);
    else
        hipLaunchKernelGGL(k_zero<double>, dim3(ew_grid(n)), dim3(kBlock), 0, st, static_cast<double *>(d.phi[0]), n);
    if (hipError_t e = hipGetLastError()) return e;
    // both ping-pong buffers: slots 5..7 of each cell are padding that the
    // sweep never writes, and checkpoints copy them
    for (int p = 0; p < 2; p++) {
        hipLaunchKernelGGL(k_zero<double>, dim3(ew_grid((size_t)8 * d.nc)), dim3(kBlock), 0, st, d.aW[p],
                           (size_t)8 * d.nc);
        if (hipError_t e = hipGetLastError()) return e;
    }
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_wall_phi0<T>, dim3(d.nw), dim3(kBlock), 0, st, d, 0));
    return hipGetLastError();
}

// Discrete-conservative equilibrium parameters P'(W[par]) of every cell
// (and dP'/dW if with_M) into mstate: kEqGroup lanes per cell, so one wave
// serves several cells and the Newton steps' reductions span a few lanes.
// On the 256x128 grid with 64x64 velocities: 1, 2, 4, 8, 16 and 32 lanes
// per cell take 113, 79, 78, 100, 149 and 243 us.
constexpr int kEqGroup = 4;

__device__ __forceinline__ void eq_params_cell(const DevSolve &d, int c, int par, int with_M)
{
    const double *Wc = d.W[par] + 4 * c;
    const double W[4] = {Wc[0], Wc[1], Wc[2], Wc[3]};
    const double rho = W[0], u1 = W[1] / rho, u2 = W[2] / rho;
    const double th = (2.0 / 3.0) * (W[3] / rho - 0.5 * (u1 * u1 + u2 * u2));
    double P[4] = {rho, u1, u2, th}, M[16];
    eq_conservative<kEqGroup>(d, W, P, with_M ? M : nullptr);
    if (threadIdx.x % kEqGroup != 0) return;
    double *o = d.mstate + kEqState * c;
#pragma unroll
    for (int a = 0; a < 4; a++) o[a] = P[a];
    if (with_M) {
#pragma unroll
        for (int q = 0; q < 16; q++) o[4 + q] = M[q];
    }
}

__global__ __launch_bounds__(kBlock) void k_eq_params(DevSolve d, int par, int with_M)
{
    const int c = blockIdx.x * (kBlock / kEqGroup) + (int)(threadIdx.x / kEqGroup);
    if (c >= d.nc) return;                      // whole groups; shuffles stay inside a group
    eq_params_cell(d, c, par, with_M);
}

// the same for a group of batch members (member a: tab[idx[a]], state in
// buffer par[a]), bitwise the single-solve kernel's results
__global__ __launch_bounds__(kBlock) void k_eq_params_group(const DevSolve *__restrict__ tab, MacroGroup g,
                                                            int with_M)
{
    const int i = blockIdx.x * (kBlock / kEqGroup) + (int)(threadIdx.x / kEqGroup);
    if (i >= g.pre[g.n]) return;                // whole lane groups
    const int a = group_member(g, i);
    eq_params_cell(tab[g.idx[a]], i - g.pre[a], g.par[a], with_M);
}

hipError_t launch_eq_params(const DevSolve &d, int par, int with_M, hipStream_t st)
{
    if (!d.mstate || !d.equil) return hipErrorInvalidValue;
    constexpr int per_block = kBlock / kEqGroup;
    hipLaunchKernelGGL(k_eq_params, dim3((d.nc + per_block - 1) / per_block), dim3(kBlock), 0, st, d, par, with_M);
    return hipGetLastError();
}

hipError_t launch_eq_params_group(const DevSolve *tab, const MacroGroup &g, int with_M, hipStream_t st)
{
    if (g.n <= 0) return hipSuccess;
    constexpr int per_block = kBlock / kEqGroup;
    hipLaunchKernelGGL(k_eq_params_group, dim3((g.pre[g.n] + per_block - 1) / per_block), dim3(kBlock), 0, st, tab, g,
                       with_M);
    return hipGetLastError();
}

hipError_t launch_adjoint_correct_moments(const DevSolve &d, int par, const double *z, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_adjoint_moments<T, true>), dim3(xcd_grid(d.np)), dim3(kPatchBlock),
                                             adjoint_lds(d), st, d, par, z));
    return hipGetLastError();
}

hipError_t launch_adjoint_moments(const DevSolve &d, int par, hipStream_t st)
{
    DVM_DISPATCH(d.mixed, hipLaunchKernelGGL((k_adjoint_moments<T, false>), dim3(xcd_grid(d.np)), dim3(kPatchBlock),
                                             adjoint_lds(d), st, d, par, nullptr));
    return hipGetLastError();
}

hipError_t launch_adjoint_sweep(const DevSolve &d, int par, int res, hipStream_t st)
{
    const int rev = d.mem[1] == kMemTurn ? par & 1 : 0;
    DVM_FLAG(d.order == 2, SO, DVM_FLAG(d.mem[1] == kMemStream, NT, DVM_FLAG(res, RES, DVM_FLAG(d.parts[1] > 1, PARTS, DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(
        (k_adjoint_sweep<T, SO, NT, RES, PARTS>), dim3(sweep_grid(d, 1)), dim3(kPatchBlock), adjoint_lds(d), st, d, par, rev))))));
    return hipGetLastError();
}

hipError_t launch_batch(const DevSolve *tab, const int32_t *blk_solve, const int32_t *blk_patch,
                        const int32_t *par0, int step, const BatchLaunch &g, int res, hipStream_t st)
{
    if (g.blocks <= 0) return hipSuccess;
    const int rev = g.mem == kMemTurn ? step & 1 : 0;
    if (g.adjoint)
        DVM_FLAG(g.so, SO, DVM_FLAG(g.mem == kMemStream, NT, DVM_FLAG(res, RES, DVM_FLAG(g.parts, PARTS, DVM_DISPATCH(g.mixed, hipLaunchKernelGGL(
            (k_batch_adjoint<T, SO, NT, RES, PARTS>), dim3(g.blocks), dim3(kPatchBlock), g.lds, st, tab, blk_solve, blk_patch,
            par0, step, rev))))));
    else
        DVM_FLAG(g.so, SO, DVM_FLAG(g.mem == kMemStream, NT, DVM_FLAG(g.parts, PARTS, DVM_DISPATCH(g.mixed, hipLaunchKernelGGL(
            (k_batch_primal<T, SO, NT, PARTS>), dim3(g.blocks), dim3(kPatchBlock), g.lds, st, tab, blk_solve, blk_patch, par0,
            step, rev)))));
    return hipGetLastError();
}

hipError_t launch_batch_tables(const DevSolve *tab, const int32_t *phase, int n, const int *nb_group,
                               int32_t *blk_solve, int32_t *blk_patch, hipStream_t st)
{
    BatchGroups grp;
    int total = 0;
    for (int g = 0; g < 4; g++) {
        grp.nb[g] = nb_group[g];
        total += nb_group[g];
    }
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_tables, dim3((total + kBlock - 1) / kBlock), dim3(kBlock), 0, st, tab, phase, n, grp,
                       blk_solve, blk_patch);
    return hipGetLastError();
}

hipError_t launch_batch_residual(const DevSolve *tab, int n, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_batch_residual, dim3(n), dim3(kResBlock), 0, st, tab, out);
    return hipGetLastError();
}

}  // namespace dvm
