// Macroscopic prediction of the primal iteration (gfx950).
//
// Sec. 3.1 accelerates the kinetic iterations with "prediction" solutions of
// approximate macroscopic equations from the continuum limit.  Every K
// sweeps (first-order scheme):
//   1. k_eq_params: each cell's discrete-conservative equilibrium
//      parameters P' and dP'/dW by Newton;
//   2. k_macro_flux, k_macro_resid, k_macro_blocks: the moments r of the kinetic residual
//      of eq. (numerpr_gov) at the current f, and the linearised macroscopic
//      system A dW = -r with A the moments of the scheme's upwind transport of
//      equilibrium perturbations: the outflow faces carry the cell's own
//      dg/dW, the inflow faces the neighbour's, the far field nothing and
//      the wall face the diffuse value's response gbar dF_l; plus the
//      pseudo-time term (|u| + c) sum_q |S_q| / CFL (CFL 1000) on the
//      diagonal, which keeps near-singular modes of the steady operator (a
//      slow wake, a sonic region) from being amplified; stored as the
//      inverse of each cell's own block and the outflow block of each face
//      (the neighbours' inflow blocks);
//   3. k_macro_prep, k_macro_gs: red-black block Gauss-Seidel half steps from
//      dW = 0 (colour (i + j) % 2 in mesh numbering, each half step reading one
//      array and writing the other);
//   4. k_macro_apply: W += dW, limited so that rho and theta change by at
//      most 20%: the next sweep relaxes towards the predicted moments.
// The residual's moments vanish at the discrete solution, so the prediction
// leaves the solution of the plain iteration unchanged.  The work is small
// next to the sweeps (a few passes over the velocity grid per cell, every K
// sweeps), so it favours plain FP64 code, all sums in a fixed order.

#include <math.h>

#include <algorithm>

#include "dvm_walk.h"

namespace dvm {

constexpr double kMacroCFL = 1000.0;

// ---------------------------------------------------------------------------
// r_c, the moments of the kinetic residual at the current f, in two kernels.
// What flows out of c through face q, O_cq = sum_{v.S_q > 0} w Psi (v.S_q) f_c,
// is what flows into the neighbour, so
//   r_c = sum_q O_cq - sum_q O_nq' + (boundary inflow) + V/tau (W - m(P'))
// needs every row once, by its own cell (k_macro_flux), and a sum over faces
// (k_macro_resid): f is read once and no neighbour row with it, but across the
// cuts of the mesh (cut_face).  The collision part takes the moments of f from
// the sweep (W) and those of the equilibrium from 1-D sums.  k_macro_flux
// leaves O_cq [face][moment] in the face-block table mO (the blocks come after
// it) and the rest of r_c in mr.
// 256x128 cells with 64x64 velocities in FP64 454 us (725 with each cell
// reading its upwind neighbours' rows), 128x64 with 32x32 in FP32 35 us (64).
// ---------------------------------------------------------------------------
// Faces whose two sides take their vectors from nodes stored apart: the
// O-grid's seam and the C-grid's wake cut (n: the neighbour across face q of
// c).  Only inside the mesh is S_nq' the very negative of S_cq; on a cut the
// residual sums the neighbour's row with the cell's own vector, as the sweep
// does, or the iteration would not stop at the sweep's solution.
__device__ __forceinline__ bool cut_face(const DevSolve &d, int c, int q, int n)
{
    const int m = d.cell_of[c], i = m % d.ni;
    return n >= 0 && (d.topo == 0 ? (q == 1 && i == d.ni - 1) || (q == 3 && i == 0) : q == 0 && m < d.ni);
}

template <typename T, int V>
__device__ __forceinline__ void macro_flux_cell(const DevSolve &d, int par, int c, bool act, int lane)
{
    const Factors fac(d, 0);
    const GridTables gt(d);
    fac.fill(gt, gt.at(threadIdx.x));
    const double *ms = d.mstate + kEqState * c;
    const double P0 = uni(ms[0]), P1 = uni(ms[1]), P2 = uni(ms[2]), P3 = uni(ms[3]), h = 0.5 / P3;
    // moments of the equilibrium: R_p = sum wx X v1^p, T_p = sum wy Y v2^p, p < 3
    double R[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = lane; i < d.n1; i += kWave) {
        const double v = d.vx[i], e = v - P1, X = d.wx[i] * exp(-e * e * h);
        R[0] += X;
        R[1] = fma(X, v, R[1]);
        R[2] = fma(X, v * v, R[2]);
    }
    for (int i = lane; i < d.n2; i += kWave) {
        const double v = d.vy[i], e = v - P2, Y = d.wy[i] * exp(-e * e * h);
        R[3] += Y;
        R[4] = fma(Y, v, R[4]);
        R[5] = fma(Y, v * v, R[5]);
    }
    const double Rs = wave_scatter8(R);
    double Sx[4], Sy[4];
    int nb[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        nb[q] = uni(d.nbr[4 * c + q]);
        Sx[q] = uni(d.S[8 * c + 2 * q]);
        Sy[q] = uni(d.S[8 * c + 2 * q + 1]);
    }
    const int rowb = d.nv * 2 * (int)sizeof(T), bstep = d.lm.brow * d.n1 * 2 * (int)sizeof(T);
    const char *f0 = static_cast<const char *>(d.f[par]);
    const __amdgpu_buffer_rsrc_t src = row_rsrc(f0 + (size_t)c * rowb, rowb);
    // faces whose inflow is summed here, and their source rows
    bool edge[4];
    __amdgpu_buffer_rsrc_t inflow[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        edge[q] = uni((int)(nb[q] < 0 || cut_face(d, c, q, nb[q]))) != 0;
        inflow[q] = row_rsrc(nb[q] >= 0 ? f0 + (size_t)nb[q] * rowb : static_cast<const char *>(nb[q] == -1 ? d.fd : d.gw2), rowb);
    }
    const bool any = edge[0] || edge[1] || edge[2] || edge[3];
    const int wl = nb[0] <= -2 ? -2 - nb[0] : -1;
    const double ratio = wl >= 0 ? d.F[par][wl] / d.D[wl] : 0.0;
    __syncthreads();
    const double thw2 = 0.5 * d.theta_w;
    double O[4][4] = {}, in[4] = {0, 0, 0, 0};
    for (int i = 0; i < d.lm.isteps; i++) {
        const Walk wk = make_walk<T, V>(d, lane, i);
        const int a = wk.a, steps = d.lm.tq + (i < d.lm.tr ? 1 : 0);
        const ColFactor *col = fac.col + a;
        int off = wk.off, b = wk.b;
        for (int t = 0; t < steps; t++, b += d.lm.brow, off += bstep) {
            const Vals<T, V> f = row_load<T, V, false>(src, off);
            const RowFactor rf = fac.row[b];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                // t = w(v1) (v.S_q)+ f1 of the V columns, with the v1 parts of Psi
                double t = 0, ty = 0, tz = 0;
#pragma unroll
                for (int v = 0; v < V; v++) {
                    const double v1 = col[v].v, s = col[v].w * max0(v1 * Sx[q] + rf.v * Sy[q]);
                    const double x = s * (double)f.x[v], y = v1 * x;
                    t += x;
                    ty += y;
                    tz = fma(0.5 * v1, y, fma(s, (double)f.y[v], tz));
                }
                O[q][0] = fma(rf.w, t, O[q][0]);
                O[q][1] = fma(rf.w, ty, O[q][1]);
                O[q][2] = fma(rf.wv, t, O[q][2]);
                O[q][3] = fma(rf.wh, t, fma(rf.w, tz, O[q][3]));
            }
            if (any) {
                // inflow through the far-field, wall and cut faces
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    if (!edge[q]) continue;
                    const Vals<T, V> g = row_load<T, V, false>(inflow[q], off);
#pragma unroll
                    for (int v = 0; v < V; v++) {
                        const double v1 = col[v].v, ws = col[v].w * rf.w * min0(v1 * Sx[q] + rf.v * Sy[q]);
                        double g1 = (double)g.x[v], g2 = (double)g.y[v];
                        if (q == 0 && wl >= 0) {
                            g1 *= ratio;
                            g2 = thw2 * g1;
                        }
                        const double i1 = ws * g1, i2 = ws * g2;
                        in[0] += i1;
                        in[1] = fma(v1, i1, in[1]);
                        in[2] = fma(rf.v, i1, in[2]);
                        in[3] = fma(0.5 * fma(v1, v1, rf.v * rf.v), i1, in[3] + i2);
                    }
                }
            }
        }
    }
    const double v0[8] = {O[0][0], O[0][1], O[0][2], O[0][3], O[1][0], O[1][1], O[1][2], O[1][3]};
    const double v1[8] = {O[2][0], O[2][1], O[2][2], O[2][3], O[3][0], O[3][1], O[3][2], O[3][3]};
    const double s0 = wave_scatter8(v0), s1 = wave_scatter8(v1);
    double ins = 0;
    if (any) {
        const double v2[8] = {in[0], in[1], in[2], in[3], 0, 0, 0, 0};
        ins = wave_scatter8(v2);
    }
    // collision part V/tau (W - m(P')), moment lane / 8 (lanes 0 .. 31)
    const double R0 = lane_value(Rs, 0), R1 = lane_value(Rs, 8), R2 = lane_value(Rs, 16);
    const double T0 = lane_value(Rs, 24), T1 = lane_value(Rs, 32), T2 = lane_value(Rs, 40);
    const double kap = P0 / (2.0 * kPi * P3);
    const int m = lane >> 3;
    const double mom = m == 0 ? R0 * T0 : m == 1 ? R1 * T0 : m == 2 ? R0 * T1
                                        : 0.5 * (R2 * T0 + R0 * T2) + 0.5 * P3 * R0 * T0;
    const double *W = d.W[par] + 4 * c;
    const double rho = uni(W[0]), u1 = uni(W[1]) / rho, u2 = uni(W[2]) / rho;
    const double th = (2.0 / 3.0) * (uni(W[3]) / rho - 0.5 * (u1 * u1 + u2 * u2));
    const double Vt = d.vol[c] * d.inv_tau_inf * rho * sqrt(2.0 * th);
    if (!act || (lane & 7) != 0) return;
    d.mO[64 * (size_t)c + m] = s0;
    d.mO[64 * (size_t)c + 8 + m] = s1;
    if (m < 4) d.mr[4 * c + m] = Vt * (W[m] - kap * mom) + ins;
}

template <typename T>
__global__ __launch_bounds__(kPatchCells *kWave) void k_macro_flux(DevSolve d, int par)
{
    const int p = xcd_item(d.np, blockIdx.x);
    if (p < 0) return;
    int w;
    bool act;
    const int c = patch_wave(d, p, w, act), lane = threadIdx.x % kWave;
    if (sizeof(T) == 4 && pair_velocities<T>(d.n1))
        macro_flux_cell<T, sizeof(T) == 4 ? 2 : 1>(d, par, c, act, lane);
    else
        macro_flux_cell<T, 1>(d, par, c, act, lane);
}

// the face of cell n that faces cell c (n a face neighbour of c)
__device__ __forceinline__ int back_face(const DevSolve &d, int n, int c)
{
    int qb = 0;
#pragma unroll
    for (int t = 3; t >= 0; t--)
        if (d.nbr[4 * n + t] == c) qb = t;
    return qb;
}

// r_c from the face fluxes, four lanes per cell
__global__ __launch_bounds__(kBlock) void k_macro_resid(DevSolve d)
{
    const int t = blockIdx.x * kBlock + threadIdx.x, c = t >> 2, m = t & 3;
    if (c >= d.nc) return;
    double r = d.mr[4 * c + m];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int n = d.nbr[4 * c + q];
        r += d.mO[64 * (size_t)c + 4 * q + m];
        if (n >= 0 && !cut_face(d, c, q, n)) r -= d.mO[64 * (size_t)n + 4 * back_face(d, n, c) + m];
    }
    d.mr[4 * c + m] = r;
}

// ---------------------------------------------------------------------------
// the macroscopic blocks of each cell, one wave per cell, no distribution
// read: each face q gets its outflow block
//   B_cq = sum_{k: v.S_q > 0} w (v.S_q) Psi_k dg_c,k/dW,
// and the cell's own block is D_c = sum_q B_cq + wall1 dF + lam I (wall1 dF:
// the diffuse wall's re-emission of the outgoing flux; lam the pseudo-time
// term).  The inflow block of the neighbour n across face q is -B_nq' (q'
// the face of n that faces c: S_nq' = -S_cq, so n's outflow half-space
// through q' is c's inflow half-space through q and the sums agree term by
// term).  The Gauss-Seidel steps read the neighbours' B instead of a
// separate off-diagonal table.
//
// The sums factor on the tensor grid.  With g = kap X(v1) Y(v2), e = v - u and
// ascending nodes, the velocities of a grid row b with v.S_q > 0 are the
// columns from some a* on (S_x > 0) or before it, so a sum over the half
// space of e1^p e2^r g is sum_b Y e2^r R_p(a*_b) with R_p the sums of X e1^p
// from either end, tabulated once per cell.  B needs p + r <= 5 (s Psi dg:
// degrees 1 + 2 + 2): 21 sums of n2 terms per face instead of 20 of n1 n2.
// a* is found by bisection on the same rounded v.S_q > 0 as the sweeps'.
// Vector instructions bound it: 256x128 cells with 64x64 velocities 1190 us
// (one term per velocity) -> 148 us, 128x64 with 32x32 186 -> 36 us.
// ---------------------------------------------------------------------------
constexpr int kBlkCells = kBlock / kWave;
constexpr int kHalfMoments = 6;               // R_p, p = 0 .. 5

inline unsigned blocks_lds(const DevSolve &d)
{
    return 8u * (d.n1 + kBlkCells * (2 * kHalfMoments * (d.n1 + 1) + 2 * d.n2));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_shift(double x)      // 0 where the lane has no source
{
    const long long u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffLL), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// inclusive scan over the wave
__device__ __forceinline__ double wave_scan(double x)
{
    x += dpp_shift<0x111, 0xf>(x);             // row_shr 1, 2, 4, 8
    x += dpp_shift<0x112, 0xf>(x);
    x += dpp_shift<0x114, 0xf>(x);
    x += dpp_shift<0x118, 0xf>(x);
    x += dpp_shift<0x142, 0xa>(x);             // last lane of rows 0, 2 to rows 1, 3
    x += dpp_shift<0x143, 0xc>(x);             // lane 31 to rows 2, 3
    return x;
}

// sum over the 16 lanes of a row, in every one of them
__device__ __forceinline__ double row_sum(double x)
{
    x += dpp_shift<0x128, 0xf>(x);             // lane ^ 8
    x += dpp_shift<0x141, 0xf>(x);             // lane ^ 7
    x += dpp_shift<0x4e, 0xf>(x);              // lane ^ 2
    x += dpp_shift<0xb1, 0xf>(x);              // lane ^ 1
    return x;
}

extern __shared__ __align__(16) double blocks_smem[];

__global__ __launch_bounds__(kBlock) void k_macro_blocks(DevSolve d, int par)
{
    const int w = uni((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
    const int n1 = d.n1, n2 = d.n2;
    double *vx = blocks_smem;
    double *half = vx + n1 + w * (2 * kHalfMoments * (n1 + 1) + 2 * n2);     // [from below, from above][a][p]
    double *wY = half + 2 * kHalfMoments * (n1 + 1), *e2 = wY + n2;
    const int c0 = uni((int)blockIdx.x * kBlkCells + w);
    const bool act = c0 < d.nc;                 // idle waves of the last workgroup only join the barrier
    const int c = act ? c0 : d.nc - 1;
    const double *ms = d.mstate + kEqState * c;
    const double rhoP = uni(ms[0]), u1 = uni(ms[1]), u2 = uni(ms[2]), th = uni(ms[3]);
    const double hh = 0.5 / th;
    for (int i = threadIdx.x; i < n1; i += kBlock) vx[i] = d.vx[i];
    for (int i = lane; i < n2; i += kWave) {
        const double e = d.vy[i] - u2;
        e2[i] = e;
        wY[i] = d.wy[i] * exp(-e * e * hh);
    }
    // R_p from below (columns < a) and from above (columns >= a), 64 columns
    // at a time, the totals so far carried along
    for (int dir = 0; dir < 2; dir++) {
        double *tab = half + dir * kHalfMoments * (n1 + 1);
        double carry[kHalfMoments];
#pragma unroll
        for (int p = 0; p < kHalfMoments; p++) carry[p] = 0;
        if (lane < kHalfMoments) tab[(dir ? n1 : 0) * kHalfMoments + lane] = 0;
        for (int i0 = 0; i0 < n1; i0 += kWave) {
            const int i = i0 + lane, a = dir ? n1 - 1 - i : i;
            const bool in = i < n1;
            const double e = in ? d.vx[a] - u1 : 0.0;
            double t = in ? d.wx[a] * exp(-e * e * hh) : 0.0;
#pragma unroll
            for (int p = 0; p < kHalfMoments; p++) {
                const double sum = wave_scan(t) + carry[p];
                if (in) tab[(dir ? a : a + 1) * kHalfMoments + p] = sum;
                carry[p] = __shfl(sum, kWave - 1, kWave);
                t *= e;
            }
        }
    }
    // lanes 16 q + i: face q, grid rows i, i + 16, ...
    const int q = lane >> 4;
    const double Sx = d.S[8 * c + 2 * q], Sy = d.S[8 * c + 2 * q + 1];
    __syncthreads();
    double M[21];                               // sums of e1^p e2^r over the face's outflow half-space
#pragma unroll
    for (int i = 0; i < 21; i++) M[i] = 0;
    int bits = 0;
    while ((1 << bits) <= n1) bits++;
    for (int b = lane & 15; b < n2; b += 16) {
        // columns [0, a) with v.S <= 0 (S_x > 0: outflow from above) or > 0 (from below)
        const double sy = d.vy[b] * Sy;
        int lo = 0, hi = n1;
        for (int t = 0; t < bits; t++) {
            const int mid = (lo + hi) >> 1;
            const bool pos = vx[min(mid, n1 - 1)] * Sx + sy > 0;
            if (lo < hi) {
                if (pos == (Sx > 0))
                    hi = mid;
                else
                    lo = mid + 1;
            }
        }
        const double *R = half + ((Sx > 0 ? n1 + 1 : 0) + lo) * kHalfMoments;
        double yr = wY[b];
        const double e = e2[b];
        int k = 0;
#pragma unroll
        for (int r = 0; r < kHalfMoments; r++) {
#pragma unroll
            for (int p = 0; p + r < kHalfMoments; p++) {
                M[k] = fma(yr, R[p], M[k]);
                k++;
            }
            yr *= e;
        }
    }
#pragma unroll
    for (int i = 0; i < 21; i++) M[i] = row_sum(M[i]);
    // K_ij = sum w s g phi_i phi_j with phi = (1, e1, e2, |e|^2/2), s = S.e + S.u:
    // m(p, r) the sum of e1^p e2^r, sm that of s e1^p e2^r
    const double kap = rhoP / (2.0 * kPi * th), su = fma(Sx, u1, Sy * u2);
    auto m = [&](int p, int r) { return M[6 * r - r * (r - 1) / 2 + p]; };
    auto sm = [&](int p, int r) { return kap * fma(Sx, m(p + 1, r), fma(Sy, m(p, r + 1), su * m(p, r))); };
    double K[4][4];
    K[0][0] = sm(0, 0);
    K[0][1] = K[1][0] = sm(1, 0);
    K[0][2] = K[2][0] = sm(0, 1);
    K[1][1] = sm(2, 0);
    K[1][2] = K[2][1] = sm(1, 1);
    K[2][2] = sm(0, 2);
    K[0][3] = K[3][0] = 0.5 * (K[1][1] + K[2][2]);
    K[1][3] = K[3][1] = 0.5 * (sm(3, 0) + sm(1, 2));
    K[2][3] = K[3][2] = 0.5 * (sm(2, 1) + sm(0, 3));
    K[3][3] = 0.25 * (sm(4, 0) + 2.0 * sm(2, 2) + sm(0, 4));
    // entry (x, mm) of B_cq in lane 16 q + 4 x + mm:
    // B = T K D dP/dW, Psi = T phi, dg1/dP = g phi D, and dg2/dP = th/2 dg1/dP + (0, 0, 0, g/2)
    // in the energy row
    const int x = (lane >> 2) & 3, mm = lane & 3;
    const double uu = 0.5 * (u1 * u1 + u2 * u2);
    const double t0 = x == 0 ? 1.0 : x == 1 ? u1 : x == 2 ? u2 : uu + 0.5 * th;
    const double t1 = x == 1 ? 1.0 : x == 3 ? u1 : 0.0, t2 = x == 2 ? 1.0 : x == 3 ? u2 : 0.0, t3 = x == 3 ? 1.0 : 0.0;
    double TK[4];
#pragma unroll
    for (int j = 0; j < 4; j++) TK[j] = fma(t0, K[0][j], fma(t1, K[1][j], fma(t2, K[2][j], t3 * K[3][j])));
    const double ith = 1.0 / th;
    const double Bp[4] = {TK[0] / rhoP, TK[1] * ith, TK[2] * ith,
                          (TK[3] * ith - TK[0]) * ith + 0.5 * t3 * K[0][0]};
    double Be = 0;
#pragma unroll
    for (int p = 0; p < 4; p++) Be = fma(Bp[p], ms[4 + 4 * p + mm], Be);
    if (act) d.mO[64 * c + lane] = Be;
    // own block: the faces' sum, the wall's response and the pseudo-time term V/dt
    double De = Be + __shfl_xor(Be, 16, kWave);
    De += __shfl_xor(De, 32, kWave);
    const int nb0 = uni(d.nbr[4 * c]);
    if (nb0 <= -2) {
        // wall cell: where the wall face is inflow, the diffuse value's
        // response; the outgoing flux's response is row 0 of B_c0 over A
        const int wl = -2 - nb0;
        const double S0x = uni(d.S[8 * c]), S0y = uni(d.S[8 * c + 1]), thw2 = 0.5 * d.theta_w, iD = 1.0 / d.D[wl];
        const double *gMd = static_cast<const double *>(d.gM);
        const float *gMf = static_cast<const float *>(d.gM);
        double wall[4] = {0, 0, 0, 0};
        for (int k = lane; k < d.nv; k += kWave) {
            const int a = k % n1, b = k / n1;
            const double v1 = vx[a], v2 = d.vy[b], s = v1 * S0x + v2 * S0y;
            if (!(s > 0)) {
                const double g = d.wx[a] * d.wy[b] * s * ((d.mixed ? (double)gMf[k] : gMd[k]) * iD);
                wall[0] += g;
                wall[1] = fma(g, v1, wall[1]);
                wall[2] = fma(g, v2, wall[2]);
                wall[3] = fma(g, fma(0.5, fma(v1, v1, v2 * v2), thw2), wall[3]);
            }
        }
        wave_sum<4>(wall);
        const double dF = __shfl(Be, mm, kWave) / d.wall_A[wl];
        const double wx4 = x == 0 ? wall[0] : x == 1 ? wall[1] : x == 2 ? wall[2] : wall[3];
        De = fma(wx4, dF, De);
    }
    const double *W = d.W[par] + 4 * c;
    const double rho = W[0], w1 = W[1] / rho, w2 = W[2] / rho;
    const double thW = (2.0 / 3.0) * (W[3] / rho - 0.5 * (w1 * w1 + w2 * w2));
    double sS = 0.0;
#pragma unroll
    for (int f = 0; f < 4; f++) sS += hypot(d.S[8 * c + 2 * f], d.S[8 * c + 2 * f + 1]);
    const double lam = (sqrt(w1 * w1 + w2 * w2) + sqrt(5.0 / 3.0 * thW)) * sS / kMacroCFL;
    if (x == mm) De += lam;
    // inverse: lane l solves for column l % 4
    double A[4][4], rhs[4], col[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        rhs[i] = i == mm ? 1.0 : 0.0;
#pragma unroll
        for (int j = 0; j < 4; j++) A[i][j] = __shfl(De, 4 * i + j, kWave);
    }
    solve4(A, rhs, col);
    if (act && lane < 16) d.mDinv[16 * c + lane] = x == 0 ? col[0] : x == 1 ? col[1] : x == 2 ? col[2] : col[3];
}

// The iteration blocks, in place of the face blocks B: 16 lanes per (cell,
// face), lane 4 x + m its entry (x, m).
//   primal   C_cq = Dinv_c B_nq' and r_c <- y_c = -Dinv_c r_c, so that a half
//            step is x_c = y_c + sum_q C_cq x_n (-B_nq' is the inflow block of
//            the neighbour n); the two blocks of a face trade places, taken
//            by its lower-numbered cell
//   adjoint  E_cq = (Dinv_n B_cq)^T, what cell n's update passes back to c
// Boundary faces get zero blocks.
template <bool ADJ>
__global__ __launch_bounds__(kBlock) void k_macro_prep(DevSolve d)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x, item = t >> 4, e = t & 15, x = e >> 2, m = e & 3;
    if (item >= 4 * d.nc) return;               // whole groups of 16 lanes
    const int c = item >> 2, q = item & 3, n = d.nbr[4 * c + q];
    double *B = d.mO + 64 * c + 16 * q;
    if (n < 0) {
        B[e] = 0.0;
    } else if constexpr (ADJ) {
        const double b = B[e], Dn = d.mDinv[16 * n + e];
        double s = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) s = fma(__shfl(Dn, 4 * m + k, 16), __shfl(b, 4 * k + x, 16), s);
        B[e] = s;
    } else if (c < n) {
        double *Bn = d.mO + 64 * n + 16 * back_face(d, n, c);
        const double bc = B[e], bn = Bn[e], Dc = d.mDinv[16 * c + e], Dn = d.mDinv[16 * n + e];
        double sc = 0, sn = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            sc = fma(__shfl(Dc, 4 * x + k, 16), __shfl(bn, 4 * k + m, 16), sc);
            sn = fma(__shfl(Dn, 4 * x + k, 16), __shfl(bc, 4 * k + m, 16), sn);
        }
        B[e] = sc;
        Bn[e] = sn;
    }
    if (!ADJ && q == 0) {
        const double p = d.mDinv[16 * c + e] * d.mr[4 * c + m];
        double s = p + __shfl_xor(p, 1, 16);
        s += __shfl_xor(s, 2, 16);
        if (m == 0) d.mr[4 * c + x] = -s;       // all lanes of the group have read r
    }
}

// device number of mesh cell (i, j) (the storage order of build_patches)
__device__ __forceinline__ int device_cell(const DevSolve &d, int i, int j)
{
    const int i0 = i - i % kTileI, j0 = j - j % kTileJ, wt = min(kTileI, d.ni - i0), ht = min(kTileJ, d.nj - j0);
    const int ii = i - i0, jj = j - j0, pi = ii - ii % kPatchI, pj = jj - jj % kPatchJ;
    const int wp = min(kPatchI, wt - pi), hp = min(kPatchJ, ht - pj);
    return i0 * d.nj + wt * j0 + wt * pj + hp * pi + (jj - pj) * wp + (ii - pi);
}

// ---------------------------------------------------------------------------
// `steps` half steps of the red-black block Gauss-Seidel iteration in one
// launch.  A workgroup owns a tile of the mesh and computes on a window of
// kGsW x kGsH cells around it, `steps` cells wider on each side: after k half
// steps the window's outer k cells are wrong, the tile is not.  A window
// follows the mesh across the periodic seam and, mirrored, across the wake
// cut; cells outside it or the mesh take part with nothing.  Four lanes per
// pair of cells (one of each colour), lane a holding row a of the blocks in
// registers, the iterates in LDS.
//
// Why: one half step a launch took 4.6 to 8 us, its launch and the chain
// neighbour - back face - block, on any mesh up to 32768 cells; here a half
// step costs two LDS reads a neighbour and a barrier, and the blocks are read
// once per launch (measured figures at gs_steps).
//
// primal, colour on:  x_c = y_c + sum_q C_cq x_n
// adjoint (the transposed half steps in reverse order), colour on:
//   s_on += v_on, then v_m = (m off: v_m) + sum_{n on} E_mq v_n; after the
//   last one z = -Dinv^T s.
// Neighbours of one colour (an odd ni across the seam) read the old values.
// ---------------------------------------------------------------------------
constexpr int kGsW = 24, kGsH = 21, kGsBlock = 1024;
static_assert(kGsW % 2 == 0 && 2 * kGsW * kGsH <= kGsBlock, "four lanes per pair of cells");

template <bool ADJ>
__device__ __forceinline__ void gs_tile(const DevSolve &d, int tile, const GsStep &st, const double *__restrict__ src,
                                        double *__restrict__ dst)
{
    __shared__ __align__(16) double xs[4 * kGsW * kGsH];
    const int g = threadIdx.x >> 2, a = threadIdx.x & 3;
    const bool lane_in = g < kGsW * kGsH / 2;
    const int tw = kGsW - 2 * st.steps, th = kGsH - 2 * st.steps, tiles_i = (d.ni + tw - 1) / tw;
    const int i0 = (tile % tiles_i) * tw - st.steps, j0 = (tile / tiles_i) * th - st.steps;
    const int wj = g / (kGsW / 2);
    const bool odd = (d.ni & 1) != 0;           // neighbours of one colour
    int cell[2], li[2], col[2], nl[2][4], same[2];
    bool own[2];
    double C[2][16], y[2], s[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const int wi = 2 * (g % (kGsW / 2)) + ((u ^ wj) & 1);
        int i = i0 + wi, j = j0 + wj;
        bool ok = lane_in && j < d.nj, mir = false;
        own[u] = ok && i >= 0 && i < d.ni && j >= 0 && wi >= st.steps && wi < st.steps + tw && wj >= st.steps &&
                 wj < st.steps + th;
        if (d.topo == 0) {
            ok = ok && j >= 0;
            i %= d.ni;
            if (i < 0) i += d.ni;
        } else {
            ok = ok && i >= 0 && i < d.ni;
            if (j < 0) {
                mir = true;
                i = d.ni - 1 - i;
                j = -1 - j;
                ok = ok && j < d.nj;
            }
        }
        li[u] = lane_in ? wj * kGsW + wi : 0;
        cell[u] = ok ? device_cell(d, i, j) : -1;
        col[u] = (i + j) & 1;
        same[u] = 0;
        const int sg = mir ? -1 : 1;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int di = sg * (q == 1 ? 1 : q == 3 ? -1 : 0), dj = sg * (q == 2 ? 1 : q == 0 ? -1 : 0);
            const bool in = wi + di >= 0 && wi + di < kGsW && wj + dj >= 0 && wj + dj < kGsH;
            nl[u][q] = in ? 4 * (li[u] + di + kGsW * dj) : 4 * li[u];
        }
        y[u] = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) C[u][k] = 0;
        double x0 = 0;
        if (ok) {
            const double *B = d.mO + 64 * (size_t)cell[u] + 4 * a;
#pragma unroll
            for (int q = 0; q < 4; q++) {
#pragma unroll
                for (int e = 0; e < 4; e++) C[u][4 * q + e] = B[16 * q + e];
                if (odd) {
                    const int n = d.nbr[4 * cell[u] + q];
                    if (n >= 0) {
                        const int mn = d.cell_of[n];
                        if (((mn % d.ni + mn / d.ni) & 1) == col[u]) same[u] |= 1 << q;
                    }
                }
            }
            if (!ADJ) y[u] = d.mr[4 * cell[u] + a];
            if (ADJ && own[u] && !st.first) s[u] = d.mr[4 * cell[u] + a];     // one running sum, whatever the launches
            if (ADJ || !st.first) x0 = src[4 * cell[u] + a];
        }
        if (lane_in) xs[4 * li[u] + a] = x0;
    }
    __syncthreads();
    for (int t = 0; t < st.steps; t++) {
        const int on = (st.colour + t) & 1;
        double nx[2];
        bool set[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const bool lit = col[u] == on;
            // primal: cells of the colour; adjoint: the others (and, next to
            // neighbours of their own colour, these too)
            set[u] = cell[u] >= 0 && (ADJ || lit);
            nx[u] = 0;
            if (!set[u]) continue;
            if (!ADJ) {
                double acc = y[u];
#pragma unroll
                for (int q = 0; q < 4; q++)
#pragma unroll
                    for (int e = 0; e < 4; e++) acc = fma(C[u][4 * q + e], xs[nl[u][q] + e], acc);
                nx[u] = acc;
            } else {
                const double v = xs[4 * li[u] + a];
                double acc = lit ? 0.0 : v;
                if (lit) s[u] += v;
                if (!lit || same[u]) {
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        if (odd && lit != (((same[u] >> q) & 1) != 0)) continue;
#pragma unroll
                        for (int e = 0; e < 4; e++) acc = fma(C[u][4 * q + e], xs[nl[u][q] + e], acc);
                    }
                }
                nx[u] = acc;
            }
        }
        if (ADJ || odd) __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; u++)
            if (set[u]) xs[4 * li[u] + a] = nx[u];
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 2; u++) {
        if (!own[u]) continue;                  // whole groups of four lanes
        const int at = 4 * cell[u] + a;
        if (!ADJ || !st.last) dst[at] = xs[4 * li[u] + a];
        if (ADJ) {
            double sum = s[u];
            if (st.last) {
                const double *Di = d.mDinv + 16 * (size_t)cell[u];
                double z = 0;
#pragma unroll
                for (int e = 0; e < 4; e++) z = fma(-Di[4 * e + a], __shfl(sum, e, 4), z);
                sum = z;
            }
            d.mr[at] = sum;
        }
    }
}

template <bool ADJ>
__global__ __launch_bounds__(kGsBlock) void k_macro_gs(DevSolve d, GsStep st, int tiles, int from)
{
    const int tile = xcd_item(tiles, blockIdx.x);
    if (tile >= 0) gs_tile<ADJ>(d, tile, st, d.mx[from], d.mx[from ^ 1]);
}

// Several solves of a batch in one launch: member a owns tiles pre[a] ..
// pre[a+1]-1 of the group.  The steps per launch may differ from a single
// solve's; each cell's arithmetic does not, so the results are bitwise the
// same.
template <bool ADJ>
__global__ __launch_bounds__(kGsBlock) void k_macro_gs_group(const DevSolve *__restrict__ tab, MacroGroup g, GsStep st,
                                                             int from)
{
    const int item = xcd_item(g.pre[g.n], blockIdx.x);
    if (item < 0) return;
    const int a = group_member(g, item);
    const DevSolve &d = tab[g.idx[a]];
    gs_tile<ADJ>(d, item - g.pre[a], st, d.mx[from], d.mx[from ^ 1]);
}

// Half steps per launch for meshes of ni[k] x nj[k] cells: more of them save
// launches but leave smaller tiles of the fixed window; a launch of more
// tiles than the chip has compute units takes another round of them (one
// window's registers fill a unit).  The line fits launches measured at 2 to 8
// half steps (6.1 to 8.4 us; 14.6 us in two rounds).  50 steps, primal /
// adjoint us, with one launch a half step and here: 64x32 cells 433 / 517 ->
// 110 / 133, 128x64 420 / 515 -> 105 / 135, 256x128 666 / 808 -> 167 / 202.
static int gs_tiles(int ni, int nj, int steps)
{
    const int tw = kGsW - 2 * steps, th = kGsH - 2 * steps;
    return ((ni + tw - 1) / tw) * ((nj + th - 1) / th);
}

static int gs_steps(const int *ni, const int *nj, int n, int total)
{
    int best = 1;
    double cost = 0;
    for (int steps = 1; steps <= kGsMaxSteps && steps <= total; steps++) {
        int tiles = 0;
        for (int k = 0; k < n; k++) tiles += gs_tiles(ni[k], nj[k], steps);
        const int launches = (total + steps - 1) / steps, rounds = (tiles + 255) / 256;
        const double c = launches * (1.5 + rounds * (3.8 + 0.45 * steps));
        if (steps == 1 || c < cost) {
            best = steps;
            cost = c;
        }
    }
    const int launches = (total + best - 1) / best;
    return (total + launches - 1) / launches;
}

__global__ __launch_bounds__(kBlock) void k_macro_zero(double *x, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.0;
}

// W += dW, limited: rho and theta change by at most kMacroLimit
constexpr double kMacroLimit = 0.2;

__device__ __forceinline__ double theta_of(const double *W)
{
    const double u1 = W[1] / W[0], u2 = W[2] / W[0];
    return (2.0 / 3.0) * (W[3] / W[0] - 0.5 * (u1 * u1 + u2 * u2));
}

__global__ __launch_bounds__(kBlock) void k_macro_apply(DevSolve d, int par, const double *__restrict__ x)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= d.nc) return;
    double *W = d.W[par] + 4 * c;
    double Wt[4];
#pragma unroll
    for (int a = 0; a < 4; a++) Wt[a] = W[a] + x[4 * c + a];
    const double th0 = theta_of(W), th1 = theta_of(Wt);
    const double ch = fmax(fabs(x[4 * c]) / W[0], fabs(th1 - th0) / th0);
    double fac = 0.0;
    if (Wt[0] > 0 && th1 > 0 && isfinite(ch)) fac = ch > kMacroLimit ? kMacroLimit / ch : 1.0;
#pragma unroll
    for (int a = 0; a < 4; a++) W[a] += fac * x[4 * c + a];
}

// primal: P' and dP'/dW of W[par], the residual's moments and the blocks;
// adjoint: the blocks (the adjoint's start has left P' and dP'/dW)
static hipError_t macro_system(const DevSolve &d, int par, bool primal, hipStream_t st)
{
    if (primal) {
        if (hipError_t e = launch_eq_params(d, par, 1, st)) return e;
        DVM_DISPATCH(d.mixed, hipLaunchKernelGGL(k_macro_flux<T>, dim3(xcd_grid(d.np)), dim3(kPatchCells * kWave),
                                                 factor_lds(d.lm), st, d, par));
        if (hipError_t e = hipGetLastError()) return e;
        hipLaunchKernelGGL(k_macro_resid, dim3((4 * d.nc + kBlock - 1) / kBlock), dim3(kBlock), 0, st, d);
        if (hipError_t e = hipGetLastError()) return e;
    }
    hipLaunchKernelGGL(k_macro_blocks, dim3((d.nc + kBlkCells - 1) / kBlkCells), dim3(kBlock), blocks_lds(d), st, d, par);
    return hipGetLastError();
}

template <bool ADJ>
static hipError_t macro_prep(const DevSolve &d, hipStream_t st)
{
    const int64_t threads = (int64_t)64 * d.nc;
    hipLaunchKernelGGL(k_macro_prep<ADJ>, dim3((unsigned)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_macro_predict_begin(const DevSolve &d, int par, int inner, hipStream_t st)
{
    if (hipError_t e = macro_system(d, par, true, st)) return e;
    if (hipError_t e = macro_prep<false>(d, st)) return e;
    if (inner > 0) return hipSuccess;
    hipLaunchKernelGGL(k_macro_zero, dim3((4 * d.nc + kBlock - 1) / kBlock), dim3(kBlock), 0, st, d.mx[0], 4 * d.nc);
    return hipGetLastError();
}

hipError_t launch_macro_predict_end(const DevSolve &d, int par, int from, hipStream_t st)
{
    hipLaunchKernelGGL(k_macro_apply, dim3((d.nc + kBlock - 1) / kBlock), dim3(kBlock), 0, st, d, par, d.mx[from]);
    return hipGetLastError();
}

// the launches of `inner` steps; `go` launches one; the result is in buffer
// (launches & 1)
template <typename F>
static hipError_t gs_launches(int total, int steps, int colour0, F go, int *from)
{
    int k = 0;
    for (int done = 0; done < total; done += steps, k++) {
        GsStep st;
        st.steps = std::min(steps, total - done);
        st.colour = (colour0 + done) & 1;
        st.first = done == 0;
        st.last = done + st.steps == total;
        go(st, k & 1);
        if (hipError_t e = hipGetLastError()) return e;
    }
    *from = k & 1;
    return hipSuccess;
}

// The forward steps run colour 0 then 1 in each of `inner`; the transposed
// ones the reverse, colour 1 first.
static hipError_t gs_single(const DevSolve &d, int inner, int adjoint, int *from, hipStream_t st)
{
    *from = 0;
    if (inner <= 0) return hipSuccess;
    const int steps = gs_steps(&d.ni, &d.nj, 1, 2 * inner);
    return gs_launches(2 * inner, steps, adjoint, [&](const GsStep &gs, int k) {
        const int tiles = gs_tiles(d.ni, d.nj, gs.steps);
        DVM_FLAG(adjoint, ADJ, hipLaunchKernelGGL(k_macro_gs<ADJ>, dim3(xcd_grid(tiles)), dim3(kGsBlock), 0, st, d, gs,
                                                  tiles, k));
    }, from);
}

hipError_t launch_macro_predict(const DevSolve &d, int par, int inner, hipStream_t st)
{
    int from = 0;
    if (hipError_t e = launch_macro_predict_begin(d, par, inner, st)) return e;
    if (hipError_t e = gs_single(d, inner, 0, &from, st)) return e;
    return launch_macro_predict_end(d, par, from, st);
}

// ---------------------------------------------------------------------------
// adjoint prediction: the transpose of the primal's accelerated sweep.
// Linearised at the converged f, the primal sweep after a prediction is
// f' = f + D^-1 Q R'(f), Q = I - H L M (M the moments, L the Gauss-Seidel
// map above, H = dg/dW V/tau + (g - f) d(V/tau)/dW: how the predicted
// moments enter the sweep).  Its transpose for the adjoint equation is
// phi' = phi_s - Psi L^T (H^T (phi_s - phi)), phi_s the plain adjoint
// sweep's result: every K-th adjoint sweep
//   1. k_macro_adj_y: y = H^T (phi_s - phi) per cell, from the adjoint
//      moments the two sweeps left (What and rho_tau are linear in phi):
//      y = V (What_s - What) / tau - V (1/tau dtau/dW) (rho_tau,s - rho_tau);
//   2. k_macro_gs<true>: z = L^T y, the Gauss-Seidel half steps transposed
//      in reverse order;
//   3. k_adjoint_correct_moments: phi_s -= (z . Psi, z_3) and the adjoint
//      moments of the corrected phi, in one pass.
// The accelerated adjoint cycle then has the eigenvalues of the primal's,
// and the correction vanishes with the sweep's change (the adjoint solution
// is the plain iteration's).
// ---------------------------------------------------------------------------

// y_c = H_c^T (phi_s - phi) from the adjoint moments of phi_s (aW[pnew]) and
// of phi (aW[pnew ^ 1]), written as the seed of the transposed solve
__global__ __launch_bounds__(kBlock) void k_macro_adj_y(DevSolve d, int pnew, double *__restrict__ y)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= d.nc) return;
    const double *an = d.aW[pnew] + 8 * c, *ao = d.aW[pnew ^ 1] + 8 * c;
    const double *ac = d.acoef + kAcoef * c;
    const double V = d.vol[c], itau = ac[4], drt = an[4] - ao[4];
#pragma unroll
    for (int m = 0; m < 4; m++) y[4 * c + m] = V * (itau * (an[m] - ao[m]) - ac[6 + m] * drt);
}

hipError_t launch_macro_adjoint_setup(const DevSolve &d, int fpar, hipStream_t st)
{
    if (hipError_t e = macro_system(d, fpar, false, st)) return e;
    return macro_prep<true>(d, st);
}

hipError_t launch_macro_adjoint_begin(const DevSolve &d, int pnew, int inner, hipStream_t st)
{
    const int gt = (d.nc + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_macro_adj_y, dim3(gt), dim3(kBlock), 0, st, d, pnew, d.mx[0]);
    if (hipError_t e = hipGetLastError()) return e;
    if (inner > 0) return hipSuccess;
    hipLaunchKernelGGL(k_macro_zero, dim3((4 * d.nc + kBlock - 1) / kBlock), dim3(kBlock), 0, st, d.mr, 4 * d.nc);
    return hipGetLastError();
}

hipError_t launch_macro_adjoint_end(const DevSolve &d, int pnew, hipStream_t st)
{
    // phi -= (z . Psi, z_3) and the adjoint moments of the result, one pass
    return launch_adjoint_correct_moments(d, pnew, d.mr, st);
}

hipError_t launch_macro_adjoint_predict(const DevSolve &d, int pnew, int inner, hipStream_t st)
{
    int from = 0;
    if (hipError_t e = launch_macro_adjoint_begin(d, pnew, inner, st)) return e;
    if (hipError_t e = gs_single(d, inner, 1, &from, st)) return e;
    return launch_macro_adjoint_end(d, pnew, st);
}

// the Gauss-Seidel steps of a group of batch members with the same inner
// count, in shared launches (g.ni, g.nj: the members' meshes)
hipError_t launch_macro_gs_group(const DevSolve *tab, MacroGroup g, int inner, int adjoint, int *from, hipStream_t st)
{
    *from = 0;
    if (g.n <= 0 || inner <= 0) return hipSuccess;
    const int steps = gs_steps(g.ni, g.nj, g.n, 2 * inner);
    return gs_launches(2 * inner, steps, adjoint, [&](const GsStep &gs, int k) {
        g.pre[0] = 0;
        for (int a = 0; a < g.n; a++) g.pre[a + 1] = g.pre[a] + gs_tiles(g.ni[a], g.nj[a], gs.steps);
        DVM_FLAG(adjoint, ADJ, hipLaunchKernelGGL(k_macro_gs_group<ADJ>, dim3(xcd_grid(g.pre[g.n])), dim3(kGsBlock), 0,
                                                  st, tab, g, gs, k));
    }, from);
}

}  // namespace dvm
