// Internal interface between the host side of libdvm and its HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

struct dvm_mesh;

namespace dvm {

constexpr int kBlock = 256;        // threads per workgroup of the per-cell and per-element kernels
constexpr int kWave = 64;          // wavefront width
constexpr int kMaxN1D = 128;       // max velocity nodes per direction
constexpr int kMaxParams = 64;
constexpr int kAcoef = 32;         // doubles per cell of the adjoint coefficients
constexpr int kEqState = 20;       // doubles per cell of mstate: P' (4), dP'/dW (16, row = parameter)

// The sweeps give each workgroup a patch of kPatchI x kPatchJ cells, one
// wave per cell; patches tile kTileI x kTileJ tiles, which follow each
// other along strips of kTileI columns.  Cells are stored (and numbered on
// the device) in that order, patch after patch.  Measured on the 256x128
// C-grid with 2304 velocities (FP64 adjoint sweep): strips of 8, 16, 32 and
// 64 columns take 775, 755, 735 and 745 us.
constexpr int kPatchI = 2, kPatchJ = 2, kPatchCells = kPatchI * kPatchJ;
constexpr int kTileI = 32, kTileJ = 16;

// How a wave's lanes walk one cell's velocities (Walk in dvm_walk.h).
// In units of V adjacent velocities (V = 2 in FP32 with an even n1), a grid
// row holds na units.  Walk i of `isteps` gives lane l the unit
// k = i ks + l, column m + i as and row r of r = k / width, m = k % width,
// and then every `brow`-th row below it: tq (+ 1 for i < tr) steps.
struct LaneMap {
    int width, ks, as, rows; // lanes with r >= rows run along outside the grid
    float inv_width;
    int isteps, tq, tr, brow;
    int n1p, n2p;            // LDS table sizes: columns and rows that some lane visits
    int total;               // steps of a row
};

// Two shapes of walk.  "phase": the units in storage order, 64 a step; the
// column of a lane repeats after isteps = na / gcd(64, na) steps, so the steps
// are taken isteps apart; with na odd that is mostly one step a walk (27x31
// velocities 14 walks, 43x39 27), whose lanes then set up a column each step.
// "block": lane rows of la units, 64 / la of them.
// The one with the fewer steps, a walk's own set-up counted a sixteenth of
// a step (an eighth in FP32); a block walk with several pieces per grid row
// touches cache lines twice and counts half more.  Measured on 128x64 cells,
// primal / adjoint us, phase against block: 59x52 velocities in FP64 187 / 267
// against 200 / 287 (48 steps against 52), 43x39 109 / 156 against 139 / 201
// (27 against 39), 10x18 14.5 / 20.9 against 13.6 / 20.4 (3 and 3), FP32
// 62x22 42 / 68 against 35 / 65 (11 and 11).
inline LaneMap lane_map(int n1, int n2, int mixed)
{
    const int V = mixed && n1 % 2 == 0 ? 2 : 1, na = n1 / V;
    int g = kWave, h = na;                      // gcd(64, na)
    while (h) {
        const int t = g % h;
        g = h;
        h = t;
    }
    LaneMap best{};
    const int total = (na * n2 + kWave - 1) / kWave;
    best.width = na;
    best.ks = kWave;
    best.as = 0;
    best.isteps = na / g < total ? na / g : total;
    best.brow = kWave / g;
    best.rows = 1 << 30;
    best.tq = total / best.isteps;
    best.tr = total % best.isteps;
    best.n1p = n1;
    best.n2p = (total * kWave - 1) / na + 1;
    const int setup = mixed ? 2 : 1;
    int cost = 16 * total + setup * best.isteps;
    for (int la = na < kWave ? na : kWave; la >= 1; la--) {
        const int isteps = (na + la - 1) / la, nb = kWave / la, bsteps = (n2 + nb - 1) / nb;
        if (isteps > 1 && la * V * (mixed ? 8 : 16) < 128) break;       // less than a cache line a piece
        const int c = (isteps > 1 ? 24 : 16) * isteps * bsteps + setup * isteps;
        if (c >= cost) continue;
        cost = c;
        best.width = la;
        best.ks = 0;
        best.as = la;
        best.rows = nb;
        best.isteps = isteps;
        best.tq = bsteps;
        best.tr = 0;
        best.brow = nb;
        best.n1p = (isteps * la + 1) * V;       // the last V: lanes outside the rows
        best.n2p = bsteps * nb;
    }
    best.inv_width = 1.0f / best.width;
    best.total = best.tq * best.isteps + best.tr;
    return best;
}

// How the rows of a sweep (of all arrays it touches) meet the 256 MiB
// memory-side cache (MALL), which non-temporal stores bypass:
//   keep    they fit: plain loads and stores (copies of up to 128 MB per
//           buffer run at 8.2 TB/s with plain and 4.7 TB/s with non-temporal
//           stores; 128x64 cells with 1024 velocities in FP64, primal: 57
//           against 76 us)
//   turn    they nearly fit: plain, and every other sweep runs backwards, so
//           that it starts with the rows the last one ended with (256x128
//           cells with 256 velocities in FP64, 268 and 403 MB: primal 67 ->
//           58 us, adjoint 98 non-temporal -> 94 us)
//   stream  non-temporal, so that neighbour rows stay longer in L2 (128x64
//           cells with 4096 velocities in FP32, 537 MB: primal 136 against
//           145 us; the 256x128 C-grid with 2304 velocities in FP64, 2.4 and
//           3.6 GB: 489 and 695 against 501 and 717 us; running backwards
//           every other time 491 and 700)
// A group of a batch goes by its own members' sum, though the other groups'
// rows pass through the cache between two of its sweeps.  Going by the sum over
// all groups measured, us a sweep: 134 + 201 MB 84 -> 85, 201 + 201 MB 99.6 ->
// 102.5, 268 + 403 MB 186 -> 183, 402 + 201 MB 148 -> 145, twice 134 + 201 MB
// 165 -> 158; the code before this rule (all rows non-temporal) 88, 102, 205,
// 152 and 176.
enum { kMemKeep = 0, kMemTurn = 1, kMemStream = 2 };
inline int sweep_memory(size_t bytes)
{
    constexpr size_t mib = size_t(1) << 20;
    return bytes <= 224 * mib ? kMemKeep : bytes <= 448 * mib ? kMemTurn : kMemStream;
}

// Into how many parts a cell's row of `steps` steps is summed (SweepUnit in
// dvm_walk.h), and how many of an XCD's `per` patches, the last ones, are
// swept by one wave a part instead of one a cell.  Measured us, primal /
// adjoint, one wave a cell against this:
//  - few cells (a wave or two per SIMD of the chip): shorter chains of steps.
//    FP64 32x16 cells with 24x24 velocities 9.7 / 11.6 -> 7.4 / 8.4, 64x32
//    with 32x32 15.8 / 22.9 -> 15.4 / 20.1 (with 16x16 7.6 / 8.6 against 8.1
//    / 9.0 in two parts: not worth it).
//  - FP64 rows from memory: a quarter as many cells in flight, so more of
//    their neighbours' rows are still in L2, and a shorter tail of last
//    workgroups.  256x128 with 48x48 488 / 692 -> 468 / 660, with 64x64 sinh
//    857 / 1219 -> 840 / 1145; 128x64 with 64x64 235 / 337 -> 230 / 309, with
//    32x32 in two parts 57 / 95 -> 52 / 86.
//  - FP32 rows from memory: the added set-up costs more than that (256x128
//    with 64x64, all in parts 427 / 602 -> 478 / 634), but a launch of few
//    long rows ends sooner with only its last patches in parts: 128x64 with
//    64x64 136 / 200 -> 126 / 185.
inline void sweep_parts(int nc, int per, int steps, int mixed, int mem, int &parts, int &tail)
{
    parts = 1;
    tail = per;
    if (nc <= 1024 && steps >= 8)
        parts = 4;
    else if ((nc <= 2048 && steps >= 8) || (nc <= 1024 && steps >= 4))
        parts = 2;
    else if (!mixed && (mem == kMemStream || (mem == kMemTurn && nc >= 8192)) && steps >= 14)
        parts = steps >= 32 ? 4 : 2;
    else if (mixed && mem == kMemStream && per <= 512 && steps >= 28) {
        parts = 4;
        tail = per < 96 ? per : 96;
    }
    if (parts == 1) tail = 0;
}

// Everything a kernel needs about one solve, passed by value (single solve)
// or read from a device table (batched).  Pointers are device pointers into
// the solver's workspace.  Storage type of f / phi / fd / gM is float in
// mixed mode and double in FP64 mode.
struct DevSolve {
    int nc, nw, nv, n1, n2;
    int np;                  // patches
    int ni, nj;              // structured grid size (cells along the wall, cells outward)
    int topo;
    int objective;
    int mixed;
    int order;               // spatial order of the scheme: 1, or 2 (reconstructed face values)
    int equil;               // equilibrium: 0 pointwise Maxwellian, 1 discrete-conservative
    int limiter;             // order 2: 0 none, 1 Venkatakrishnan
    int mem[2];              // sweep_memory of the primal and the adjoint
    int parts[2], tail[2];   // sweep_parts of the primal and the adjoint
    LaneMap lm;
    // mesh
    const int32_t *nbr;      // [nc][4] (device cell numbering)
    const int32_t *patch;    // [np + 1] first cell of each patch; patch p = cells [patch[p], patch[p+1])
    const int32_t *cell_of;  // [nc] mesh cell number (i + ni*j) of each device cell
    const double *S;         // [nc][4][2]
    const double *vol;       // [nc]
    const int32_t *wall_cell;// [nw]
    const double *wall_A;    // [nw]
    const double *wall_n;    // [nw][2]
    const double *wall_a;    // [nw][2]
    const double *wall_b;    // [nw][2]
    const double *D;         // [nw] eq. (barg) normaliser
    // velocity grid (1-D factors)
    const double *vx, *vy, *wx, *wy;
    const void *fd;          // [nv][2] far-field values (storage type)
    const void *gM;          // [nv]    g_M1(1, 0, theta_w) (storage type)
    const void *gw2;         // [nv][2] (g_M1, theta_w/2 g_M1)(1, 0, theta_w) (storage type)
    // flow
    double inv_tau_inf, u_inf, theta_w, cd_scale;
    // primal state (ping-pong)
    void *f[2];
    double *W[2];            // [nc][4]
    double *F[2];            // [nw]
    double *red;             // [nc][2] per-cell residual partials of the last sweep
    // adjoint state
    void *phi[2];
    double *aW[2];           // [nc][8]: What (4), rho_tau, pad
    double *Phi[2];          // [nw]
    const void *fstar;       // frozen primal f (= f[primal parity at adjoint init])
    double *acoef;           // [nc][kAcoef] per-cell adjoint coefficients (see k_adjoint_coef)
    // sensitivity / objective
    double *Jl;              // [nw]
    double *sens;            // [nw][5]: S_A, S_x(2), S_n(2)
    double *dJdn;            // [nw][2]
    double *jac;             // [nw][2][kMaxParams]
    double *dJda;            // [kMaxParams]
    double *msens;           // [nc][4][2] per mesh cell: dL/d(corner coordinates)
    double *dJdx;            // [(nj+1)(ni+1)][2] dL/d(node coordinates), mesh node numbering
    double *out;             // [16] small scalar outputs
    // second-order scheme (order 2 only; null otherwise)
    const double *rf;        // [nc][4][2] face midpoint minus the cell's centroid
    const double *rn;        // [nc][4][2] face midpoint minus the neighbour's centroid (interior faces)
    void *G;                 // [nc] rows of 4 nv: limited slopes, adjoint: B (storage type; order in a row: Slopes)
    void *corr;              // [nc][nv][2] held flux correction c; adjoint: held term E (storage type)
    void *psi;               // [nc][nv][2] limiter factors of the frozen f (storage type)
    double *dF;              // [nw] held wall-flux correction
    // macroscopic prediction (primal acceleration; null when off)
    double *mstate;          // [nc][kEqState] equilibrium parameters P' and dP'/dW (conservative equilibrium)
    double *mr;              // [nc][4] moments of the kinetic residual
    double *mDinv;           // [nc][16] inverse of the cell's own block
    double *mO;              // [nc][4][16] outflow block of each face (dg/dW form)
    double *mx[2];           // [nc][4] red-black iterates
};

// dynamic LDS of the patch kernels (layouts in dvm_walk.h and dvm_kernels.hip); a thread of
// the adjoint's parks kWalkSums sums there between walks
constexpr int kWalkSums = 6;
inline unsigned factor_lds(const LaneMap &m) { return 32u * m.n2p + 16u * m.n1p; }
inline unsigned primal_lds(const DevSolve &d)
{
    const unsigned tables = factor_lds(d.lm) + kPatchCells * (d.lm.n1p + d.lm.n2p) * (d.mixed ? 4u : 8u);
    const unsigned sums = d.parts[0] > 1 ? kPatchCells * kWave * 8u : 0u;   // join_parts
    return tables > sums ? tables : sums;
}
inline unsigned adjoint_lds(const DevSolve &d)
{
    return kWalkSums * 8u * kPatchCells * kWave + factor_lds(d.lm) + kPatchCells * (d.lm.n2p * (32u + (d.mixed ? 4u : 8u)) + d.lm.n1p * 8u);
}

// launches (all on `st`); par = index of the current f / phi buffer; res:
// the adjoint sweep also leaves its residual partials
hipError_t launch_primal_init(const DevSolve &d, hipStream_t st);
hipError_t launch_primal_sweep(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_moments(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_residual(const DevSolve &d, int adjoint, hipStream_t st);
hipError_t launch_objective(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_adjoint_init(const DevSolve &d, int fpar, hipStream_t st);
hipError_t launch_adjoint_sweep(const DevSolve &d, int par, int res, hipStream_t st);
// adjoint moments (What, rho_tau) and wall multipliers of phi[par] (a loaded phi)
hipError_t launch_adjoint_moments(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_adjoint_correct_moments(const DevSolve &d, int par, const double *z, hipStream_t st);
hipError_t launch_eq_params(const DevSolve &d, int par, int with_M, hipStream_t st);
hipError_t launch_wall_sens(const DevSolve &d, int fpar, int ppar, int n_params, hipStream_t st);
hipError_t launch_mesh_sens(const DevSolve &d, int fpar, int ppar, hipStream_t st);
// macroscopic prediction of the moments W[par] of f[par] (first-order
// scheme): assembly, `inner` red-black block Gauss-Seidel steps, limited
// update of W[par]
hipError_t launch_macro_predict(const DevSolve &d, int par, int inner, hipStream_t st);
// adjoint prediction: the system at the frozen f[fpar] and its transpose
// (at the adjoint's start); every K adjoint sweeps, A^T dl = -r* and What of
// phi[ppar] += dl
hipError_t launch_macro_adjoint_setup(const DevSolve &d, int fpar, hipStream_t st);
hipError_t launch_macro_adjoint_predict(const DevSolve &d, int ppar, int inner, hipStream_t st);
// A group of batch members for one launch: member a is tab[idx[a]], owns
// items (cells or tiles) pre[a] .. pre[a+1]-1 of the launch; its state is in
// buffer par[a] and its mesh has ni[a] x nj[a] cells.
constexpr int kMacroGroup = 64;
struct MacroGroup {
    int n;
    int idx[kMacroGroup];
    int par[kMacroGroup];
    int ni[kMacroGroup], nj[kMacroGroup];
    int pre[kMacroGroup + 1];
};
// `steps` Gauss-Seidel half steps of a launch, the first of colour `colour`;
// first / last of the iteration
constexpr int kGsMaxSteps = 8;
struct GsStep {
    int steps, colour, first, last;
};
// one prediction in parts, for members of a batch; `from`: the buffer mx the
// Gauss-Seidel launches left the increment in
hipError_t launch_macro_predict_begin(const DevSolve &d, int par, int inner, hipStream_t st);
hipError_t launch_macro_predict_end(const DevSolve &d, int par, int from, hipStream_t st);
hipError_t launch_macro_adjoint_begin(const DevSolve &d, int pnew, int inner, hipStream_t st);
hipError_t launch_macro_adjoint_end(const DevSolve &d, int pnew, hipStream_t st);
hipError_t launch_macro_gs_group(const DevSolve *tab, MacroGroup g, int inner, int adjoint, int *from, hipStream_t st);
hipError_t launch_eq_params_group(const DevSolve *tab, const MacroGroup &g, int with_M, hipStream_t st);

// second-order scheme: the slopes G and dF of f[par]; the held primal
// correction c (with G and dF) from f[par]; the
// limiter factors psi of f[fpar] for the adjoint; the held adjoint term E
// from phi[par]; the drag with reconstructed wall values (per element)
hipError_t launch_so_slopes(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_so_correction(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_so_freeze(const DevSolve &d, int fpar, hipStream_t st);
hipError_t launch_so_adjoint_term(const DevSolve &d, int par, hipStream_t st);
hipError_t launch_so_objective_elem(const DevSolve &d, int par, hipStream_t st);

// batched: table of DevSolve on the device, per-block (solve, patch) map,
// per-solve buffer parity at batch creation; step = sweeps done since batch
// creation; adjoint selects the kernel of that phase, so the scheme (the
// blocks of one launch are members of one phase and one scheme)
struct BatchLaunch {
    int blocks = 0, mixed = 0, adjoint = 0, so = 0, mem = 0;
    int parts = 0;           // some member's rows are summed in parts
    unsigned lds = 0;        // the largest member's
};
hipError_t launch_batch(const DevSolve *tab, const int32_t *blk_solve, const int32_t *blk_patch,
                        const int32_t *par0, int step, const BatchLaunch &g, int res, hipStream_t st);
hipError_t launch_batch_residual(const DevSolve *tab, int n, double *out, hipStream_t st);

// The allocation-free batch (dvm_batch_create_static) keeps its launch
// tables in one fixed device array per GPU, of kStaticBatchBytes, for at
// most kStaticBatchMaxMembers members.  static_batch_scratch gives the
// current device's copy of the array (its address is looked up once per
// device); launch_batch_tables writes the per-workgroup (member, patch) map
// of the four groups (group g = 2 * phase + (order == 2), nb_group[g]
// workgroups each, in that order) from the member table and phases, in the
// layout dvm_batch_create builds on the host.
constexpr size_t kStaticBatchBytes = size_t(8) << 20;
constexpr int kStaticBatchMaxMembers = 64;
hipError_t static_batch_scratch(char **out);
hipError_t launch_batch_tables(const DevSolve *tab, const int32_t *phase, int n, const int *nb_group,
                               int32_t *blk_solve, int32_t *blk_patch, hipStream_t st);


// radial-basis-function mesh motion (Wendland C0, support 1/inv_r):
// apply: out[n] = wall[widx[n]] for wall nodes, else x0[n] + sum_w gamma[w]
// phi(|x0[n] - c[w]| inv_r); chain: h[w] = sum over non-wall nodes n of
// phi(|x0[n] - c[w]| inv_r) g[n], via per-chunk partials part[chunk][nw]
// summed in chunk order.  Points are double2 = (x, y).
constexpr int kRbfChainNodes = 256;    // nodes per workgroup of the chain kernel
constexpr int kRbfTile = 64;           // centres per workgroup of the chain kernel
inline int rbf_chunks(int nn) { return (nn + kRbfChainNodes - 1) / kRbfChainNodes; }
hipError_t launch_rbf_apply(const double *x0, const int32_t *widx, int nn, const double *c,
                            const double *gamma, const double *wall, int nw, double inv_r, double *out,
                            hipStream_t st);
hipError_t launch_rbf_chain(const double *x0, const int32_t *widx, const double *g, int nn, const double *c,
                            int nw, double inv_r, double *part, double *h, hipStream_t st);

// for host sources other than dvm_host.cpp: set the thread's error message
// (returns code), and the node grid of a mesh
int set_error(int code, const char *fmt, ...);
struct MeshNodes {
    int topo, ni, nj, nwake, nw;
    const double *nodes;     // [(nj+1)(ni+1)][2]
};
MeshNodes mesh_nodes(const dvm_mesh *m);

}  // namespace dvm
