// Argument blocks of the per-step march kernels.
#pragma once

#include "mj_internal.h"

namespace mj {

constexpr int kMaxLocal = 64;   // largest history depth kept in real space

struct MacArg {
    const double *Khat;      // [nk][Nz/2+1][Ny/2+1][Hp][6] real, lags 1..nk
    const double2 *ring_base;// [ring][nrhs][3][Nz][Ny][Hp]
    double2 *Shat;           // [nrhs][3][Nz][Ny][Hp]
    int Hx, Hp, Ny, Nz;      // Hx = Nx/2 + 1 frequencies in rows of pitch Hp
    int nk;                  // number of lags summed (1..nk)
    int ring;                // ring slots
    int slot_nm1;            // slot of Jhat_{n-1}
    int nrhs;
};

struct BlockMacArg {
    const double *Khat;        // [ell][Nz/2+1][Ny/2+1][Hp][6]
    const double2 *ring_base;  // [ring][nrhs][3][Nz][Ny][Hp]
    double2 *far;              // [TB][nrhs][3][Nz][Ny][Hp]
    int Hx, Hp, Ny, Nz;        // Hx = Nx/2 + 1 frequencies in rows of pitch Hp
    int nk;                    // ell (far: lags 1..nk)
    int ring;
    int nb;                    // first step of the block
    int ntarget;               // targets written by the far kernel (<= TB)
    int t;                     // near: position of the step in the block
    int nrhs;
    int jmin;                  // far: sources before step jmin count as zero (<= 1: none dropped)
    const double2 *init;       // far: partial sums the targets start from, laid out like far (NULL: zero)
    int jmax;                  // windowed far kernel: sources after step jmax count as zero (<= 0: none
                               // dropped); its lag loop then starts at nb - jmax
};

constexpr int kMaxSeries = 16;   // highest power of x^2 in a wave's series

struct WaveArg {
    double k[3], pol[3], rref[3];
    double width, ct0, amp;
    // How the voxel average is taken (set by the host from the spreads |k_i| h_i / width): form 3 a series in
    // the Gaussian's derivatives, coefficients ser[0 .. ns] of the polynomial in x^2 that multiplies
    // exp(-x^2); else, with two or more non-zero direction components, the axes by decreasing spread enter as
    // their products k_i h_i, and form 1 takes erf on the widest and a Gauss-Legendre rule of nq points on
    // the other two, 2 the two widest in closed form and the rule on the third; form 0 is the 8-point rule
    // along the one axis of the wave.
    double kh[3];
    int nq[3];
    int form;
    int ns;
    double ser[kMaxSeries + 1];
};

struct EpiArg {
    long M;
    int U, V, W;
    int nrhs;
    int n;                   // current step
    double h, hy, hz, c_dt;  // voxel edges (x, y, z) and c dt
    const double *chi, *schi, *inv_eps;
    const double *fir;       // device taps (nfir)
    int nfir;
    int nloc;                // local history depth used (>= nguess)
    int slot_of[kMaxLocal + 1];  // real-ring slot of J_{n-k}, k = 1..nloc
    int nguess;              // the solve starts from sum_{k=1}^{nguess} gx[k-1] J_{n-k} (<= nloc)
    double gx[kMaxLocal];    // extrapolation weights (the polynomial through nguess past steps)
    const double *Jring;     // [depth][nrhs][3][M]
    const double *S;         // [nrhs][3][M] convolution (normalised) or NULL at n = 1
    const WaveArg *waves;    // [nrhs]
    double glx8[8], glw8[8]; // 8-point rule on [-1/2, 1/2], weights summing to 1
    const double *gl;        // n-point rules on [-1/2, 1/2], n = 1..8: row n holds 8 nodes then 8 weights
    double *b;               // right-hand side of the Z_0 system, haloed [nrhs][3][(W+2)(V+2)(U+2)]
    double *w0;              // extrapolated J_n the solve starts from, same layout
    // transposed march only
    const double *Lring;     // lambda history [depth][nrhs][3][M] (the local terms act on lambda)
    const double *G;         // adjoint source g_j [nrhs][3][M]
    double *bq;              // b'_j, kept for the voxels with chi = 0 [nrhs][3][M]
    const double *k0;        // the solver's K_0 stencil (the gradient term B_n)
    int series;              // every wave takes its average by the series (form 3)
};

// Adjoint of the probe objective and the eps-gradient (see mj_march.hip).
struct AdjArg {
    long M;
    int U, V, W, nrhs;
    // adjoint source from the stored probe field
    const double *table_v;   // probe kernel table by voxel: [nw][np][M][6] (zeros where there is no pair)
    const int *kmin_v;       // [np][M] first lag of the pair's window, -1 if no pair
    const double *Ehist;     // [N][nrhs][np][3]
    int np, nw, N, j;        // j: forward step of this adjoint step (the source: the first of ntarget,
                             // j, j - 1, ...)
    int ntarget;             // steps the source is formed for, at most kProbeSteps
    double *G;               // out [nrhs][3][M]; the source: [ntarget][nrhs][3][M]
    // lambda from the solve
    const double *schi, *c0, *bq, *nu;   // nu: [nrhs][3][M] of this step
    double *lam;             // out [nrhs][3][M]
    // gradient
    const double *Bj;        // B_j [nrhs][3][M]
    const double *inv_eps;
    double *grad;            // [M], accumulated
    const double *k0;        // the solver's K_0 stencil (the adjoint's local term)
};

struct CgScalars {
    double rz[2];            // r.z of the current and the previous iteration (alternating slots)
    double pq, rr, bb;
    int conv;                // iteration whose convergence test passed (INT_MAX: none yet)
};

// per right-hand side, read back by the host in one copy
struct CgStatus {
    int done;                // the last test passed
    int ended;               // CG: no further iteration runs (the stopping residual is reached)
    int iters;               // iterations taken
    double res;              // relative residual |r| / |b| at the last test (passes: of the iterate before the
                             // one they leave)
    double bb;               // |b|^2 of the solve's right-hand side (growth detector)
};

// Coefficients of a three-term iteration, (a_k, b_k) per pass k, and the squared relative residual
// |r_k|^2 / |b|^2 that CG saw before pass k.
constexpr int kMaxCoef = 192;

struct CgArg {
    long M;
    int U, V, W;
    long Mp;                 // (U+2)(V+2)(W+2): vectors read by the stencil carry a zero halo
    int nrhs, nblk;          // nblk = ceil(M / 256): one voxel per thread
    double tol2;             // squared relative residual of the convergence test
    double stop2;            // ... at which the iteration ends (<= tol2)
    double d0, k0c;          // delta_0 and K_0^{xx}(0): c_0 and diag(A) follow from sqrt(chi)
    const double *schi;
    const double *b, *w;     // right-hand side and the current the solve starts from, haloed [nrhs][3][Mp]
    double *y, *p, *q, *u;   // u = sqrt(chi) M^-1 r stands for the residual r (haloed)
    double *part;            // [nrhs][3][nblk]
    CgScalars *scal;         // [nrhs]
    CgStatus *stat;          // [nrhs]
    double *coef;            // [nrhs][kMaxCoef][2]: receives the three-term coefficients of each iteration (or NULL)
    double *rhist;           // [nrhs][kMaxCoef]: and its relative residuals (or NULL)
    // the solver's K_0(D) on its 27-point support [27][6] in device memory: entry
    // 13 + dx + 3 dy + 9 dz, components xx yy zz xy xz yz; read through the scalar cache
    const double *k0;
};

// One pass of a three-term iteration on Z_0 J = b with given coefficients (see mj_march.hip): no inner
// products, one stencil application per pass.
struct PassArg {
    int px, py, pz;          // U + 2, V + 2, W + 2
    long Mp;
    double d0, k0c, tol2;
    const double *chi;       // haloed [Mp], zero in the halo
    const double *b;         // haloed [nrhs][3][Mp]
    const double *w;         // w_k
    double *v;               // w_{k-1} in, w_{k+1} out
    const double *k0;
    const double *coef;      // (a_k, b_k) of right-hand side r at coef + r coef_stride + 2 k
    long coef_stride;
    int coef_len;            // entries that coef holds
    int k;                   // this pass's entry
    int first;               // the first pass of a solve: there is no w_{k-1}
    int want_norm;           // sums |r_k|^2 and |b|^2 of w_k, and the test follows the pass
    int rhs0, nr;            // the right-hand sides rhs0 .. rhs0 + nr - 1
    double *part;            // [nrhs][2][blocks]
    int part_cap;            // values per right-hand side that part holds
    CgStatus *stat;          // [nrhs]
};
// blocks that a pass over nr right-hand sides takes for each of them
int z0_pass_blocks(int U, int V, int W, int nr);
// passes: those taken before this one, for the status that the test leaves
void launch_z0_pass(const PassArg &a, int passes, hipStream_t st);
// pseudo-random right-hand side (zero where sqrt(chi) = 0), haloed
void launch_fill_trial(const double *schi, int U, int V, int W, double *b, hipStream_t st);

// Scattered field at probe points: E^s_p(n) = sum_{k=0}^{ell} sum_s K_k(r_p - r_s) J_{n-k}(s)
// over the source voxels s of the scatterer, for the ntarget steps n0 .. n0 + ntarget - 1 at once.  Pairs
// (p, s) are stored per probe sorted by the first lag kmin of their window of nw lags; the host cuts each
// probe's pairs into chunks for the waves.
constexpr int kProbeChunk = 128;    // pairs handled by one wave
constexpr int kProbeSteps = 8;      // steps taken together
struct ProbeStepArg {
    const double *table;     // [nw][npairs][6], zero for lags above ell
    const int *pair_vox;     // [npairs]
    const int *pair_kmin;    // [npairs]
    int np, nw, nrhs, n0, ntarget;
    int ell;                 // last lag
    // chunk c covers pairs [ck_lo[c], ck_hi[c]) of one probe; probe p owns chunks [ck_start[p], ck_start[p + 1])
    const int *ck_lo, *ck_hi, *ck_start;
    long nck;
    long M, npairs;
    const double *Jring;     // [rdepth][nrhs][3][M], rdepth > ell + ntarget - 1
    int rdepth;
    double *part;            // [nrhs][nck][kProbeSteps][3]
    double *out;             // [ntarget][nrhs][np][3]
};

void launch_mac(const MacArg &a, hipStream_t st);
void launch_mac_far(const BlockMacArg &a, int tb, hipStream_t st);
void launch_probes(const ProbeStepArg &a, hipStream_t st);
void launch_grad_term(const EpiArg &e, const double *Jn, const double *Jn1, double *Bout, hipStream_t st);
void launch_adj_source(const AdjArg &a, hipStream_t st);
// table_v[wl][p][m] = table[wl][inv[p][m]], kmin_v[p][m] = pair_kmin[inv[p][m]] (-1, zeros where none)
void launch_probe_table_by_voxel(const double *table, const int *pair_kmin, const int *inv, long npairs, int np,
                                 int nw, long M, double *table_v, int *kmin_v, hipStream_t st);
void launch_adj_epilogue(const EpiArg &e, hipStream_t st);
void launch_adj_lambda(const AdjArg &a, hipStream_t st);
void launch_grad_accum(const AdjArg &a, hipStream_t st);
void launch_mac_near(const BlockMacArg &a, hipStream_t st);
// far part with the rotation-free source window: tb = 4, 8, 10, 12, 14 or 16 targets
void launch_mac_win(const BlockMacArg &a, int tb, hipStream_t st, size_t lds_reserve = 0);
void launch_epilogue(const EpiArg &e, hipStream_t st);
void launch_history_local(const double *Jh, int depth, const double *S, const double *chi, const double *inv_eps,
                          const double *fir, int nfir, long M, double *P, hipStream_t st);
void launch_cg_init(const CgArg &a, hipStream_t st);
void launch_cg_a(const CgArg &a, int it, hipStream_t st);
void launch_cg_b(const CgArg &a, int it, hipStream_t st);
void launch_cg_end(const CgArg &a, int it, hipStream_t st);
// J_n = sqrt(chi) y (w NULL) or w, haloed, into the real-space ring and, if not NULL, Jout
void launch_cg_finish(const double *y, const double *schi, const double *w, int U, int V, int W, int nrhs, double *J,
                      double *Jout, hipStream_t st);

}  // namespace mj
