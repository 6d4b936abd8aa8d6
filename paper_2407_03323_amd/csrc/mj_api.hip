// C interface and host orchestration of the MOT-JVIE march (see include/motjvie.h).
#include "motjvie.h"
#include "mj_march.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

using mj::ArgError;
using mj::HipError;
using mj::MemError;
using mj::UnstableError;

namespace {

thread_local std::string g_err;

// voxels (per right-hand side) up to which z0_solver = 0 takes the Chebyshev solve
constexpr long kChebMaxUnknowns = 1L << 19;
// bytes of solve vectors per group of right-hand sides that three-term passes take at once: what they
// stream (w_k, w_{k-1} and b, 72 bytes per voxel and right-hand side) stays in the 256 MB last-level cache
// from one pass to the next
constexpr size_t kPassGroupBytes = 190000000;

// entries of the Chebyshev iteration's coefficient table, at most (cg_maxit may be any number)
constexpr int kChebCoefMax = 65536;

constexpr int kStepEvents = 9;   // events of a timed step (see StepIO)

// whether outer_overlap = 0 runs the outer level of three on the second stream
constexpr bool kOverlapDefault = false;
// LDS each block of the second stream's launch claims: above half of a CU's 160 KB, so that a
// CU holds one such block (one wave per SIMD) and keeps room for the march's kernels
constexpr size_t kSideLdsReserve = 96 * 1024;

// ---------------------------------------------------------------------------- static staging
// mj_kernel_values_noalloc stages its requests and results through this file-scope array
// instead of allocating: kNoAllocMax requests, laid out as results [max][6] doubles, then
// lags [max] and offsets [max][3] as int32.  Every GPU the library runs on holds its own copy
// until the process ends.  In host code the name `scratch` is only a stand-in: the array's
// device address is looked up per device with hipGetSymbolAddress (with that device
// current) and kept in g_scratch; host code passes that address, never the name.
constexpr int kNoAllocMax = 65536;
constexpr size_t kNoAllocBytes = (size_t)kNoAllocMax * (6 * sizeof(double) + 4 * sizeof(int32_t));
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

std::mutex g_scratch_mu;                 // guards g_scratch
std::vector<unsigned char *> g_scratch;  // device address of `scratch` per device id (null: not looked up)
std::mutex g_noalloc_mu;                 // calls of one process take turns on the staging array

// Address of this device's copy of `scratch`; dev must be the current device.
unsigned char *scratch_ptr(int dev)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch.size() <= dev) g_scratch.resize((size_t)dev + 1, nullptr);
    if (!g_scratch[(size_t)dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            throw HipError(std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch[(size_t)dev] = (unsigned char *)ptr;
    }
    return g_scratch[(size_t)dev];
}

__global__ void k_extract_octant(const double2 *__restrict__ X, int Hx, int Hp, int Ny, int Nz, double scale,
                                 double *__restrict__ out)
{
    const int Nyo = Ny / 2 + 1, Nzo = Nz / 2 + 1;
    const long n = (long)Hp * Nyo * Nzo;
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int kx = (int)(t % Hp), qy = (int)((t / Hp) % Nyo), qz = (int)(t / ((long)Hp * Nyo));
    const long plane = (long)Nz * Ny * Hp;
    for (int c = 0; c < 6; c++)
        out[6 * t + c] = kx < Hx ? scale * X[c * plane + ((long)qz * Ny + qy) * Hp + kx].x : 0.0;
}

struct Events {
    std::vector<hipEvent_t> ev;
    void ensure(size_t n)
    {
        while (ev.size() < n) {
            hipEvent_t e;
            MJ_CHECK(hipEventCreate(&e));
            ev.push_back(e);
        }
    }
    ~Events()
    {
        for (auto e : ev) (void)hipEventDestroy(e);
    }
};

}  // namespace

// n-point Gauss-Legendre rule on [-1/2, 1/2] (Newton on P_n from the Chebyshev-like start),
// weights summing to 1
static void gl_half(int n, double *x, double *w)
{
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int i = 0; i < n; i++) {
        long double zz = cosl(pi * (i + 0.75L) / (n + 0.5L));
        long double dp = 0;
        for (int itn = 0; itn < 50; itn++) {
            long double p0 = 1, p1 = zz;
            for (int j = 2; j <= n; j++) {
                long double p2 = ((2 * j - 1) * zz * p1 - (j - 1) * p0) / j;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (zz * p1 - p0) / (zz * zz - 1);
            long double d = p1 / dp;
            zz -= d;
            if (fabsl(d) < 1e-19L) break;
        }
        x[i] = n == 1 ? 0.0 : (double)(0.5L * zz);
        w[i] = n == 1 ? 1.0 : (double)(1.0L / ((1 - zz * zz) * dp * dp));
    }
}

// Gauss-Legendre order for averaging exp(-((T - k h x) / w)^2) over x in [-1/2, 1/2] with spread
// s = |k| h / w: the least n <= 8 (the most the device tables hold) whose remainder bound
// (n!)^4 / ((2n + 1) ((2n)!)^3) s^2n max|H_2n(x) exp(-x^2)|, with Cramer's bound
// |H_m(x)| exp(-x^2 / 2) <= 1.0865 sqrt(2^m m!), stays below 2^-53, or 9 when none does.  0 spread takes the 1-point rule, which is then exact.
static int gl_order(double s)
{
    if (s == 0.0) return 1;
    for (int n = 1; n <= 8; n++) {
        double f = 1.0, f2 = 1.0;
        for (int i = 2; i <= n; i++) f *= i;
        for (int i = 2; i <= 2 * n; i++) f2 *= i;
        const double c = std::pow(f, 4) / ((2 * n + 1) * f2 * f2 * f2) * 1.0865 * std::sqrt(std::ldexp(f2, 2 * n));
        if (c * std::pow(s, 2 * n) <= std::ldexp(1.0, -53)) return n;
    }
    return 9;
}

// The averaging plan of a wave on voxels of edges (h, hy, hz); see the fields of WaveArg.
static void plan_wave(mj::WaveArg &w, double h, double hy, double hz)
{
    const double kh[3] = {w.k[0] * h, w.k[1] * hy, w.k[2] * hz};
    int ax[3] = {0, 1, 2};
    std::stable_sort(ax, ax + 3, [&](int a, int b) { return std::fabs(kh[a]) > std::fabs(kh[b]); });
    int order[3];
    for (int i = 0; i < 3; i++) {
        w.kh[i] = kh[ax[i]];
        order[i] = gl_order(std::fabs(kh[ax[i]]) / w.width);
        w.nq[i] = std::min(order[i], 8);
    }
    // the series: c_j up to well beyond what kMaxSeries terms can leave out
    constexpr int J = 48;
    std::vector<long double> c(J + 1, 0.0L), f(J + 1), q(J + 1);
    c[0] = 1.0L;
    for (int i = 0; i < 3; i++) {
        const long double a = 0.5L * std::fabs(kh[i]) / w.width;
        f[0] = 1.0L;
        for (int m = 1; m <= J; m++) f[m] = f[m - 1] * a * a / ((2.0L * m) * (2.0L * m + 1.0L));
        for (int j = 0; j <= J; j++) {
            q[j] = 0.0L;
            for (int m = 0; m <= j; m++) q[j] += c[m] * f[j - m];
        }
        c = q;
    }
    // terms left out, largest index first: c_j max|H_2j exp(-x^2)|
    long double left = 0.0L;
    int ns = J;
    for (; ns > 0; ns--) {
        long double root = 1.0865L;   // sqrt(2^2j (2j)!)
        for (int i = 1; i <= 2 * ns; i++) root *= std::sqrt(2.0L * i);
        if (!(left + c[ns] * root <= std::ldexp(1.0L, -53))) break;   // also where c overflows (no number)
        left += c[ns] * root;
    }
    if (ns <= mj::kMaxSeries) {
        // sum_j c_j H_2j(x) as a polynomial in x^2, H_{n+1} = 2 x H_n - 2 n H_{n-1}
        std::vector<long double> poly(ns + 1, 0.0L), h0(2 * ns + 2, 0.0L), h1(2 * ns + 2, 0.0L);
        h0[0] = 1.0L;
        h1[1] = 2.0L;
        for (int n = 0; n <= 2 * ns; n++) {   // h0 = H_n, h1 = H_{n+1}
            if (n % 2 == 0)
                for (int i = 0; i <= n; i += 2) poly[i / 2] += c[n / 2] * h0[i];
            std::vector<long double> h2(2 * ns + 2, 0.0L);
            for (int i = 0; i + 1 < 2 * ns + 2; i++) h2[i + 1] = 2.0L * h1[i];
            for (int i = 0; i < 2 * ns + 2; i++) h2[i] -= 2.0L * (n + 1) * h0[i];
            h0 = h1;
            h1 = h2;
        }
        w.form = 3;
        w.ns = ns;
        for (int i = 0; i <= ns; i++) w.ser[i] = (double)poly[i];
        return;
    }
    w.form = (kh[0] != 0.0) + (kh[1] != 0.0) + (kh[2] != 0.0) < 2 ? 0 : order[1] > 8 ? 2 : 1;
}

struct mj_solver {
    // geometry and configuration
    int U = 0, V = 0, W = 0;
    long M = 0;
    double h = 1.0, hy = 1.0, hz = 1.0, c_dt = 1.0;
    int nrhs = 1, ell = 0;
    int Nx = 0, Ny = 0, Nz = 0, Hx = 0, Hp = 0;
    std::vector<double> fir;
    double cg_rtol = 1e-13;
    int cg_maxit = 200;
    int B = 1;                      // steps per (inner) time block
    int B2 = 0;                     // steps per outer time block (three levels), 0: two levels
    int nquad = 0;                  // quadrature points per cell of the kernels (0: by distance)
    hipStream_t st = nullptr;
    int nloc = 5, rdepth = 6;
    int sdepth = 6;                 // steps of the real-space history that later steps read, and that a state
                                    // holds (with probes the ring holds kProbeSteps - 1 more)
    // degree of the extrapolated initial guess of the Z_0 solve (at most; the steps it goes through
    // are those the taps read anyway, and seven at least).  Iterations with degree 4, 6 and 8: 104^3
    // 16, 14, 12; 64^3 21, 19, 18; 32^3 24, 23, 23.  At 104^3 degree 10 took more again: higher
    // degrees amplify the rounding noise of the history
    int guess_deg = 8;
    // device state
    mj::DevAlloc da;                // hipMalloc, or the caller's allocator (mj_config.alloc)
    size_t bytes = 0;
    std::vector<void *> allocs;
    double *chi = nullptr, *schi = nullptr, *inv_eps = nullptr, *c0 = nullptr;
    double *fir_d = nullptr;
    double *Khat = nullptr;
    double2 *ring = nullptr, *Shat = nullptr, *farbuf = nullptr;
    double2 *gbuf = nullptr;        // outer-block partial sums [B2][nrhs][3][plane] (three levels)
    // Overlapped outer level (three levels): while an outer block marches, a second stream forms
    // the next block's outer sums over the sources before the current block; at the next block
    // start the sources of the block just marched are added on the caller's stream.
    bool overlap = false;
    double2 *hbuf = nullptr;        // those sums [B2][nrhs][3][plane], of the block starting at h_block
    int h_block = 0;                // 0: hbuf holds no block's sums
    hipStream_t side = nullptr;     // the library's second stream (non-blocking, default priority)
    hipEvent_t ev_main = nullptr, ev_side = nullptr;
    bool side_pending = false;      // work on `side` may still run: `st` waits for ev_side first
    static constexpr int kSideTimers = 8;
    hipEvent_t side_t[kSideTimers][2] = {};   // start and end of recent launches on `side`
    bool side_busy[kSideTimers] = {};
    int side_count = 0, side_done = 0;
    double side_ms = 0.0;
    double *S = nullptr, *Jr = nullptr;
    double *y = nullptr, *p = nullptr, *q = nullptr, *u = nullptr;   // CG's vectors
    double *bh = nullptr;           // right-hand side of the solve, haloed
    double *wbuf[2] = {};           // w_k and w_{k-1} of the three-term passes, haloed; wbuf[0] starts the solve
    double *chih = nullptr;         // chi, haloed
    const double *w_end = nullptr;  // solution of the last solve: a wbuf, or NULL: sqrt(chi) y
    double *parts = nullptr;
    int part_cap = 0;               // values per right-hand side in parts
    mj::CgScalars *scal = nullptr;
    int cg_guess = 8;
    // Z_0 solver: 0 Chebyshev iteration (needs spectral bounds of M^-1 A), 1 CG; with `replays` that one only
    // stands behind the replayed passes
    int z0_method = 0;
    bool replays = false;
    struct Replay {                 // see solve_z0
        int K = 0;                  // passes before the first test
        int K0 = 0;                 // ... as CG left it
        int L = 0;                  // passes with coefficients
        int learn = 1;              // the next solve takes CG and records it
        int fails = 0;              // replays in a row that missed the tolerance
        int hold = 0;               // steps left without replays
        int unused[2] = {};
    } rp;
    static constexpr int kMaxFails = 6;   // misses that lengthen the pause (to 4 << kMaxFails steps)
    double *coef = nullptr;         // recorded coefficients [nrhs][kMaxCoef][2]
    double *rhist = nullptr;        // and relative residuals [nrhs][kMaxCoef]
    double *ccoef = nullptr;        // coefficients of the Chebyshev iteration [ccoef_len()][2]
    double lam_lo = 0.0, lam_hi = 0.0;   // bounds of the eigenvalues of M^-1 A (0: not estimated)
    int cheb_pred = 0;                   // passes predicted for the next Chebyshev solve (0: none yet)
    bool use_graphs = false;             // launch batches of passes from captured HIP graphs
    hipStream_t cap_st = nullptr;        // the library's own stream, for capturing (never the null stream)
    std::map<long, hipGraphExec_t> pass_graphs;   // captured batches by (group, coefficients, first pass, passes)
    mj::CgStatus *cgstat = nullptr, *cgstat_h = nullptr;
    hipEvent_t ev_status = nullptr;
    mj::WaveArg *waves_d = nullptr;
    bool waves_set = false;
    std::vector<mj::WaveArg> waves;
    mj::Fft3D fft{};
    mj::GenResult gen{};
    double K0_27[27 * 6] = {};
    double *k0_d = nullptr;         // K0_27 on the device (the Z_0 stencil of this solver)
    double *gl_d = nullptr;         // Gauss-Legendre rules of 1..8 points for the excitation
    int nblk = 1;
    int n = 0;
    int dev = 0;                    // device current at mj_create
    std::string err;
    // probes: scattered field at test voxels centred at arbitrary points
    std::vector<double> eps_h;
    int np = 0, nw = 0;
    long npairs = 0;
    double *probe_pos = nullptr, *ptable = nullptr, *ppart = nullptr;
    int *pair_vox = nullptr, *pair_kmin = nullptr, *pinv = nullptr;
    int *ck_lo = nullptr, *ck_hi = nullptr, *ck_start = nullptr;   // chunks of the probes' pairs
    double *probe_out = nullptr;    // where the probe field of the steps taken but not yet formed goes
    int probe_n0 = 0, probe_steps = 0;   // those steps
    double *ptable_v = nullptr;   // probe kernel table ordered by voxel (adjoint source)
    int *pkmin_v = nullptr;
    long pnck = 0;
    // transposed march: local history lambda, and the right-hand side before its sqrt(chi) scaling
    double *Lr = nullptr, *bq = nullptr;
    // statistics of the last run
    double t_gen_ms = 0, t_spec_ms = 0, t_probe_ms = 0;
    double t_mac_tune_ms = 0;       // MAC time per step of the timed choice (time_block < 0)
    double stat[21] = {};
    Events events;

    template <class T>
    T *dalloc(size_t count, const char *what)
    {
        size_t b = count * sizeof(T);
        if (b == 0) b = sizeof(T);
        void *ptr = da.get(b, what);
        allocs.push_back(ptr);
        bytes += b;
        return (T *)ptr;
    }

    ~mj_solver()
    {
        if (st) (void)hipStreamSynchronize(st);
        if (side) {
            (void)hipStreamSynchronize(side);
            (void)hipStreamDestroy(side);
        }
        for (hipEvent_t e : {ev_main, ev_side})
            if (e) (void)hipEventDestroy(e);
        for (auto &pr : side_t)
            for (hipEvent_t e : pr)
                if (e) (void)hipEventDestroy(e);
        clear_graphs();
        if (cap_st) (void)hipStreamDestroy(cap_st);
        mj::fft3d_free(fft);
        da.put(gen.moments);
        for (void *a : allocs) da.put(a);
        if (cgstat_h) (void)hipHostFree(cgstat_h);
        if (ev_status) (void)hipEventDestroy(ev_status);
    }

    void dfree(void *&ptr)
    {
        if (!ptr) return;
        for (size_t i = 0; i < allocs.size(); i++)
            if (allocs[i] == ptr) {
                allocs.erase(allocs.begin() + (long)i);
                break;
            }
        da.put(ptr);
        ptr = nullptr;
    }

    long spec_plane() const { return (long)Nz * Ny * Hp; }
    long koct() const { return (long)Hp * (Ny / 2 + 1) * (Nz / 2 + 1); }
    int slotS(int j) const { return j % ell; }
    int slotR(int j) const { return j % rdepth; }

    void create(const mj_config &c);
    void build_spectra();
    void set_material(const double *eps);
    struct StepIO {
        // kStepEvents events, or NULL: 0 - 1 forward transform, 7 - 2 history sum, 2 - 3 inverse transform, 3 - 4
        // right-hand side, 4 - 5 solve and J_n, 8 - 6 probes (recorded if they run)
        hipEvent_t *ev = nullptr;
        bool more = false;              // another step follows in this call, on the same rings; its events are
                                        // ev + kStepEvents
        double *Jout = nullptr;         // forward: J_n copy
        double *Pout = nullptr;         // forward: the probe field of the step goes here (NULL: not formed), once
                                        // kProbeSteps of them are due or flush_probes is called; those of
                                        // successive steps follow each other
        double *Bout = nullptr;         // forward: gradient term B_n
        char *far_kind = nullptr;       // 1 far (outer) launch, 2 near launch, 3 middle launch
        char *probes_ran = nullptr;     // set to 1 if the probe field was formed (events 8 and 6 recorded)
        bool adjoint = false;           // transposed march
        const double *G = nullptr;      // adjoint: source g_j
        const double *Bj = nullptr;     // adjoint: B_j for the gradient (NULL: none)
        double *grad = nullptr;         // adjoint: gradient accumulator
    };
    mj::EpiArg epi_arg() const;
    const double2 *mac(int n, int *kind);
    void outer_sums(int nb, hipStream_t stream);
    void outer_overlapped(int nb);
    // `st` waits for the work on the second stream
    void join_side()
    {
        if (!side_pending) return;
        MJ_CHECK(hipStreamWaitEvent(st, ev_side, 0));
        side_pending = false;
    }
    // ... and forgets the sums it formed (the march, the ring or the time division changes)
    void drop_side()
    {
        join_side();
        h_block = 0;
    }
    void collect_side_timers(bool wait);
    void mac_autotune();
    void default_time_division();
    // arguments of a time-block MAC launch writing to `out`, first target step nb
    mj::BlockMacArg block_arg(double2 *out, int nb) const
    {
        mj::BlockMacArg a{};
        a.Khat = Khat;
        a.ring_base = ring;
        a.far = out;
        a.Hx = Hx;
        a.Hp = Hp;
        a.Ny = Ny;
        a.Nz = Nz;
        a.nk = ell;
        a.ring = ell;
        a.nb = nb;
        a.nrhs = nrhs;
        a.jmin = 1;
        return a;
    }
    mj::AdjArg adj_arg() const;
    void step(const StepIO &io);
    void follow(const StepIO &io, const double *w);
    void transform(int j, hipEvent_t *ev);
    const StepIO *cur = nullptr;          // the step whose solve runs
    const double *followed = nullptr;     // the solution that follow() last took for it
    int transformed = -1;                 // see step
    void flush_probes();
    void flush_after_failure()
    {
        try {
            flush_probes();
        } catch (...) {   // the step's own failure is the one to report
        }
        probe_steps = 0;
    }
    void check_growth() const;
    void run(int n_steps, double *Jout, double *Pout, int j_every = 1);
    void restart();
    void adjoint_gradient(int n_steps, int ckpt_every, double *phi, double *grad_dev, double *probe_hist);
    size_t state_bytes() const;
    void get_state(void *buf) const;
    void set_state(const void *buf, size_t bytes);
    void set_probes(int n_probes, const double *pos);
    void build_probes(int n_probes, const double *pos);
    void drop_probes();
    void offgrid_values(int n, const int *probe, const int *vox, const int *lag, double *out);
    void solve_z0();
    mj::CgArg cg_arg() const;
    bool run_cg(const mj::CgArg &a, int batch);
    void solve_cg();
    void learn();
    void cg_after_passes(int total, int batch);
    void replay();
    int group_size() const;
    void enqueue_passes(bool recorded, int g0, int g1, int T, int K);
    bool read_status(const double *w = nullptr);
    void solve_z0_chebyshev();
    void estimate_spectrum();
    // Passes with Chebyshev coefficients of their own; later ones take the last.  They approach their limit as
    // ((sqrt(kappa) - 1) / (sqrt(kappa) + 1))^2k, so up to a condition number kappa of 1e7 the last is the limit
    int ccoef_len() const { return std::min(cg_maxit, kChebCoefMax - 2) + 2; }
    size_t coef_count() const { return (size_t)nrhs * 2 * mj::kMaxCoef; }
    void clear_graphs()
    {
        for (auto &kv : pass_graphs) (void)hipGraphExecDestroy(kv.second);
        pass_graphs.clear();
    }
    void history_sum(const double *Jh, int depth, double *P);
};

void mj_solver::create(const mj_config &c)
{
    if (c.U < 1 || c.V < 1 || c.W < 1) throw ArgError("U, V, W must be >= 1");
    if (!(c.h > 0.0) || !std::isfinite(c.h)) throw ArgError("h must be positive and finite");
    if (!(c.c_dt > 0.0) || !std::isfinite(c.c_dt)) throw ArgError("c_dt must be positive and finite");
    if (!(c.hy >= 0.0) || !(c.hz >= 0.0) || !std::isfinite(c.hy) || !std::isfinite(c.hz))
        throw ArgError("hy, hz must be finite and >= 0 (0: equal to h)");
    {
        // c dt <= every edge keeps K_0 on the 27-point stencil the Z_0 solve is built for
        const double ey = c.hy > 0.0 ? c.hy : c.h, ez = c.hz > 0.0 ? c.hz : c.h;
        const double hmin = std::min(c.h, std::min(ey, ez)), hmax = std::max(c.h, std::max(ey, ez));
        if (!(c.c_dt <= hmin * (1.0 + 1e-12) && c.c_dt >= mj::kMinCdtOverH * hmax))
            throw ArgError("c_dt must lie in [0.3 max(h, hy, hz), min(h, hy, hz)]");
    }
    if (!c.eps_r) throw ArgError("eps_r is NULL");
    if (c.n_fir < 0 || (c.n_fir > 0 && !c.fir)) throw ArgError("bad FIR taps");
    if (c.n_fir > mj::kMaxLocal) throw ArgError("at most 64 FIR taps");
    if (c.n_rhs < 1 || c.n_rhs > 64) throw ArgError("n_rhs must be in [1, 64]");
    if (c.fft_pencils < 0) throw ArgError("fft_pencils must be >= 0 (0: autotune)");
    if ((c.alloc == nullptr) != (c.free_ == nullptr)) throw ArgError("alloc and free_ are given together or not at all");
    if (c.z0_solver < 0 || c.z0_solver > 2) throw ArgError("z0_solver must be 0 (by size), 1 (CG) or 2 (Chebyshev)");
    if (c.outer_overlap < 0 || c.outer_overlap > 2)
        throw ArgError("outer_overlap must be 0 (default), 1 (in line) or 2 (on a second stream)");
    use_graphs = c.z0_graphs != 0;
    da.fn_alloc = c.alloc;
    da.fn_free = c.free_;
    da.ctx = c.alloc_ctx;
    U = c.U;
    V = c.V;
    W = c.W;
    M = (long)U * V * W;
    h = c.h;
    hy = c.hy > 0.0 ? c.hy : c.h;
    hz = c.hz > 0.0 ? c.hz : c.h;
    c_dt = c.c_dt;
    nrhs = c.n_rhs;
    cg_rtol = c.cg_rtol > 0 ? c.cg_rtol : 1e-13;
    cg_maxit = c.cg_maxit > 0 ? c.cg_maxit : 200;
    nquad = c.quad_order > 0 ? c.quad_order : 0;
    st = (hipStream_t)c.stream;
    fir.assign(c.fir, c.fir + c.n_fir);
    for (double d : fir)
        if (!std::isfinite(d)) throw ArgError("FIR taps must be finite");
    std::vector<double> eps(c.eps_r, c.eps_r + M);
    eps_h = eps;
    for (double e : eps)
        if (!(e >= 1.0) || !std::isfinite(e)) throw ArgError("eps_r must be finite and >= 1");
    // eq:Ell
    double diag = std::sqrt((U * h) * (U * h) + (V * hy) * (V * hy) + (W * hz) * (W * hz));
    ell = (int)std::floor(diag / c_dt + 1e-12) + 2;
    // zero padding N >= 2U - 1 per axis (Appendix A)
    Nx = mj::fft_pick_size(2 * U - 1);
    Ny = mj::fft_pick_size(2 * V - 1);
    Nz = mj::fft_pick_size(2 * W - 1);
    Hx = Nx / 2 + 1;
    Hp = mj::spectrum_pitch(Hx);
    const bool tune_mac = c.time_block < 0;
    B = c.time_block > 0 ? c.time_block : 8;
    if (!(B == 1 || B == 4 || B == 32 || (B >= 8 && B <= 16 && B % 2 == 0)))
        throw ArgError("time_block must be -1 (timed), 0 (default), 1, 4, 8, 10, 12, 14, 16 or 32");
    B2 = c.outer_block > 1 ? c.outer_block : 0;
    if (c.time_block == 0 && c.outer_block == 0) default_time_division();
    if (B2 && !(B == 4 || B == 8) ) throw ArgError("outer_block needs time_block 4 or 8");
    if (B2 && !(B2 > B && B2 % B == 0 && B2 >= 8 && B2 <= 16 && B2 % 2 == 0))
        throw ArgError("outer_block must be a multiple of time_block in 8 .. 16 (even), or 0");
    // steps kept for the initial guess (7 or more) and the taps; the guess takes up to 9 of them
    nloc = std::max(7, (int)fir.size() - 1);
    rdepth = sdepth = nloc + 1;

    // The Z_0 solve.  By default the passes of an earlier step's CG are replayed (solve_z0); behind
    // them stands the Chebyshev iteration on small grids, whose launches decide (32^3: 4 us a pass
    // against 20 us per CG iteration of four launches), and CG's fewer iterations on large ones.
    z0_method = c.z0_solver == 1 ? 1 : c.z0_solver == 2 ? 0 : (M <= kChebMaxUnknowns ? 0 : 1);
    replays = c.z0_solver == 0;
    MJ_CHECK(hipGetDevice(&dev));
    if (use_graphs) MJ_CHECK(hipStreamCreateWithFlags(&cap_st, hipStreamNonBlocking));
    (void)scratch_ptr(dev);   // this device's staging array (mj_kernel_values_noalloc)
    chi = dalloc<double>(M, "chi");
    chih = dalloc<double>((size_t)(U + 2) * (V + 2) * (W + 2), "chi, haloed");
    schi = dalloc<double>(M, "sqrt chi");
    inv_eps = dalloc<double>(M, "1/eps");
    c0 = dalloc<double>(M, "c0");
    fir_d = dalloc<double>(std::max<size_t>(fir.size(), 1), "fir");
    if (!fir.empty()) MJ_CHECK(hipMemcpy(fir_d, fir.data(), fir.size() * 8, hipMemcpyHostToDevice));

    build_spectra();
    set_material(eps.data());

    // march state
    const long sp = spec_plane();
    ring = dalloc<double2>((size_t)ell * nrhs * 3 * sp, "spectral history ring");
    Shat = dalloc<double2>((size_t)nrhs * 3 * sp, "spectral sum");
    // a timed choice of the time division tries blocks of up to 16 steps at both levels
    const int fb_targets = tune_mac ? 16 : B, gb_targets = tune_mac ? 16 : B2;
    if (fb_targets > 1) farbuf = dalloc<double2>((size_t)fb_targets * nrhs * 3 * sp, "time-block partial sums");
    if (gb_targets) gbuf = dalloc<double2>((size_t)gb_targets * nrhs * 3 * sp, "outer-block partial sums");
    const bool want_overlap = c.outer_overlap == 2 || (c.outer_overlap == 0 && kOverlapDefault);
    if (gb_targets && want_overlap) {
        hbuf = dalloc<double2>((size_t)gb_targets * nrhs * 3 * sp, "next outer block's sums");
        MJ_CHECK(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
        MJ_CHECK(hipEventCreateWithFlags(&ev_main, hipEventDisableTiming));
        MJ_CHECK(hipEventCreateWithFlags(&ev_side, hipEventDisableTiming));
        for (auto &pr : side_t)
            for (hipEvent_t &e : pr) MJ_CHECK(hipEventCreate(&e));
    }
    S = dalloc<double>((size_t)nrhs * 3 * M, "convolution");
    Jr = dalloc<double>((size_t)rdepth * nrhs * 3 * M, "current history");
    y = dalloc<double>((size_t)nrhs * 3 * M, "cg y");
    p = dalloc<double>((size_t)nrhs * 3 * M, "cg p");
    q = dalloc<double>((size_t)nrhs * 3 * M, "cg q");
    const size_t Mp = (size_t)(U + 2) * (V + 2) * (W + 2);
    u = dalloc<double>((size_t)nrhs * 3 * Mp, "cg u");
    bh = dalloc<double>((size_t)nrhs * 3 * Mp, "solve rhs");
    // the one-voxel halo of these is never written and stays zero
    MJ_CHECK(hipMemset(u, 0, sizeof(double) * nrhs * 3 * Mp));
    MJ_CHECK(hipMemset(bh, 0, sizeof(double) * nrhs * 3 * Mp));
    for (double *&w : wbuf) {
        w = dalloc<double>((size_t)nrhs * 3 * Mp, "solve vector");
        MJ_CHECK(hipMemset(w, 0, sizeof(double) * nrhs * 3 * Mp));
    }
    coef = dalloc<double>(coef_count(), "recorded coefficients");
    rhist = dalloc<double>((size_t)nrhs * mj::kMaxCoef, "recorded residuals");
    ccoef = dalloc<double>(2 * (size_t)ccoef_len(), "Chebyshev coefficients");
    nblk = (int)((M + 255) / 256);
    part_cap = 3 * nblk;
    {
        const int G = group_size();
        for (int nr = 1; nr <= G; nr++) part_cap = std::max(part_cap, 2 * mj::z0_pass_blocks(U, V, W, nr));
    }
    parts = dalloc<double>((size_t)nrhs * part_cap, "solve partials");
    scal = dalloc<mj::CgScalars>(nrhs, "cg scalars");
    cgstat = dalloc<mj::CgStatus>(nrhs, "cg status");
    waves_d = dalloc<mj::WaveArg>(nrhs, "waves");
    {
        double rules[9 * 16] = {};
        for (int n = 1; n <= 8; n++) gl_half(n, rules + 16 * n, rules + 16 * n + 8);
        gl_d = dalloc<double>(9 * 16, "quadrature rules");
        MJ_CHECK(hipMemcpy(gl_d, rules, sizeof rules, hipMemcpyHostToDevice));
    }
    MJ_CHECK(hipEventCreateWithFlags(&ev_status, hipEventDisableTiming));
    MJ_CHECK(hipHostMalloc((void **)&cgstat_h, sizeof(mj::CgStatus) * nrhs, hipHostMallocDefault));
    mj::fft3d_init(fft, U, V, W, 3 * nrhs, Nx, Ny, Nz, da);
    bytes += sizeof(double2) * ((size_t)3 * nrhs * W * V * Hp + (size_t)3 * nrhs * W * Ny * Hp);
    if (c.fft_pencils > 0) mj::fft3d_set_pencils(fft, c.fft_pencils);
    else mj::fft3d_autotune(fft, st);
    if (tune_mac) mac_autotune();
    overlap = hbuf != nullptr && B2 > 0;
    if (z0_method == 0) estimate_spectrum();
    n = 0;
    MJ_CHECK(hipStreamSynchronize(st));
}

// chi, sqrt chi, 1/eps, c_0 = T(0)/eps + delta_0 and the Jacobi preconditioner
// diag(A) = c_0 - chi K_0^{bb}(0) of the symmetrised Z_0 (needs K_0 from build_spectra)
void mj_solver::set_material(const double *eps)
{
    for (long i = 0; i < M; i++)
        if (!(eps[i] >= 1.0) || !std::isfinite(eps[i])) throw ArgError("eps_r must be finite and >= 1");
    eps_h.assign(eps, eps + M);
    std::vector<double> chi_h(M), schi_h(M), ie_h(M), c0_h(M);
    const double d0 = fir.empty() ? 0.0 : fir[0];
    for (long i = 0; i < M; i++) {
        chi_h[i] = (eps[i] - 1.0) / eps[i];
        schi_h[i] = std::sqrt(chi_h[i]);
        ie_h[i] = 1.0 / eps[i];
        c0_h[i] = 0.5 * ie_h[i] + d0;   // T(0)/eps + delta_0
    }
    MJ_CHECK(hipMemcpy(chi, chi_h.data(), M * 8, hipMemcpyHostToDevice));
    MJ_CHECK(hipMemcpy(schi, schi_h.data(), M * 8, hipMemcpyHostToDevice));
    MJ_CHECK(hipMemcpy(inv_eps, ie_h.data(), M * 8, hipMemcpyHostToDevice));
    MJ_CHECK(hipMemcpy(c0, c0_h.data(), M * 8, hipMemcpyHostToDevice));
    std::vector<double> ch((size_t)(U + 2) * (V + 2) * (W + 2), 0.0);
    for (int z = 0; z < W; z++)
        for (int v = 0; v < V; v++)
            std::copy_n(&chi_h[((size_t)z * V + v) * U], U, &ch[((size_t)(z + 1) * (V + 2) + (v + 1)) * (U + 2) + 1]);
    MJ_CHECK(hipMemcpy(chih, ch.data(), ch.size() * 8, hipMemcpyHostToDevice));
}

void mj_solver::build_spectra()
{
    auto t0 = std::chrono::steady_clock::now();
    {
        // generator units: the x edge
        const double hv[3] = {1.0, hy / h, hz / h};
        mj::gen_moments(gen, U, V, W, c_dt / h, hv, nquad, da, st);
    }
    bytes += (size_t)M * gen.ms * mj::kMoments * sizeof(double);
    MJ_CHECK(hipStreamSynchronize(st));
    auto t1 = std::chrono::steady_clock::now();
    t_gen_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();

    // K_0 stencil (27 offsets, 6 components) for the Z_0 solve
    {
        std::vector<int> lag(27, 0), off(81);
        int o = 0;
        for (int dz = -1; dz <= 1; dz++)
            for (int dy = -1; dy <= 1; dy++)
                for (int dx = -1; dx <= 1; dx++, o++) {
                    off[3 * o] = (U > 1 || dx == 0) ? dx : 0;
                    off[3 * o + 1] = (V > 1 || dy == 0) ? dy : 0;
                    off[3 * o + 2] = (W > 1 || dz == 0) ? dz : 0;
                }
        mj::DevTemp tl(da, 27 * sizeof(int), "stencil request");
        mj::DevTemp to(da, 81 * sizeof(int), "stencil request");
        mj::DevTemp tv(da, 162 * sizeof(double), "stencil values");
        int *lag_d = tl.as<int>(), *off_d = to.as<int>();
        double *out_d = tv.as<double>();
        MJ_CHECK(hipMemcpy(lag_d, lag.data(), 27 * sizeof(int), hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(off_d, off.data(), 81 * sizeof(int), hipMemcpyHostToDevice));
        mj::gen_kernel_values(gen, 27, lag_d, off_d, out_d, st);
        MJ_CHECK(hipMemcpyAsync(K0_27, out_d, 162 * sizeof(double), hipMemcpyDeviceToHost, st));
        MJ_CHECK(hipStreamSynchronize(st));
        // offsets that fall outside a one-voxel-thick axis do not couple
        o = 0;
        for (int dz = -1; dz <= 1; dz++)
            for (int dy = -1; dy <= 1; dy++)
                for (int dx = -1; dx <= 1; dx++, o++)
                    if ((U == 1 && dx != 0) || (V == 1 && dy != 0) || (W == 1 && dz != 0))
                        for (int c = 0; c < 6; c++) K0_27[6 * o + c] = 0.0;
        k0_d = dalloc<double>(27 * 6, "K_0 stencil");
        MJ_CHECK(hipMemcpy(k0_d, K0_27, sizeof K0_27, hipMemcpyHostToDevice));
    }

    // spectra of lags 1..ell on the padded grid, octant only, with 1/(Nx Ny Nz) folded in
    const long ko = koct();
    Khat = dalloc<double>((size_t)ell * 6 * ko, "kernel spectra");
    mj::Fft3D kf{};
    double *grid = nullptr;
    double2 *X = nullptr;
    const size_t ng = (size_t)Nx * Ny * Nz;
    try {
        mj::fft3d_init(kf, Nx, Ny, Nz, 6, Nx, Ny, Nz, da);
        grid = (double *)da.get(6 * ng * sizeof(double), "kernel grid");
        X = (double2 *)da.get(6 * (size_t)Nz * Ny * Hp * sizeof(double2), "kernel spectrum");
        const double scale = 1.0 / ((double)Nx * Ny * Nz);
        for (int k = 1; k <= ell; k++) {
            mj::gen_kernel_grid(gen, k, Nx, Ny, Nz, grid, st);
            mj::fft3d_forward(kf, grid, X, 6, st);
            hipLaunchKernelGGL(k_extract_octant, dim3((unsigned)((ko + 255) / 256)), dim3(256), 0, st, X, Hx, Hp, Ny, Nz,
                               scale, Khat + (size_t)(k - 1) * 6 * ko);
            MJ_CHECK(hipGetLastError());
        }
        MJ_CHECK(hipStreamSynchronize(st));
    } catch (...) {
        mj::fft3d_free(kf);
        da.put(grid);
        da.put(X);
        throw;
    }
    mj::fft3d_free(kf);
    da.put(grid);
    da.put(X);
    auto t2 = std::chrono::steady_clock::now();
    t_spec_ms = std::chrono::duration<double, std::milli>(t2 - t1).count();
}

mj::CgArg mj_solver::cg_arg() const
{
    mj::CgArg a{};
    a.M = M;
    a.U = U;
    a.V = V;
    a.W = W;
    a.Mp = (long)(U + 2) * (V + 2) * (W + 2);
    a.nrhs = nrhs;
    a.nblk = nblk;
    a.tol2 = a.stop2 = cg_rtol * cg_rtol;
    a.schi = schi;
    a.d0 = fir.empty() ? 0.0 : fir[0];
    a.k0c = K0_27[13 * 6 + 0];
    a.k0 = k0_d;
    a.b = bh;
    a.w = wbuf[0];
    a.y = y;
    a.p = p;
    a.q = q;
    a.u = u;
    a.part = parts;
    a.scal = scal;
    a.stat = cgstat;
    return a;
}

// CG iterations from the vectors of `a` until every right-hand side has ended or cg_maxit; the first look at
// the status comes after `batch` of them (kernels after a solve's end return at once).  The solution is left
// in y.  Returns whether every right-hand side met the tolerance.
bool mj_solver::run_cg(const mj::CgArg &a, int batch)
{
    mj::launch_cg_init(a, st);   // also clears the status records
    int it = 0;
    batch = std::max(2, std::min(cg_maxit, batch));
    bool ended = false, done = false;
    while (it < cg_maxit && !ended) {
        const int upto = std::min(cg_maxit, it + batch);
        for (; it < upto; it++) {
            mj::launch_cg_a(a, it, st);
            mj::launch_cg_b(a, it, st);
        }
        done = read_status();
        ended = true;
        for (int i = 0; i < nrhs; i++) ended = ended && cgstat_h[i].ended;
        batch = 2;
    }
    // the last update of y (a no-op for the right-hand sides whose solve already ended)
    mj::launch_cg_end(a, it, st);
    w_end = nullptr;
    return done;
}

void mj_solver::solve_cg()
{
    run_cg(cg_arg(), cg_guess);
    int mx = 0;
    for (int i = 0; i < nrhs; i++) mx = std::max(mx, cgstat_h[i].iters);
    cg_guess = mx + 1;
}

// The status of every right-hand side; true if all met the tolerance.  w (or NULL): the solution if they
// did.  What follows the solve is then enqueued before the host waits for the status, so that the device
// works on while the host wakes up; if some right-hand side goes on, it is enqueued again with the final
// solution (follow writes only what it will write again).
bool mj_solver::read_status(const double *w)
{
    MJ_CHECK(hipMemcpyAsync(cgstat_h, cgstat, sizeof(mj::CgStatus) * nrhs, hipMemcpyDeviceToHost, st));
    MJ_CHECK(hipEventRecord(ev_status, st));
    followed = nullptr;
    if (w && cur) {
        follow(*cur, w);
        followed = w;
    }
    MJ_CHECK(hipEventSynchronize(ev_status));
    bool done = true;
    for (int i = 0; i < nrhs; i++) done = done && cgstat_h[i].done;
    return done;
}

// Right-hand sides per group of three-term passes.  A group's passes follow each other, so that what
// they stream (w_k, w_{k-1} and b) stays in the last-level cache; groups are as even as they go.
int mj_solver::group_size() const
{
    const size_t per_rhs = sizeof(double) * 9 * (size_t)(U + 2) * (V + 2) * (W + 2);
    const int most = (int)std::max<size_t>(1, std::min<size_t>((size_t)nrhs, kPassGroupBytes / per_rhs));
    const int groups = (nrhs + most - 1) / most;
    return (nrhs + groups - 1) / groups;
}

// Passes T .. T + K - 1 of the right-hand sides g0 .. g1 - 1, with the recorded coefficients or those of the
// Chebyshev iteration; the test of w_{T+K-1} follows the last.  The arguments depend only on these numbers, so
// a captured batch can be launched again.
void mj_solver::enqueue_passes(bool recorded, int g0, int g1, int T, int K)
{
    auto launch = [&](hipStream_t s_) {
        mj::PassArg a{};
        a.px = U + 2;
        a.py = V + 2;
        a.pz = W + 2;
        a.Mp = (long)a.px * a.py * a.pz;
        a.d0 = fir.empty() ? 0.0 : fir[0];
        a.k0c = K0_27[13 * 6 + 0];
        a.tol2 = cg_rtol * cg_rtol;
        a.chi = chih;
        a.b = bh;
        a.k0 = k0_d;
        a.coef = recorded ? coef : ccoef;
        a.coef_stride = recorded ? 2 * mj::kMaxCoef : 0;
        a.coef_len = recorded ? mj::kMaxCoef : ccoef_len();
        a.rhs0 = g0;
        a.nr = g1 - g0;
        a.part = parts;
        a.part_cap = part_cap;
        a.stat = cgstat;
        for (int k = T; k < T + K; k++) {
            a.k = recorded ? k : std::min(k, a.coef_len - 1);
            a.first = k == 0;
            a.want_norm = k == T + K - 1;
            a.w = wbuf[k & 1];
            a.v = wbuf[(k + 1) & 1];
            mj::launch_z0_pass(a, k, s_);
        }
    };
    if (!use_graphs) {
        launch(st);
        return;
    }
    const long key = ((long)g0 << 48) | ((long)recorded << 40) | ((long)T << 20) | K;
    auto it = pass_graphs.find(key);
    if (it == pass_graphs.end()) {
        hipGraph_t g = nullptr;
        hipGraphExec_t ex = nullptr;
        MJ_CHECK(hipStreamBeginCapture(cap_st, hipStreamCaptureModeRelaxed));
        try {
            launch(cap_st);
        } catch (...) {
            (void)hipStreamEndCapture(cap_st, &g);
            if (g) (void)hipGraphDestroy(g);
            throw;
        }
        MJ_CHECK(hipStreamEndCapture(cap_st, &g));
        const hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        MJ_CHECK(e);
        it = pass_graphs.emplace(key, ex).first;
    }
    MJ_CHECK(hipGraphLaunch(it->second, st));
}

// Z_0 J_n = b (eq:MOTInversion) from the extrapolated current in wbuf[0].
//
// By default most steps replay the iteration that CG took in an earlier step of the same march: its
// three-term coefficients, recorded per right-hand side on the device, applied by k_z0_pass without inner
// products (see there).  CG runs, and is recorded, at steps 1, 4, 16, 64, 128, 256, ... (the residuals change
// most as the wave enters, and one CG solve in 128 costs little), and after a replay that
// missed the tolerance; on small grids, where a CG solve costs six of the Chebyshev iteration (32^3: 0.8 ms
// against 0.13), that one takes the first 15 steps.  Every solve is tested on its own residual, so a record that
// no longer fits costs passes, never accuracy.  (The test is that of the last pass's input; its output, one update
// further, is the solution.  Over 540 solves, with a change of waves among them and eps up to 1e4, that one's
// residual was 0.29 to 0.55 of the tested one at the median, at most 0.95 of it after Chebyshev passes, and never
// above 6.6e-14 with the test at 1e-13.)  What decides which steps run CG, and how many passes a replay takes
// before its test, depends on the march alone and travels with its state.
void mj_solver::solve_z0()
{
    auto base = [&] {
        if (z0_method == 0 && lam_hi > 0.0) solve_z0_chebyshev();
        else solve_cg();
    };
    if (!replays) {
        base();
        return;
    }
    if (rp.hold > 0) {
        rp.hold--;
        base();
        return;
    }
    if (z0_method == 0 && lam_hi > 0.0 && n < 16) {
        base();
        return;
    }
    // (a resumed state's record may ask for more passes than this solver is allowed)
    if (rp.learn || rp.K > cg_maxit || n == 1 || n == 4 || n == 16 || n == 64 || n % 128 == 0) learn();
    else replay();
}

// A CG solve that records its coefficients.  It runs on to 1/100 of the tolerance, so that replays have
// a few passes to spare.
void mj_solver::learn()
{
    mj::CgArg a = cg_arg();
    a.stop2 = 1e-4 * a.tol2;
    a.coef = coef;
    a.rhist = rhist;
    const bool done = run_cg(a, cg_guess);
    std::vector<double> h((size_t)nrhs * mj::kMaxCoef);
    MJ_CHECK(hipMemcpyAsync(h.data(), rhist, sizeof(double) * h.size(), hipMemcpyDeviceToHost, st));
    MJ_CHECK(hipStreamSynchronize(st));
    int K = 0, L = 0;
    for (int i = 0; i < nrhs; i++) {
        const int its = std::min(cgstat_h[i].iters, mj::kMaxCoef - 1);
        int k = 0;
        while (k < its && !(h[(size_t)i * mj::kMaxCoef + k] <= a.tol2)) k++;
        K = std::max(K, k);
        L = std::max(L, cgstat_h[i].iters);
    }
    cg_guess = L + 1;
    rp.K = rp.K0 = K;
    rp.L = std::min(L, mj::kMaxCoef);
    rp.learn = !done || K < 1;   // nothing to replay: zero right-hand sides, or no convergence
    if (done && L > mj::kMaxCoef - 4) {   // too long to record
        rp.learn = 1;
        rp.hold = 64;
    }
}

// CG from where `total` passes ended, or from zero for a right-hand side that they left further off than that:
// CG tests the residual of its recurrence, which hides what cancels from the first one, about 1e-16 of it (and
// coefficients that do not fit a spectrum can take the iterate anywhere, also out of the finite range).
void mj_solver::cg_after_passes(int total, int batch)
{
    double *w = wbuf[(total + 1) & 1];
    const size_t v = (size_t)3 * (U + 2) * (V + 2) * (W + 2);
    for (int i = 0; i < nrhs; i++)
        if (!(cgstat_h[i].res <= 1.0)) MJ_CHECK(hipMemsetAsync(w + i * v, 0, sizeof(double) * v, st));
    mj::CgArg a = cg_arg();
    a.w = w;
    run_cg(a, batch);
    for (int i = 0; i < nrhs; i++) cgstat_h[i].iters += total;
}

void mj_solver::replay()
{
    const int G = group_size(), K = rp.K;
    for (int g0 = 0; g0 < nrhs; g0 += G) enqueue_passes(true, g0, std::min(nrhs, g0 + G), 0, K + 1);
    bool done = read_status(wbuf[(K + 1) & 1]);
    int total = K;
    // groups that missed go on, two passes at a time, so that the solution stays in the same wbuf
    for (int more = 0; !done && more < 2 && total + 2 < std::min(rp.L, cg_maxit); more++) {
        for (int g0 = 0; g0 < nrhs; g0 += G) {
            const int g1 = std::min(nrhs, g0 + G);
            bool ok = true;
            for (int i = g0; i < g1; i++) ok = ok && cgstat_h[i].done;
            if (!ok) enqueue_passes(true, g0, g1, total + 1, 2);
        }
        total += 2;
        done = read_status(wbuf[(total + 1) & 1]);
    }
    w_end = wbuf[(total + 1) & 1];
    if (done) {
        double res = 0.0;
        for (int i = 0; i < nrhs; i++) res = std::max(res, cgstat_h[i].res);
        rp.fails = 0;
        rp.K = total;
        if (res <= 0.1 * cg_rtol && K > 1) rp.K = total - 1;   // a pass gains a factor of 2 to 4
        if (rp.K > rp.K0 + 3) rp.learn = 1;
        return;
    }
    for (int i = 0; i < nrhs; i++)
        if (!std::isfinite(cgstat_h[i].bb) || cgstat_h[i].bb > 1e200) return;   // the march ends (check_growth)
    // the record does not fit any more: CG from where the passes ended, and a new record in the next step;
    // after several misses in a row, some steps without replays
    cg_after_passes(total, cg_guess);
    rp.learn = 1;
    rp.fails = std::min(rp.fails + 1, kMaxFails);
    if (rp.fails >= 2) rp.hold = 4 << rp.fails;
}

// Number of eigenvalues below x of the symmetric tridiagonal matrix (diagonal a, off-diagonal
// b, b[0] unused): the Sturm count of the LDL^T pivots.
static int sturm_count(const std::vector<double> &a, const std::vector<double> &b, double x)
{
    int cnt = 0;
    double q = 1.0;
    for (size_t j = 0; j < a.size(); j++) {
        const double off = j ? b[j] * b[j] / q : 0.0;
        q = a[j] - x - off;
        if (q == 0.0) q = -1e-300;
        if (q < 0.0) cnt++;
    }
    return cnt;
}

// Extreme eigenvalues of M^-1 A (M the Jacobi preconditioner) for the Chebyshev solve: a CG run
// on a pseudo-random right-hand side is a Lanczos process, whose tridiagonal matrix
// T (T_jj = 1/alpha_j + beta_{j-1}/alpha_{j-1}, T_{j,j+1} = sqrt(beta_j)/alpha_j) has extreme
// eigenvalues that approach those of M^-1 A from inside; bisection on its Sturm counts gives
// them.  The bounds used are widened by 10 % below and 5 % above.  A spectrum with nothing in
// it (no voxel with eps != 1) leaves the bounds at 0, which selects the CG solve.
void mj_solver::estimate_spectrum()
{
    lam_lo = lam_hi = 0.0;
    mj::CgArg a = cg_arg();
    a.nrhs = 1;
    a.tol2 = a.stop2 = 0.0;   // run every iteration
    a.coef = coef;
    const size_t Mp = (size_t)(U + 2) * (V + 2) * (W + 2);
    MJ_CHECK(hipMemsetAsync(wbuf[0], 0, sizeof(double) * Mp * 3, st));
    mj::launch_fill_trial(schi, U, V, W, bh, st);
    const int m = std::min(40, 3 * (int)std::min<long>(M, 1000));
    mj::launch_cg_init(a, st);
    for (int it = 0; it < m; it++) {
        mj::launch_cg_a(a, it, st);
        mj::launch_cg_b(a, it, st);
    }
    std::vector<double> ab(2 * (size_t)m);
    MJ_CHECK(hipMemcpyAsync(ab.data(), coef, sizeof(double) * ab.size(), hipMemcpyDeviceToHost, st));
    restart();
    // alpha_j = a_j and beta_j = b_{j+1} a_j / a_{j+1} of the recorded iterations, up to where the Krylov
    // space is exhausted (tiny grids: the residual has vanished)
    std::vector<double> alpha, beta;
    double rz = 1.0;
    for (int j = 0; j < m; j++) {
        if (!(ab[2 * j] > 0.0) || !std::isfinite(ab[2 * j])) break;
        if (j > 0) {
            const double bj = ab[2 * j + 1] * ab[2 * j - 2] / ab[2 * j];
            rz *= bj;
            if (!(rz > 1e-28)) break;
            beta.push_back(bj);
        }
        alpha.push_back(ab[2 * j]);
    }
    const size_t k = alpha.size();
    if (k == 0) return;
    std::vector<double> d(k), e(k, 0.0);
    for (size_t j = 0; j < k; j++) {
        d[j] = 1.0 / alpha[j] + (j ? beta[j - 1] / alpha[j - 1] : 0.0);
        if (j) e[j] = std::sqrt(beta[j - 1]) / alpha[j - 1];
    }
    double lo = 1e300, hi = -1e300;
    for (size_t j = 0; j < k; j++) {   // Gershgorin interval of T
        const double rad = (j ? std::fabs(e[j]) : 0.0) + (j + 1 < k ? std::fabs(e[j + 1]) : 0.0);
        lo = std::min(lo, d[j] - rad);
        hi = std::max(hi, d[j] + rad);
    }
    auto kth = [&](int idx) {   // eigenvalue number idx (0-based, ascending) by bisection
        double l = lo, h = hi;
        for (int b = 0; b < 200 && h - l > 1e-14 * std::max(1.0, std::fabs(h)); b++) {
            const double mid = 0.5 * (l + h);
            if (sturm_count(d, e, mid) > idx) h = mid;
            else l = mid;
        }
        return 0.5 * (l + h);
    };
    const double emin = kth(0), emax = kth((int)k - 1);
    if (!(emin > 0.0) || !(emax >= emin)) return;
    lam_lo = 0.9 * emin;
    lam_hi = 1.05 * emax;
    // the three-term coefficients of the Chebyshev iteration for these bounds
    const double theta = 0.5 * (lam_hi + lam_lo), rho = (lam_hi - lam_lo) / (lam_hi + lam_lo);
    std::vector<double> cc(2 * (size_t)ccoef_len());
    double om = 1.0;
    for (size_t j = 0; j < cc.size() / 2; j++) {
        om = j == 0 ? 1.0 : j == 1 ? 1.0 / (1.0 - 0.5 * rho * rho) : 1.0 / (1.0 - 0.25 * om * rho * rho);
        cc[2 * j] = om / theta;
        cc[2 * j + 1] = om - 1.0;
    }
    MJ_CHECK(hipMemcpy(ccoef, cc.data(), sizeof(double) * cc.size(), hipMemcpyHostToDevice));
}

// The Z_0 solve by Chebyshev iteration on the estimated spectrum: three-term passes with its
// coefficients, as many as the last solve needed before the first test, then as many more as the
// polynomials' convergence factor asks for.  An iteration gains the factor rho, so the next solve takes
// fewer passes by what this one's residual fell short of the tolerance.
// A tolerance below the residual's rounding (1e-16 of b on small grids with eps up to 20; more with the condition
// of Z_0) is left to CG.
void mj_solver::solve_z0_chebyshev()
{
    const double kappa = lam_hi / lam_lo;
    const double lrho = std::log((std::sqrt(kappa) - 1.0) / (std::sqrt(kappa) + 1.0));
    const int G = group_size();
    auto passes = [&](int T, int K) {
        for (int g0 = 0; g0 < nrhs; g0 += G) enqueue_passes(false, g0, std::min(nrhs, g0 + G), T, K);
        return read_status(wbuf[(T + K) & 1]);
    };
    auto worst = [&] {
        double res = 0.0;
        for (int i = 0; i < nrhs; i++) res = std::max(res, std::isfinite(cgstat_h[i].res) ? cgstat_h[i].res : 0.0);
        return res;
    };
    auto steps = [&](double ratio) { return lrho < 0.0 ? std::log(ratio) / lrho : 1.0; };
    int total = std::max(1, std::min(cg_maxit, cheb_pred > 0 ? cheb_pred : (int)std::ceil(steps(cg_rtol)) + 1));
    bool done = passes(0, total + 1), stalled = false;
    while (!done && !stalled && total < cg_maxit) {
        const double res = worst();
        if (!(res > cg_rtol)) break;   // not finite
        const int K = std::max(1, std::min(cg_maxit - total, (int)std::ceil(steps(cg_rtol / res)) + 1));
        done = passes(total + 1, K);
        // less than half of what the polynomials promise (on a logarithmic scale): the residual, formed anew in
        // every pass, has come down to its own rounding, and no pass will lower it
        stalled = !done && worst() > res * std::exp(0.5 * lrho * K);
        cheb_pred = total;   // of a solve that stalls: what it took to get there
        total += K;
    }
    w_end = wbuf[(total + 1) & 1];
    if (stalled) {   // CG keeps its residual by recurrence, so any tolerance ends it
        cg_after_passes(total, 2);
        return;
    }
    const double res = worst();
    cheb_pred = total;
    if (done && res > 0.0 && res < 0.5 * cg_rtol)
        cheb_pred = std::max(1, total - (int)std::min(1000.0, std::floor(steps(2.0 * res / cg_rtol))));
    else if (res == 0.0) cheb_pred = 0;
}

mj::EpiArg mj_solver::epi_arg() const
{
    mj::EpiArg e{};
    e.k0 = k0_d;
    e.series = 1;
    for (const mj::WaveArg &w : waves)
        if (w.form != 3) e.series = 0;
    e.M = M;
    e.U = U;
    e.V = V;
    e.W = W;
    e.nrhs = nrhs;
    e.n = n;
    e.h = h;
    e.hy = hy;
    e.hz = hz;
    e.c_dt = c_dt;
    e.chi = chi;
    e.schi = schi;
    e.inv_eps = inv_eps;
    e.fir = fir_d;
    e.nfir = (int)fir.size();
    e.nloc = nloc;
    for (int k = 1; k <= nloc; k++) e.slot_of[k] = n - k >= 1 ? slotR(n - k) : 0;
    // extrapolation through m = nguess equally spaced past steps to the next one:
    // weight of J_{n-k} is (-1)^(k+1) binomial(m, k)
    e.nguess = std::min(guess_deg + 1, nloc);
    for (int k = 1; k <= e.nguess; k++) {
        double bin = 1.0;
        for (int q = 1; q <= k; q++) bin = bin * (e.nguess - q + 1) / q;
        e.gx[k - 1] = (k & 1) ? bin : -bin;
    }
    e.Jring = Jr;
    e.waves = waves_d;
    gl_half(8, e.glx8, e.glw8);
    e.gl = gl_d;
    e.b = bh;
    e.w0 = wbuf[0];
    return e;
}

// The spectral history sum of step n >= 2 (sources J_1 .. J_{n-1} in the ring), launched as the
// configured time division requires; returns where the step's sum is left.  *kind: 1 far (outer)
// launch, 2 near, 3 middle, 0 none of these (no time blocking).
const double2 *mj_solver::mac(int n, int *kind)
{
    const long sp = spec_plane();
    const double2 *spec = Shat;
    int far_kind = 0;
    if (B == 1) {
        mj::MacArg a{};
        a.Khat = Khat;
        a.ring_base = ring;
        a.Shat = Shat;
        a.Hx = Hx;
        a.Hp = Hp;
        a.Ny = Ny;
        a.Nz = Nz;
        a.nk = std::min(ell, n - 1);
        a.ring = ell;
        a.slot_nm1 = slotS(n - 1);
        a.nrhs = nrhs;
        mj::launch_mac(a, st);
    } else if (B2 == 0) {
        // blocks of B steps starting at n_b = 2, 2 + B, ...: the far part of every step of the
        // block is formed at n_b, when all of its sources are in the ring
        const int t = (n - 2) % B;
        mj::BlockMacArg a = block_arg(farbuf, n - t);
        a.ntarget = B;
        a.t = t;
        if (t == 0) mj::launch_mac_far(a, B, st);
        else mj::launch_mac_near(a, st);
        far_kind = t == 0 ? 1 : 2;
        spec = farbuf + (size_t)t * nrhs * 3 * sp;
    } else {
        // three levels (the Toeplitz division of Sec. 4.1 applied twice): outer blocks of B2
        // steps start at N_b = 2, 2 + B2, ...; each splits into inner blocks of B steps.
        //   outer, at N_b:  G[tau] = sum_{k > tau} Khat_k Jhat_{N_b + tau - k} over sources before N_b
        //   middle, at each inner start n_b > N_b:  F[t] = G[n_b - N_b + t] + the terms of the
        //                   sources N_b .. n_b - 1 (inside the outer block, before the inner one)
        //   near, every step:  + the terms of the sources n_b .. n - 1
        // The first inner block needs no middle part: its sums stay in G.
        const int tau = (n - 2) % B2, t = tau % B, q = tau / B;
        double2 *fb = q == 0 ? gbuf : farbuf;
        if (tau == 0) {
            if (overlap) {
                outer_overlapped(n);
            } else {
                mj::BlockMacArg a = block_arg(gbuf, n);
                a.ntarget = B2;
                mj::launch_mac_win(a, B2, st);
            }
            far_kind = 1;
        } else if (t == 0) {
            mj::BlockMacArg a = block_arg(farbuf, n);
            a.ntarget = B;
            a.jmin = n - tau;
            a.init = gbuf + (size_t)tau * nrhs * 3 * sp;
            mj::launch_mac_win(a, B, st);
            far_kind = 3;
        } else {
            mj::BlockMacArg a = block_arg(fb, n - t);
            a.t = t;
            mj::launch_mac_near(a, st);
            far_kind = 2;
        }
        spec = fb + (size_t)t * nrhs * 3 * sp;
    }
    *kind = far_kind;
    return spec;
}

// The outer sums of the block starting at nb over the sources before nb - B2 (lags above B2),
// into hbuf on `stream`: the work that can run while the block before nb marches.
void mj_solver::outer_sums(int nb, hipStream_t stream)
{
    if (nb - B2 - 1 < 1) throw std::logic_error("outer sums without sources");
    mj::BlockMacArg a = block_arg(hbuf, nb);
    a.ntarget = B2;
    a.jmax = nb - B2 - 1;
    mj::launch_mac_win(a, B2, stream, stream == side ? kSideLdsReserve : 0);
}

// The outer level at the start nb of an outer block, overlapped (Sec. 4.1's division with the
// outer sums split at nb - B2):
//   G[tau] = H[tau] + sum over the sources nb - B2 .. nb - 1 of Khat_k Jhat_{nb + tau - k},
// H being the sums over the sources before nb - B2, formed on the second stream while the block
// before marched (or here, in line, after a restart).  Then the second stream starts on the
// next block's H, over the sources before nb.  It reads ring slots of sources nb + B2 - ell ..
// nb - 1 while this block's steps write the slots of sources nb - ell .. nb + B2 - 1 - ell, and
// writes hbuf, which only the next block start reads, after waiting for it.
void mj_solver::outer_overlapped(int nb)
{
    join_side();
    const bool have_h = nb - B2 - 1 >= 1;
    if (have_h && h_block != nb) outer_sums(nb, st);
    mj::BlockMacArg a = block_arg(gbuf, nb);
    a.ntarget = B2;
    a.jmin = nb - B2;
    a.init = have_h ? hbuf : nullptr;
    mj::launch_mac_win(a, B2, st);
    MJ_CHECK(hipEventRecord(ev_main, st));
    MJ_CHECK(hipStreamWaitEvent(side, ev_main, 0));
    const int slot = side_count % kSideTimers;
    if (side_busy[slot]) {
        MJ_CHECK(hipEventSynchronize(side_t[slot][1]));
        collect_side_timers(false);
    }
    MJ_CHECK(hipEventRecord(side_t[slot][0], side));
    outer_sums(nb + B2, side);
    MJ_CHECK(hipEventRecord(side_t[slot][1], side));
    side_busy[slot] = true;
    side_count++;
    MJ_CHECK(hipEventRecord(ev_side, side));
    side_pending = true;
    h_block = nb + B2;
}

// Adds the durations of the finished launches on the second stream to side_ms (waiting for
// all of them with wait).
void mj_solver::collect_side_timers(bool wait)
{
    for (int i = 0; i < kSideTimers; i++) {
        if (!side_busy[i]) continue;
        if (wait) MJ_CHECK(hipEventSynchronize(side_t[i][1]));
        const hipError_t q = hipEventQuery(side_t[i][1]);
        if (q == hipErrorNotReady) {
            (void)hipGetLastError();   // not an error: keep it from the next launch check
            continue;
        }
        MJ_CHECK(q);
        float ms = 0.0f;
        MJ_CHECK(hipEventElapsedTime(&ms, side_t[i][0], side_t[i][1]));
        side_ms += ms;
        side_done++;
        side_busy[i] = false;
    }
}

// Default time division when the caller sets neither block: three levels, blocks of 4 in
// outer blocks of 16, once the kernel reaches far enough back in time (ell >= 64) for the
// outer level to pay; else two levels with blocks of 8.  The history sum per step, blocks of 8 against
// 4 in 16: 16^3 (ell 29) 7.9 and 8.7 us, 24^3 (43) 10.6 and 10.5, 32^3 (57) 24.8 and 20.8, 36^3 (64) 37.1 and
// 28.4, 48^3 (85) 96 and 70, 64^3 (112) 279 and 188, 104^3 (182) 1740 and 1119.  (They meet at ell = 43: the line
// was drawn with an outer kernel that took longer.)
void mj_solver::default_time_division()
{
    if (ell >= 64) {
        B = 4;
        B2 = 16;
    } else {
        B = 8;
        B2 = 0;
    }
}

// Picks the time division (time block B, outer block B2) by timing the history sum of one
// period of steps at steady state for each candidate: every lag live (the steps timed lie
// beyond ell), on a cleared ring (the values do not change the time).  The candidates only
// group the terms of eq:PnMOT differently, so results depend on the choice at rounding level.
void mj_solver::mac_autotune()
{
    static const int cand[][2] = {{8, 0}, {12, 0}, {16, 0}, {4, 8}, {4, 12}, {4, 16}, {8, 16}};
    MJ_CHECK(hipMemsetAsync(ring, 0, sizeof(double2) * (size_t)ell * nrhs * 3 * spec_plane(), st));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    MJ_CHECK(hipEventCreate(&e0));
    MJ_CHECK(hipEventCreate(&e1));
    double best = -1.0;
    int bestB = 8, bestB2 = 0;
    try {
        for (const auto &cd : cand) {
            B = cd[0];
            B2 = cd[1];
            const int period = B2 ? B2 : B;
            const int n0 = 2 + period * ((ell + period - 1) / period);
            double tmin = -1.0;
            for (int rep = 0; rep < 3; rep++) {
                MJ_CHECK(hipEventRecord(e0, st));
                for (int i = 0; i < period; i++) {
                    int kind = 0;
                    (void)mac(n0 + i, &kind);
                }
                MJ_CHECK(hipEventRecord(e1, st));
                MJ_CHECK(hipEventSynchronize(e1));
                float ms = 0.0f;
                MJ_CHECK(hipEventElapsedTime(&ms, e0, e1));
                if (rep > 0 && (tmin < 0.0 || ms < tmin)) tmin = ms;
            }
            const double per_step = tmin / period;
            if (best < 0.0 || per_step < best) {
                best = per_step;
                bestB = cd[0];
                bestB2 = cd[1];
            }
        }
    } catch (...) {
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        throw;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    B = bestB;
    B2 = bestB2;
    t_mac_tune_ms = best;
}

// What follows the solve of step n whatever comes next: J_n = w (haloed; NULL: s y) into the real ring, and
// the forward transform that the next step starts with.
void mj_solver::follow(const StepIO &io, const double *w)
{
    double *Jn = Jr + (size_t)slotR(n) * nrhs * 3 * M;
    mj::launch_cg_finish(y, schi, w, U, V, W, nrhs, Jn, io.Jout, st);
    if (io.ev) MJ_CHECK(hipEventRecord(io.ev[5], st));
    if (io.more) transform(n, io.ev ? io.ev + kStepEvents : nullptr);
}

// Jhat_j of a past current, into the spectral ring.
void mj_solver::transform(int j, hipEvent_t *ev)
{
    if (ev) MJ_CHECK(hipEventRecord(ev[0], st));
    mj::fft3d_forward(fft, Jr + (size_t)slotR(j) * nrhs * 3 * M, ring + (size_t)slotS(j) * nrhs * 3 * spec_plane(),
                      3 * nrhs, st);
    if (ev) MJ_CHECK(hipEventRecord(ev[1], st));
    transformed = j;
}

// One step n -> n + 1 of the march on the current track: FFT of the newest source, spectral
// history sum (plain or time-blocked), inverse FFT, right-hand side, Z_0 solve, and the
// outputs asked for.  io.adjoint runs the transposed march instead (sources nu, local
// history lambda in Lr, right-hand side from io.G).
// `transformed` holds the last step whose transform was enqueued by the step itself; a call that starts
// or moves the march forgets it, so it never outlives the rings' contents.
void mj_solver::step(const StepIO &io)
{
    const long sp = spec_plane();
    hipEvent_t *ev = io.ev;
    n += 1;
    const bool hist = n >= 2;
    if (hist && transformed != n - 1) transform(n - 1, ev);
    transformed = -1;
    if (ev && !hist) {
        MJ_CHECK(hipEventRecord(ev[0], st));
        MJ_CHECK(hipEventRecord(ev[1], st));
    }
    if (ev) MJ_CHECK(hipEventRecord(ev[7], st));
    int far_kind = 0;
    const double2 *spec = hist ? mac(n, &far_kind) : Shat;
    if (io.far_kind) *io.far_kind = (char)far_kind;
    if (ev) MJ_CHECK(hipEventRecord(ev[2], st));
    if (hist) mj::fft3d_inverse(fft, spec, S, 3 * nrhs, st);
    if (ev) MJ_CHECK(hipEventRecord(ev[3], st));
    mj::EpiArg e = epi_arg();
    e.S = hist ? S : nullptr;
    if (io.adjoint) {
        e.Lring = Lr;
        e.G = io.G;
        e.bq = bq;
        mj::launch_adj_epilogue(e, st);
    } else {
        mj::launch_epilogue(e, st);
    }
    if (ev) MJ_CHECK(hipEventRecord(ev[4], st));
    cur = &io;
    followed = nullptr;
    try {
        solve_z0();
    } catch (...) {
        cur = nullptr;
        transformed = -1;
        throw;
    }
    cur = nullptr;
    if (!followed || followed != w_end) follow(io, w_end);
    double *Jn = Jr + (size_t)slotR(n) * nrhs * 3 * M;
    if (io.adjoint) {
        mj::AdjArg a = adj_arg();
        a.nu = Jn;
        a.bq = bq;
        a.lam = Lr + (size_t)slotR(n) * nrhs * 3 * M;
        mj::launch_adj_lambda(a, st);
        if (io.Bj) {
            a.Bj = io.Bj;
            a.grad = io.grad;
            mj::launch_grad_accum(a, st);
        }
    } else {
        if (np > 0 && io.Pout) {
            if (probe_steps == 0) {
                probe_out = io.Pout;
                probe_n0 = n;
            }
            if (++probe_steps == mj::kProbeSteps) {
                if (ev) MJ_CHECK(hipEventRecord(ev[8], st));
                flush_probes();
                if (ev) MJ_CHECK(hipEventRecord(ev[6], st));
                if (io.probes_ran) *io.probes_ran = 1;
            }
        }
        if (io.Bout)
            mj::launch_grad_term(e, Jn, n >= 2 ? Jr + (size_t)slotR(n - 1) * nrhs * 3 * M : nullptr, io.Bout, st);
    }
}

// Forms the probe field of the steps that wait for it.
void mj_solver::flush_probes()
{
    if (probe_steps == 0) return;
    mj::ProbeStepArg pa{};
    pa.table = ptable;
    pa.pair_vox = pair_vox;
    pa.pair_kmin = pair_kmin;
    pa.np = np;
    pa.nw = nw;
    pa.nrhs = nrhs;
    pa.n0 = probe_n0;
    pa.ntarget = probe_steps;
    pa.ell = ell;
    pa.M = M;
    pa.npairs = npairs;
    pa.Jring = Jr;
    pa.rdepth = rdepth;
    pa.part = ppart;
    pa.ck_lo = ck_lo;
    pa.ck_hi = ck_hi;
    pa.ck_start = ck_start;
    pa.nck = pnck;
    pa.out = probe_out;
    probe_steps = 0;
    mj::launch_probes(pa, st);
}

// The march grows without bound (Sec. 5.2 and 6: the alternating mode at f = 1/(2 dt)): stop once the
// right-hand side of a Z_0 solve leaves the finite range or passes 1e100 in norm.
void mj_solver::check_growth() const
{
    for (int i = 0; i < nrhs; i++) {
        const double bb = cgstat_h[i].bb;
        if (!std::isfinite(bb) || bb > 1e200 || !std::isfinite(cgstat_h[i].res))
            throw UnstableError("the march is unstable: the Z_0 right-hand side of step " + std::to_string(n) +
                                " exceeds 1e100 in norm or is not finite");
    }
}

mj::AdjArg mj_solver::adj_arg() const
{
    mj::AdjArg a{};
    a.k0 = k0_d;
    a.M = M;
    a.U = U;
    a.V = V;
    a.W = W;
    a.nrhs = nrhs;
    a.table_v = ptable_v;
    a.kmin_v = pkmin_v;
    a.np = np;
    a.nw = nw;
    a.schi = schi;
    a.c0 = c0;
    a.inv_eps = inv_eps;
    return a;
}

// J_n goes to Jout for every j_every-th step of the call (steps s = j_every - 1, 2 j_every - 1, ...
// counted from 0), entry (s + 1) / j_every - 1; the probe field of every step goes to Pout.
void mj_solver::run(int n_steps, double *Jout, double *Pout, int j_every)
{
    if (!waves_set) throw std::logic_error("plane waves not set (mj_set_plane_waves)");
    events.ensure((size_t)kStepEvents * std::max(n_steps, 1));
    transformed = -1;
    double cg_iter_sum = 0, cg_res_max = 0, cg_iter_max = 0;
    bool noconv = false;
    std::vector<char> step_far(n_steps, 0), step_probes(n_steps, 0);
    side_ms = 0.0;
    side_done = 0;
    for (int s = 0; s < n_steps; s++) {
        StepIO io;
        io.ev = &events.ev[(size_t)kStepEvents * s];
        io.more = s + 1 < n_steps;
        io.Jout = (Jout && (s + 1) % j_every == 0) ? Jout + (size_t)((s + 1) / j_every - 1) * nrhs * 3 * M : nullptr;
        io.Pout = Pout ? Pout + (size_t)s * nrhs * np * 3 : nullptr;
        io.far_kind = &step_far[s];
        io.probes_ran = &step_probes[s];
        try {
            step(io);
            check_growth();
        } catch (...) {
            flush_after_failure();
            throw;
        }
        for (int i = 0; i < nrhs; i++) {
            cg_iter_sum += cgstat_h[i].iters;
            cg_iter_max = std::max(cg_iter_max, (double)cgstat_h[i].iters);
            cg_res_max = std::max(cg_res_max, cgstat_h[i].res);
            if (!cgstat_h[i].done) noconv = true;
        }
    }
    hipEvent_t *const ev_last = n_steps > 0 ? &events.ev[(size_t)kStepEvents * (n_steps - 1)] : nullptr;
    if (ev_last && !step_probes[n_steps - 1]) MJ_CHECK(hipEventRecord(ev_last[8], st));
    flush_probes();
    if (ev_last) {
        MJ_CHECK(hipEventRecord(ev_last[6], st));   // with the last probes
        step_probes[n_steps - 1] = 1;
    }
    MJ_CHECK(hipStreamSynchronize(st));
    double ph[6] = {0, 0, 0, 0, 0, 0}, probe_ms = 0;
    double far_ms = 0, near_ms = 0, mid_ms = 0;
    int nfar = 0, nnear = 0, nmid = 0;
    for (int s = 0; s < n_steps; s++) {
        hipEvent_t *ev = &events.ev[(size_t)kStepEvents * s];
        for (int k = 0; k < 5; k++) {
            float ms = 0;
            MJ_CHECK(hipEventElapsedTime(&ms, ev[k == 1 ? 7 : k], ev[k + 1]));
            ph[k] += ms;
            if (k == 1 && step_far[s] == 1) { far_ms += ms; nfar++; }
            if (k == 1 && step_far[s] == 2) { near_ms += ms; nnear++; }
            if (k == 1 && step_far[s] == 3) { mid_ms += ms; nmid++; }
        }
        float pms = 0;
        if (step_probes[s]) MJ_CHECK(hipEventElapsedTime(&pms, ev[8], ev[6]));
        probe_ms += pms;
    }
    if (ev_last) {
        float tot = 0;
        MJ_CHECK(hipEventElapsedTime(&tot, events.ev[0], ev_last[6]));
        ph[5] = tot;
    }
    const double ns = std::max(n_steps, 1);
    for (int k = 0; k < 6; k++) stat[k] = ph[k] / ns;
    stat[6] = cg_iter_sum / (ns * nrhs);
    stat[7] = cg_res_max;
    stat[8] = n_steps;
    stat[9] = cg_iter_max;
    stat[10] = nfar ? far_ms / nfar : 0.0;
    stat[11] = nfar;
    stat[12] = nnear ? near_ms / nnear : 0.0;
    stat[13] = probe_ms / ns;
    stat[18] = nmid ? mid_ms / nmid : 0.0;
    if (side) collect_side_timers(false);
    stat[19] = side_done ? side_ms / side_done : 0.0;
    stat[20] = side_done;
    if (noconv) throw std::range_error("Z_0 solve did not converge");
}

// Back to n = 0 with every past current zero.  (CG's p and q need no clearing: a solve's first iteration takes
// neither, see k_cg_a.)
void mj_solver::restart()
{
    drop_side();
    const size_t v = sizeof(double) * (size_t)nrhs * 3 * M;
    MJ_CHECK(hipMemsetAsync(y, 0, v, st));
    // voxels whose eps changed to 1 must read as zero in the stencil
    const size_t vp = sizeof(double) * (size_t)nrhs * 3 * (U + 2) * (V + 2) * (W + 2);
    MJ_CHECK(hipMemsetAsync(u, 0, vp, st));
    for (double *w : wbuf) MJ_CHECK(hipMemsetAsync(w, 0, vp, st));
    MJ_CHECK(hipStreamSynchronize(st));
    cg_guess = 8;
    cheb_pred = 0;
    rp = Replay();
    probe_steps = 0;
    n = 0;
}

void mj_solver::history_sum(const double *Jh, int depth, double *P)
{
    drop_side();
    const long sp = spec_plane();
    const int nfake = ell + 1;
    for (int k = 1; k <= ell; k++) {
        double2 *slot = ring + (size_t)slotS(nfake - k) * nrhs * 3 * sp;
        if (k <= depth) mj::fft3d_forward(fft, Jh + (size_t)(k - 1) * 3 * M, slot, 3, st);
        else MJ_CHECK(hipMemsetAsync(slot, 0, sizeof(double2) * 3 * sp, st));
    }
    const double2 *spec = Shat;
    if (B == 1) {
        mj::MacArg a{};
        a.Khat = Khat;
        a.ring_base = ring;
        a.Shat = Shat;
        a.Hx = Hx;
        a.Hp = Hp;
        a.Ny = Ny;
        a.Nz = Nz;
        a.nk = ell;
        a.ring = ell;
        a.slot_nm1 = slotS(nfake - 1);
        a.nrhs = nrhs;   // ring stride; only right-hand side 0 is meaningful here
        mj::launch_mac(a, st);
    } else {
        // the far part of the first step of a block starting at n = ell + 1 is the whole sum
        mj::BlockMacArg a{};
        a.Khat = Khat;
        a.ring_base = ring;
        a.far = farbuf;
        a.Hx = Hx;
        a.Hp = Hp;
        a.Ny = Ny;
        a.Nz = Nz;
        a.nk = ell;
        a.ring = ell;
        a.nb = nfake;
        a.ntarget = 1;
        a.t = 0;
        a.nrhs = nrhs;
        mj::launch_mac_far(a, B, st);
        spec = farbuf;
    }
    mj::fft3d_inverse(fft, spec, S, 3, st);
    mj::launch_history_local(Jh, depth, S, chi, inv_eps, fir_d, (int)fir.size(), M, P, st);
    MJ_CHECK(hipStreamSynchronize(st));
    n = 0;
}

// Probes: test voxels of side h centred at arbitrary points.  Pairs (probe, scatterer voxel)
// whose lag window [kmin, kmin + nw) meets 0..ell are kept, per probe sorted by kmin, with the
// kernel values of their window generated on the device once.
void mj_solver::set_probes(int n_probes, const double *pos)
{
    if (n != 0) throw std::logic_error("probes are set before the first step (or after mj_reset)");
    if (n_probes < 0 || n_probes > 65536) throw ArgError("n_probes must be in [0, 65536]");
    if (n_probes > 0 && !pos) throw ArgError("probe positions are NULL");
    for (int i = 0; i < 3 * n_probes; i++)
        if (!std::isfinite(pos[i])) throw ArgError("probe positions must be finite");
    drop_probes();
    if (n_probes == 0) return;
    try {
        build_probes(n_probes, pos);
    } catch (...) {   // out of memory: no probes rather than some of their tables
        (void)hipStreamSynchronize(st);
        drop_probes();
        throw;
    }
}

void mj_solver::drop_probes()
{
    dfree((void *&)probe_pos);
    dfree((void *&)ptable);
    dfree((void *&)ppart);
    dfree((void *&)pair_vox);
    dfree((void *&)pair_kmin);
    dfree((void *&)pinv);
    dfree((void *&)ck_lo);
    dfree((void *&)ck_hi);
    dfree((void *&)ck_start);
    dfree((void *&)ptable_v);
    dfree((void *&)pkmin_v);
    pnck = 0;
    np = 0;
    nw = 0;
    npairs = 0;
}

void mj_solver::build_probes(int n_probes, const double *pos)
{
    // probe points in voxel steps per axis; distances in units of the x edge
    const double r = c_dt / h;
    const double edge[3] = {h, hy, hz}, hv[3] = {1.0, hy / h, hz / h};
    std::vector<double> P(3 * (size_t)n_probes);
    for (size_t i = 0; i < P.size(); i++) P[i] = pos[i] / edge[i % 3];
    // every voxel is a source: voxels with eps_r = 1 carry no current in the march, but the
    // transposed march needs the probe kernels there (their lambda enters the eps-gradient)
    std::vector<int> src((size_t)M);
    for (long m = 0; m < M; m++) src[(size_t)m] = (int)m;
    struct Pair {
        int kmin, vox;
    };
    std::vector<int> pp, pv, pk, clo, chi_, cst;
    int nwin = 1;
    for (int p = 0; p < n_probes; p++) {
        std::vector<Pair> list;
        for (int m : src) {
            const int u = m % U, v = (m / U) % V, w = m / (U * V);
            const double d[3] = {P[3 * p] - (u + 0.5), P[3 * p + 1] - (v + 0.5), P[3 * p + 2] - (w + 0.5)};
            double a2 = 0, b2 = 0;
            for (int i = 0; i < 3; i++) {
                const double ad = std::fabs(d[i]);
                const double e = ad > 1.0 ? (ad - 1.0) * hv[i] : 0.0;
                a2 += e * e;
                b2 += ((ad + 1.0) * hv[i]) * ((ad + 1.0) * hv[i]);
            }
            // lags with r(k + 1) > R_min and r(k - 2) < R_max
            const int kmin = std::max(0, (int)std::floor(std::sqrt(a2) / r));
            const int kmax = std::min(ell, (int)std::ceil(std::sqrt(b2) / r + 2.0) - 1);
            if (kmin > kmax) continue;
            nwin = std::max(nwin, kmax - kmin + 1);
            list.push_back({kmin, m});
        }
        std::stable_sort(list.begin(), list.end(), [](const Pair &a, const Pair &b) { return a.kmin < b.kmin; });
        // chunks of at most kProbeChunk pairs, probe by probe
        const int base = (int)pp.size(), end = base + (int)list.size();
        cst.push_back((int)clo.size());
        for (int q = base; q < end; q += mj::kProbeChunk) {
            clo.push_back(q);
            chi_.push_back(std::min(end, q + mj::kProbeChunk));
        }
        for (const Pair &x : list) {
            pp.push_back(p);
            pv.push_back(x.vox);
            pk.push_back(x.kmin);
        }
    }
    np = n_probes;
    nw = nwin;
    npairs = (long)pp.size();
    probe_pos = dalloc<double>(P.size(), "probe positions");
    pair_vox = dalloc<int>(std::max<size_t>(pv.size(), 1), "probe pairs");
    pair_kmin = dalloc<int>(std::max<size_t>(pk.size(), 1), "probe windows");
    {
        std::vector<int> inv((size_t)n_probes * M, -1);
        for (size_t q = 0; q < pp.size(); q++) inv[(size_t)pp[q] * M + pv[q]] = (int)q;
        pinv = dalloc<int>(inv.size(), "probe pair index");
        MJ_CHECK(hipMemcpy(pinv, inv.data(), sizeof(int) * inv.size(), hipMemcpyHostToDevice));
    }
    int *pair_probe = dalloc<int>(std::max<size_t>(pp.size(), 1), "probe pair owners");
    ptable = dalloc<double>((size_t)std::max<long>(npairs, 1) * nw * 6, "probe kernel table");
    {
        cst.push_back((int)clo.size());
        pnck = (long)clo.size();
        ck_lo = dalloc<int>(std::max<size_t>(clo.size(), 1), "probe chunks");
        ck_hi = dalloc<int>(std::max<size_t>(clo.size(), 1), "probe chunks");
        ck_start = dalloc<int>(cst.size(), "probe chunks");
        if (pnck > 0) {
            MJ_CHECK(hipMemcpy(ck_lo, clo.data(), sizeof(int) * clo.size(), hipMemcpyHostToDevice));
            MJ_CHECK(hipMemcpy(ck_hi, chi_.data(), sizeof(int) * chi_.size(), hipMemcpyHostToDevice));
        }
        MJ_CHECK(hipMemcpy(ck_start, cst.data(), sizeof(int) * cst.size(), hipMemcpyHostToDevice));
    }
    ppart = dalloc<double>((size_t)nrhs * std::max<long>(pnck, 1) * mj::kProbeSteps * 3, "probe partial sums");
    MJ_CHECK(hipMemcpy(probe_pos, P.data(), sizeof(double) * P.size(), hipMemcpyHostToDevice));
    if (npairs > 0) {
        MJ_CHECK(hipMemcpy(pair_vox, pv.data(), sizeof(int) * pv.size(), hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(pair_kmin, pk.data(), sizeof(int) * pk.size(), hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(pair_probe, pp.data(), sizeof(int) * pp.size(), hipMemcpyHostToDevice));
        hipEvent_t e0, e1;
        MJ_CHECK(hipEventCreate(&e0));
        MJ_CHECK(hipEventCreate(&e1));
        MJ_CHECK(hipEventRecord(e0, st));
        mj::gen_offgrid_table(probe_pos, pair_probe, pair_vox, pair_kmin, npairs, U, V, gen.r, gen.hv, nw, ell, nquad, ptable, da, st);
        MJ_CHECK(hipEventRecord(e1, st));
        MJ_CHECK(hipEventSynchronize(e1));
        float ms = 0;
        MJ_CHECK(hipEventElapsedTime(&ms, e0, e1));
        t_probe_ms = ms;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    dfree((void *&)pair_probe);
    // the adjoint source walks the table voxel by voxel: a copy in that order
    ptable_v = dalloc<double>((size_t)nw * n_probes * M * 6, "probe kernel table by voxel");
    pkmin_v = dalloc<int>((size_t)n_probes * M, "probe windows by voxel");
    mj::launch_probe_table_by_voxel(ptable, pair_kmin, pinv, npairs, n_probes, nw, M, ptable_v, pkmin_v, st);
    // the probe sums of kProbeSteps steps read J_{n-k} for k = 0..ell from the real-space ring
    if (rdepth < ell + mj::kProbeSteps) {
        const int depth = ell + mj::kProbeSteps;
        double *ring_r = dalloc<double>((size_t)depth * nrhs * 3 * M, "current history");
        dfree((void *&)Jr);
        Jr = ring_r;
        rdepth = depth;
    }
    sdepth = std::max(sdepth, ell + 1);
    MJ_CHECK(hipStreamSynchronize(st));
}

// Kernel values at (probe, voxel, lag) triples through the same off-grid generator.
void mj_solver::offgrid_values(int cnt, const int *probe, const int *vox3, const int *lag, double *out)
{
    if (cnt <= 0) return;
    if (!probe_pos) throw std::logic_error("no probes set");
    std::vector<int> pp(cnt), pv(cnt), pk(cnt);
    for (int i = 0; i < cnt; i++) {
        if (probe[i] < 0 || probe[i] >= np) throw ArgError("probe index out of range");
        const int u = vox3[3 * i], v = vox3[3 * i + 1], w = vox3[3 * i + 2];
        if (u < 0 || u >= U || v < 0 || v >= V || w < 0 || w >= W) throw ArgError("voxel out of range");
        if (lag[i] < 0) throw ArgError("lag < 0");
        pp[i] = probe[i];
        pv[i] = u + U * (v + V * w);
        pk[i] = lag[i];
    }
    int *d_p = nullptr, *d_v = nullptr, *d_k = nullptr;
    double *d_o = nullptr;
    try {
        d_p = (int *)da.get(sizeof(int) * cnt, "probe request");
        d_v = (int *)da.get(sizeof(int) * cnt, "probe request");
        d_k = (int *)da.get(sizeof(int) * cnt, "probe request");
        d_o = (double *)da.get(sizeof(double) * 6 * cnt, "probe values");
        MJ_CHECK(hipMemcpy(d_p, pp.data(), sizeof(int) * cnt, hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(d_v, pv.data(), sizeof(int) * cnt, hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(d_k, pk.data(), sizeof(int) * cnt, hipMemcpyHostToDevice));
        mj::gen_offgrid_table(probe_pos, d_p, d_v, d_k, cnt, U, V, gen.r, gen.hv, 1, 0x7fffffff, nquad, d_o, da, st);
        MJ_CHECK(hipStreamSynchronize(st));
        MJ_CHECK(hipMemcpy(out, d_o, sizeof(double) * 6 * cnt, hipMemcpyDeviceToHost));
    } catch (...) {
        da.put(d_p);
        da.put(d_v);
        da.put(d_k);
        da.put(d_o);
        throw;
    }
    da.put(d_p);
    da.put(d_v);
    da.put(d_k);
    da.put(d_o);
}

// March state: a fixed header, then the spectral ring, the time block's far sums and the
// real-space history, each copied whole (slots the march does not read yet copy as they are).
namespace {
struct StateHeader {
    char magic[8];
    int32_t version, U, V, W, nrhs, ell, B, rdepth, Nx, Ny, Nz, Hp, B2, cheb_pred;
    int64_t n, ring_bytes, far_bytes, jr_bytes, outer_bytes;
};
// version 3 has the replayed passes of the Z_0 solve (their counts and coefficients) after the header;
// version 2, without them, is read too: the solve then takes CG first
constexpr int kStateVersion = 3;
constexpr char kStateMagic[8] = {'M', 'J', 'S', 'T', 'A', 'T', 'E', '2'};
}  // namespace

size_t mj_solver::state_bytes() const
{
    const size_t sp = (size_t)spec_plane(), v3 = (size_t)nrhs * 3;
    return sizeof(StateHeader) + sizeof(Replay) + sizeof(double) * coef_count() + sizeof(double2) * (size_t)ell * v3 * sp +
           (farbuf ? sizeof(double2) * (size_t)B * v3 * sp : 0) + (gbuf ? sizeof(double2) * (size_t)B2 * v3 * sp : 0) +
           sizeof(double) * (size_t)sdepth * v3 * M;
}

void mj_solver::get_state(void *buf) const
{
    const size_t sp = (size_t)spec_plane(), v3 = (size_t)nrhs * 3;
    StateHeader h{};
    std::memcpy(h.magic, kStateMagic, 8);
    h.version = kStateVersion;
    h.U = U;
    h.V = V;
    h.W = W;
    h.nrhs = nrhs;
    h.ell = ell;
    h.B = B;
    h.rdepth = sdepth;
    h.Nx = Nx;
    h.Ny = Ny;
    h.Nz = Nz;
    h.Hp = Hp;
    h.B2 = B2;
    h.cheb_pred = cheb_pred;   // the next Z_0 solve's first batch of passes (part of its arithmetic)
    h.n = n;
    h.ring_bytes = (int64_t)(sizeof(double2) * (size_t)ell * v3 * sp);
    h.far_bytes = farbuf ? (int64_t)(sizeof(double2) * (size_t)B * v3 * sp) : 0;
    h.jr_bytes = (int64_t)(sizeof(double) * (size_t)h.rdepth * v3 * M);
    h.outer_bytes = gbuf ? (int64_t)(sizeof(double2) * (size_t)B2 * v3 * sp) : 0;
    char *p = (char *)buf;
    std::memcpy(p, &h, sizeof h);
    p += sizeof h;
    MJ_CHECK(hipStreamSynchronize(st));
    std::memcpy(p, &rp, sizeof rp);
    p += sizeof rp;
    MJ_CHECK(hipMemcpy(p, coef, sizeof(double) * coef_count(), hipMemcpyDeviceToHost));
    p += sizeof(double) * coef_count();
    MJ_CHECK(hipMemcpy(p, ring, (size_t)h.ring_bytes, hipMemcpyDeviceToHost));
    p += h.ring_bytes;
    if (h.far_bytes) MJ_CHECK(hipMemcpy(p, farbuf, (size_t)h.far_bytes, hipMemcpyDeviceToHost));
    p += h.far_bytes;
    if (h.rdepth == rdepth) {
        MJ_CHECK(hipMemcpy(p, Jr, (size_t)h.jr_bytes, hipMemcpyDeviceToHost));
    } else {
        // step j of the last h.rdepth ones at slot j mod h.rdepth
        const size_t vec = v3 * M;
        std::memset(p, 0, (size_t)h.jr_bytes);
        for (int j = std::max(1, n - h.rdepth + 1); j <= n; j++)
            MJ_CHECK(hipMemcpy(p + (size_t)(j % h.rdepth) * vec * 8, Jr + (size_t)slotR(j) * vec, vec * 8,
                               hipMemcpyDeviceToHost));
    }
    p += h.jr_bytes;
    if (h.outer_bytes) MJ_CHECK(hipMemcpy(p, gbuf, (size_t)h.outer_bytes, hipMemcpyDeviceToHost));
}

void mj_solver::set_state(const void *buf, size_t bytes)
{
    StateHeader h;
    if (bytes < sizeof h) throw ArgError("state buffer too short");
    std::memcpy(&h, buf, sizeof h);
    if (std::memcmp(h.magic, kStateMagic, 8) != 0 || (h.version != kStateVersion && h.version != 2)) throw ArgError("not a march state");
    if (h.U != U || h.V != V || h.W != W || h.nrhs != nrhs || h.ell != ell || h.B != B || h.B2 != B2 ||
        h.Nx != Nx || h.Ny != Ny || h.Nz != Nz || h.Hp != Hp)
        throw ArgError("state of a solver with another grid, n_rhs, ell or time blocks");
    if (h.rdepth != sdepth) throw ArgError("state of a solver with another history depth (probes differ)");
    const size_t solve_bytes = sizeof(Replay) + sizeof(double) * coef_count();
    const size_t need = state_bytes() - (h.version == 2 ? solve_bytes : 0);
    const size_t v3 = (size_t)nrhs * 3, spec = sizeof(double2) * v3 * (size_t)spec_plane();
    // each part by itself: the copies below trust these sizes
    if (bytes < need || (size_t)h.ring_bytes != spec * (size_t)ell || (size_t)h.far_bytes != (farbuf ? spec * (size_t)B : 0) ||
        (size_t)h.jr_bytes != sizeof(double) * (size_t)sdepth * v3 * (size_t)M ||
        (size_t)h.outer_bytes != (gbuf ? spec * (size_t)B2 : 0))
        throw ArgError("state buffer has the wrong size");
    if (h.n < 0 || h.n > INT32_MAX) throw ArgError("bad step count in the state");
    const char *p = (const char *)buf + sizeof h;
    Replay rp_new;
    if (h.version != 2) {
        std::memcpy(&rp_new, p, sizeof rp_new);
        auto in = [](int x, int most) { return x >= 0 && x <= most; };
        if (!in(rp_new.K, mj::kMaxCoef - 1) || !in(rp_new.K0, mj::kMaxCoef - 1) || !in(rp_new.L, mj::kMaxCoef) ||
            !in(rp_new.fails, kMaxFails) || !in(rp_new.hold, 4 << kMaxFails) || (rp_new.K < 1 && !rp_new.learn))
            throw ArgError("bad solve record in the state");
    }
    drop_side();
    MJ_CHECK(hipStreamSynchronize(st));
    rp = rp_new;
    if (h.version != 2) {
        MJ_CHECK(hipMemcpy(coef, p + sizeof(Replay), sizeof(double) * coef_count(), hipMemcpyHostToDevice));
        p += solve_bytes;
    }
    MJ_CHECK(hipMemcpy(ring, p, (size_t)h.ring_bytes, hipMemcpyHostToDevice));
    p += h.ring_bytes;
    if (h.far_bytes) MJ_CHECK(hipMemcpy(farbuf, p, (size_t)h.far_bytes, hipMemcpyHostToDevice));
    p += h.far_bytes;
    if (h.rdepth == rdepth) {
        MJ_CHECK(hipMemcpy(Jr, p, (size_t)h.jr_bytes, hipMemcpyHostToDevice));
    } else {
        const size_t vec = (size_t)nrhs * 3 * M;
        for (int j = (int)std::max<int64_t>(1, h.n - h.rdepth + 1); j <= h.n; j++)
            MJ_CHECK(hipMemcpy(Jr + (size_t)slotR(j) * vec, p + (size_t)(j % h.rdepth) * vec * 8, vec * 8,
                               hipMemcpyHostToDevice));
    }
    p += h.jr_bytes;
    if (h.outer_bytes) MJ_CHECK(hipMemcpy(gbuf, p, (size_t)h.outer_bytes, hipMemcpyHostToDevice));
    n = (int)h.n;
    cheb_pred = std::max(0, (int)h.cheb_pred);
}

// Gradient of Phi = sum_{n=1}^{N} sum_r sum_p |E^s_{r,p}(n)|^2 with respect to eps_r of every
// voxel, by the transposed march (see mj_march.hip) with checkpointing:
//  1. forward march of all N steps, keeping the probe field of every step and, at the start
//     of every segment but the first, the real-space history J_{n0-ell-1} .. J_{n0-1} that a
//     restart at n0 needs; segments start at time-block starts, so a restart begins with a
//     far-part launch like the original march did;
//  2. segments from last to first: recompute the segment's forward steps from its checkpoint
//     (the last one is kept from step 1), storing B_n, then run the transposed march over the
//     segment's steps in reversed time, accumulating lambda_n . B_n / eps^2.
// The recomputed steps repeat the original arithmetic exactly.  Leaves the march at n = 0.
void mj_solver::adjoint_gradient(int N, int ckpt_every, double *phi, double *grad_dev, double *probe_hist)
{
    if (!waves_set) throw std::logic_error("plane waves not set (mj_set_plane_waves)");
    if (np <= 0) throw std::logic_error("the objective is the probe field: set probes first");
    if (n != 0) throw std::logic_error("the gradient run starts at n = 0 (mj_reset)");
    if (N < 1) throw ArgError("n_steps must be >= 1");
    if (rdepth < ell + 1) throw std::logic_error("probe history depth");
    // segment starts: 1, then block starts 2 + c L with L a multiple of the time block
    int L = ckpt_every > 0 ? ckpt_every : N;
    // restarts at (outer) time-block starts repeat the original arithmetic exactly
    const int period = B2 ? B2 : B;
    if (period > 1) L = ((L + period - 1) / period) * period;
    std::vector<int> starts{1};
    for (long s0 = 2 + (long)L; s0 <= N; s0 += L) starts.push_back((int)s0);
    const int C = (int)starts.size();
    auto seg_end = [&](int c) { return c + 1 < C ? starts[c + 1] - 1 : N; };
    int maxseg = 0;
    for (int c = 0; c < C; c++) maxseg = std::max(maxseg, seg_end(c) - starts[c] + 1);
    const size_t vec = (size_t)nrhs * 3 * M;
    // every step j that a restart reads (j = s0 - 1 - ell .. s0 - 1 for a segment start s0 > 1)
    // is kept once, in one pool indexed through pool_of[j], however the windows overlap
    std::vector<long> pool_of((size_t)N + 1, -1);
    long npool = 0;
    for (int c = 1; c < C; c++)
        for (int j = std::max(1, starts[c] - 1 - ell); j <= starts[c] - 1; j++)
            if (pool_of[(size_t)j] < 0) pool_of[(size_t)j] = 1;
    for (int j = 1; j <= N; j++)
        if (pool_of[(size_t)j] > 0) pool_of[(size_t)j] = npool++;
    const long sp = spec_plane();
    std::vector<void *> tmp;
    auto talloc = [&](size_t bytes, const char *what) {
        void *ptr = nullptr;
        try {
            ptr = da.get(std::max<size_t>(bytes, 8), what);
        } catch (...) {
            for (void *q : tmp) da.put(q);
            throw;
        }
        tmp.push_back(ptr);
        return ptr;
    };
    double *Ehist = (double *)talloc(sizeof(double) * (size_t)N * nrhs * np * 3, "probe history");
    double *ckpt = (double *)talloc(sizeof(double) * (size_t)std::max<long>(npool, 1) * vec, "checkpoints");
    double *Bbuf = (double *)talloc(sizeof(double) * (size_t)maxseg * vec, "gradient terms");
    double *G = (double *)talloc(sizeof(double) * mj::kProbeSteps * vec, "adjoint source");
    double *bqb = (double *)talloc(sizeof(double) * vec, "adjoint rhs");
    double2 *ring_a = (double2 *)talloc(sizeof(double2) * (size_t)ell * nrhs * 3 * sp, "adjoint ring");
    double2 *far_a = B > 1 ? (double2 *)talloc(sizeof(double2) * (size_t)B * nrhs * 3 * sp, "adjoint blocks") : nullptr;
    double2 *g_a = B2 ? (double2 *)talloc(sizeof(double2) * (size_t)B2 * nrhs * 3 * sp, "adjoint outer blocks") : nullptr;
    double *nu_r = (double *)talloc(sizeof(double) * (size_t)rdepth * vec, "adjoint history");
    double *lam_r = (double *)talloc(sizeof(double) * (size_t)rdepth * vec, "adjoint local history");
    MJ_CHECK(hipMemsetAsync(grad_dev, 0, sizeof(double) * M, st));
    // what the solve of a segment's first step starts from (passes predicted or recorded), kept so that
    // a recomputed segment repeats the original arithmetic; the transposed march has its own
    struct SolveRecord {
        int cheb_pred = 0;
        Replay rp;
    };
    std::vector<SolveRecord> rec_at((size_t)C);
    SolveRecord rec_adj;
    double *coef_at = (double *)talloc(sizeof(double) * (size_t)(C + 1) * coef_count(), "recorded coefficients");
    auto save_record = [&](SolveRecord &sr, int slot) {
        sr = SolveRecord{cheb_pred, rp};
        MJ_CHECK(hipMemcpyAsync(coef_at + (size_t)slot * coef_count(), coef, sizeof(double) * coef_count(),
                                hipMemcpyDeviceToDevice, st));
    };
    auto load_record = [&](const SolveRecord &sr, int slot) {
        cheb_pred = sr.cheb_pred;
        rp = sr.rp;
        if (!rp.learn)
            MJ_CHECK(hipMemcpyAsync(coef, coef_at + (size_t)slot * coef_count(), sizeof(double) * coef_count(),
                                    hipMemcpyDeviceToDevice, st));
    };
    double2 *const ring_f = ring, *const far_f = farbuf, *const g_f = gbuf;
    double *const Jr_f = Jr;
    hipEvent_t tev[3];
    for (auto &tv : tev) MJ_CHECK(hipEventCreate(&tv));
    MJ_CHECK(hipEventRecord(tev[0], st));
    bool noconv = false;
    auto check_cg = [&] {
        for (int i = 0; i < nrhs; i++)
            if (!cgstat_h[i].done) noconv = true;
    };
    transformed = -1;
    try {
        // 1. forward
        const int last0 = starts[C - 1];
        int seg = 0;
        for (int t = 1; t <= N; t++) {
            if (seg < C && t == starts[(size_t)seg]) {
                save_record(rec_at[(size_t)seg], seg);
                seg++;
            }
            StepIO io;
            io.Pout = Ehist + (size_t)(t - 1) * nrhs * np * 3;
            io.Bout = t >= last0 ? Bbuf + (size_t)(t - last0) * vec : nullptr;
            io.more = t < N;
            step(io);
            check_growth();
            check_cg();
            if (pool_of[(size_t)t] >= 0)
                MJ_CHECK(hipMemcpyAsync(ckpt + (size_t)pool_of[(size_t)t] * vec, Jr + (size_t)slotR(t) * vec,
                                        sizeof(double) * vec, hipMemcpyDeviceToDevice, st));
        }
        flush_probes();
        if (probe_hist)
            MJ_CHECK(hipMemcpyAsync(probe_hist, Ehist, sizeof(double) * (size_t)N * nrhs * np * 3,
                                    hipMemcpyDeviceToDevice, st));
        std::vector<double> Eh((size_t)N * nrhs * np * 3);
        MJ_CHECK(hipMemcpyAsync(Eh.data(), Ehist, sizeof(double) * Eh.size(), hipMemcpyDeviceToHost, st));
        MJ_CHECK(hipStreamSynchronize(st));
        double ph = 0.0;
        for (double v : Eh) ph += v * v;
        if (phi) *phi = ph;
        MJ_CHECK(hipEventRecord(tev[1], st));
        // 2. backward; the transposed march has its own rings, swapped in while it runs
        int n_adj = 0;
        for (int c = C - 1; c >= 0; c--) {
            const int s0 = starts[c], s1 = seg_end(c);
            if (c < C - 1) {
                // restart the forward march at s0 from its checkpoint and recompute the segment
                drop_side();
                n = s0 - 1;
                transformed = -1;
                if (c > 0) {
                    const int j0 = s0 - 1 - ell;   // first stored step
                    for (int j = std::max(1, j0); j <= s0 - 1; j++) {
                        const double *src = ckpt + (size_t)pool_of[(size_t)j] * vec;
                        MJ_CHECK(hipMemcpyAsync(Jr + (size_t)slotR(j) * vec, src, sizeof(double) * vec,
                                                hipMemcpyDeviceToDevice, st));
                        if (j <= s0 - 2)
                            mj::fft3d_forward(fft, src, ring + (size_t)slotS(j) * nrhs * 3 * sp, 3 * nrhs, st);
                    }
                }
                load_record(rec_at[(size_t)c], c);
                for (int t = s0; t <= s1; t++) {
                    StepIO io;
                    io.Bout = Bbuf + (size_t)(t - s0) * vec;
                    io.more = t < s1;
                    step(io);
                    check_cg();
                }
            }
            // transposed march over j = s1 .. s0 (reversed step n' = N + 1 - j)
            drop_side();
            ring = ring_a;
            farbuf = far_a;
            gbuf = g_a;
            Jr = nu_r;
            Lr = lam_r;
            bq = bqb;
            n = n_adj;
            transformed = -1;
            load_record(rec_adj, C);
            for (int j = s1; j >= s0; j--) {
                const int at = (s1 - j) % mj::kProbeSteps;   // the source of up to kProbeSteps steps at once
                if (at == 0) {
                    mj::AdjArg a = adj_arg();
                    a.Ehist = Ehist;
                    a.N = N;
                    a.j = j;
                    a.ntarget = std::min(mj::kProbeSteps, j - s0 + 1);
                    a.G = G;
                    mj::launch_adj_source(a, st);
                }
                StepIO io;
                io.adjoint = true;
                io.G = G + (size_t)at * vec;
                io.Bj = Bbuf + (size_t)(j - s0) * vec;
                io.grad = grad_dev;
                io.more = j > s0;
                step(io);
                check_cg();
            }
            n_adj = n;
            save_record(rec_adj, C);
            drop_side();
            ring = ring_f;
            farbuf = far_f;
            gbuf = g_f;
            Jr = Jr_f;
            Lr = nullptr;
            bq = nullptr;
        }
        MJ_CHECK(hipEventRecord(tev[2], st));
        MJ_CHECK(hipStreamSynchronize(st));
    } catch (...) {
        (void)hipStreamSynchronize(st);
        if (side) (void)hipStreamSynchronize(side);
        side_pending = false;
        h_block = 0;
        ring = ring_f;
        farbuf = far_f;
        gbuf = g_f;
        Jr = Jr_f;
        Lr = nullptr;
        bq = nullptr;
        probe_steps = 0;
        for (void *q : tmp) da.put(q);
        for (auto &tv : tev) (void)hipEventDestroy(tv);
        rp = Replay();
        cheb_pred = 0;
        n = 0;
        throw;
    }
    float f_ms = 0, b_ms = 0;
    MJ_CHECK(hipEventElapsedTime(&f_ms, tev[0], tev[1]));
    MJ_CHECK(hipEventElapsedTime(&b_ms, tev[1], tev[2]));
    stat[14] = f_ms;
    stat[15] = b_ms;
    stat[16] = C;
    stat[17] = (double)npool * vec * sizeof(double);
    for (void *q : tmp) da.put(q);
    for (auto &tv : tev) (void)hipEventDestroy(tv);
    rp = Replay();   // the next march records its own
    cheb_pred = 0;
    n = 0;
    if (noconv) throw std::range_error("Z_0 solve did not converge");
}

// ============================================================================ C ABI
namespace {
int fail(mj_solver *s, int code, const std::string &msg)
{
    if (s) s->err = msg;
    else g_err = msg;
    return code;
}

template <class F>
int guarded(mj_solver *s, F &&f)
{
    try {
        f();
        return MJ_OK;
    } catch (const ArgError &e) {
        return fail(s, MJ_EINVAL, e.what());
    } catch (const MemError &e) {
        return fail(s, MJ_ENOMEM, e.what());
    } catch (const HipError &e) {
        return fail(s, MJ_EHIP, e.what());
    } catch (const UnstableError &e) {
        return fail(s, MJ_EUNSTABLE, e.what());
    } catch (const std::range_error &e) {
        return fail(s, MJ_ENOCONV, e.what());
    } catch (const std::logic_error &e) {
        return fail(s, MJ_ESTATE, e.what());
    } catch (const std::exception &e) {
        return fail(s, MJ_EHIP, e.what());
    } catch (...) {
        return fail(s, MJ_EHIP, "unknown error");
    }
}
}  // namespace

extern "C" {

int mj_create(const mj_config *cfg, mj_solver **out)
{
    if (!cfg || !out) return fail(nullptr, MJ_EINVAL, "NULL argument");
    *out = nullptr;
    mj_solver *s = new (std::nothrow) mj_solver();
    if (!s) return fail(nullptr, MJ_ENOMEM, "host allocation failed");
    int rc = guarded(nullptr, [&] { s->create(*cfg); });
    if (rc != MJ_OK) {
        delete s;
        return rc;
    }
    *out = s;
    return MJ_OK;
}

void mj_destroy(mj_solver *s) { delete s; }

const char *mj_last_error(const mj_solver *s) { return s ? s->err.c_str() : g_err.c_str(); }

int mj_info(const mj_solver *s, double *out, int32_t n)
{
    if (!s || !out) return MJ_EINVAL;
    double v[24] = {(double)s->ell, (double)s->Nx, (double)s->Ny, (double)s->Nz, (double)s->B,
                    (double)s->sdepth, (double)s->nrhs, (double)s->n, (double)s->bytes, s->t_gen_ms,
                    s->t_spec_ms, (double)s->fir.size(), (double)s->np, (double)s->nw, (double)s->npairs,
                    s->t_probe_ms, (double)s->fft.Px, (double)s->fft.Py, (double)s->fft.Pz, (double)s->B2,
                    (double)s->z0_method, s->lam_lo, s->lam_hi, s->overlap ? 1.0 : 0.0};
    for (int i = 0; i < n && i < 24; i++) out[i] = v[i];
    return MJ_OK;
}

int mj_set_plane_waves(mj_solver *s, const double *khat, const double *pol, const double *width, const double *ct0,
                       const double *amp, const double *r_ref)
{
    if (!s) return MJ_EINVAL;
    return guarded(s, [&] {
        if (!khat || !pol || !width || !ct0 || !amp || !r_ref) throw ArgError("NULL wave parameter");
        std::vector<mj::WaveArg> w(s->nrhs);
        for (int i = 0; i < s->nrhs; i++) {
            double kn = 0;
            for (int c = 0; c < 3; c++) {
                w[i].k[c] = khat[3 * i + c];
                w[i].pol[c] = pol[3 * i + c];
                w[i].rref[c] = r_ref[3 * i + c];
                kn += khat[3 * i + c] * khat[3 * i + c];
            }
            if (!(std::fabs(kn - 1.0) < 1e-12)) throw ArgError("khat must be a unit vector");
            if (!(width[i] > 0.0) || !std::isfinite(width[i])) throw ArgError("width must be positive and finite");
            bool fin = std::isfinite(ct0[i]) && std::isfinite(amp[i]);
            for (int c = 0; c < 3; c++) fin = fin && std::isfinite(pol[3 * i + c]) && std::isfinite(r_ref[3 * i + c]);
            if (!fin) throw ArgError("wave parameters must be finite");
            w[i].width = width[i];
            w[i].ct0 = ct0[i];
            w[i].amp = amp[i];
            plan_wave(w[i], s->h, s->hy, s->hz);
        }
        MJ_CHECK(hipMemcpy(s->waves_d, w.data(), sizeof(mj::WaveArg) * s->nrhs, hipMemcpyHostToDevice));
        s->waves = w;
        s->waves_set = true;
    });
}

int mj_run(mj_solver *s, int32_t n_steps, double *J_hist)
{
    if (!s) return MJ_EINVAL;
    if (n_steps < 0) return fail(s, MJ_EINVAL, "n_steps < 0");
    return guarded(s, [&] { s->run(n_steps, J_hist, nullptr); });
}

int mj_march(mj_solver *s, int32_t n_steps, double *J_hist, double *probe_hist)
{
    if (!s) return MJ_EINVAL;
    if (n_steps < 0) return fail(s, MJ_EINVAL, "n_steps < 0");
    return guarded(s, [&] { s->run(n_steps, J_hist, probe_hist); });
}

int mj_step(mj_solver *s, double *J_dev, double *probe)
{
    if (!s) return MJ_EINVAL;
    return guarded(s, [&] { s->run(1, J_dev, probe); });
}

int mj_march_every(mj_solver *s, int32_t n_steps, int32_t j_every, double *J_hist, double *probe_hist)
{
    if (!s) return MJ_EINVAL;
    if (n_steps < 0) return fail(s, MJ_EINVAL, "n_steps < 0");
    if (j_every < 1) return fail(s, MJ_EINVAL, "j_every < 1");
    return guarded(s, [&] { s->run(n_steps, J_hist, probe_hist, j_every); });
}

int mj_set_eps(mj_solver *s, const double *eps_r)
{
    if (!s || !eps_r) return MJ_EINVAL;
    return guarded(s, [&] {
        if (s->n != 0) throw std::logic_error("eps is changed at n = 0 (after mj_create or mj_reset)");
        s->set_material(eps_r);
        s->restart();
        if (s->z0_method == 0) s->estimate_spectrum();
    });
}

int mj_adjoint_gradient(mj_solver *s, int32_t n_steps, int32_t ckpt_every, double *phi, double *dphi_deps,
                        double *probe_hist)
{
    if (!s || !dphi_deps) return MJ_EINVAL;
    if (n_steps < 1) return fail(s, MJ_EINVAL, "n_steps < 1");
    return guarded(s, [&] { s->adjoint_gradient(n_steps, ckpt_every, phi, dphi_deps, probe_hist); });
}

int mj_set_probes(mj_solver *s, int32_t n_probes, const double *pos)
{
    if (!s) return MJ_EINVAL;
    return guarded(s, [&] { s->set_probes(n_probes, pos); });
}

int mj_probe_kernel_values(mj_solver *s, int32_t n, const int32_t *probe, const int32_t *voxel,
                           const int32_t *lag, double *out)
{
    if (!s) return MJ_EINVAL;
    if (n < 0 || (n > 0 && (!probe || !voxel || !lag || !out))) return fail(s, MJ_EINVAL, "bad arguments");
    return guarded(s, [&] { s->offgrid_values(n, probe, voxel, lag, out); });
}

int mj_reset(mj_solver *s)
{
    if (!s) return MJ_EINVAL;
    return guarded(s, [&] { s->restart(); });
}

int mj_get_state(const mj_solver *s, void *buf, size_t *bytes)
{
    if (!s || !bytes) return MJ_EINVAL;
    mj_solver *sm = const_cast<mj_solver *>(s);
    return guarded(sm, [&] {
        const size_t need = s->state_bytes();
        if (buf) {
            if (*bytes < need) throw ArgError("state buffer too small");
            s->get_state(buf);
        }
        *bytes = need;
    });
}

int mj_set_state(mj_solver *s, const void *buf, size_t bytes)
{
    if (!s) return MJ_EINVAL;
    if (!buf) return fail(s, MJ_EINVAL, "state buffer is NULL");
    return guarded(s, [&] { s->set_state(buf, bytes); });
}

int mj_history_sum(mj_solver *s, const double *J_hist, int32_t depth, double *P)
{
    if (!s) return MJ_EINVAL;
    if (!J_hist || !P || depth < 1) return fail(s, MJ_EINVAL, "bad history arguments");
    return guarded(s, [&] { s->history_sum(J_hist, depth, P); });
}

int mj_kernel_values(mj_solver *s, int32_t n, const int32_t *lag, const int32_t *offset, double *out)
{
    if (!s) return MJ_EINVAL;
    if (n < 0 || (n > 0 && (!lag || !offset || !out))) return fail(s, MJ_EINVAL, "bad kernel value request");
    return guarded(s, [&] {
        for (int i = 0; i < n; i++) {
            if (lag[i] < 0 || lag[i] > s->ell) throw ArgError("lag out of range");
            if (std::abs(offset[3 * i]) >= s->U || std::abs(offset[3 * i + 1]) >= s->V ||
                std::abs(offset[3 * i + 2]) >= s->W)
                throw ArgError("offset out of range");
        }
        if (n == 0) return;
        mj::DevTemp tl(s->da, sizeof(int) * n, "kernel value request");
        mj::DevTemp to(s->da, sizeof(int) * 3 * n, "kernel value request");
        mj::DevTemp tv(s->da, sizeof(double) * 6 * n, "kernel values");
        int *lag_d = tl.as<int>(), *off_d = to.as<int>();
        double *out_d = tv.as<double>();
        MJ_CHECK(hipMemcpy(lag_d, lag, sizeof(int) * n, hipMemcpyHostToDevice));
        MJ_CHECK(hipMemcpy(off_d, offset, sizeof(int) * 3 * n, hipMemcpyHostToDevice));
        mj::gen_kernel_values(s->gen, n, lag_d, off_d, out_d, s->st);
        MJ_CHECK(hipMemcpyAsync(out, out_d, sizeof(double) * 6 * n, hipMemcpyDeviceToHost, s->st));
        MJ_CHECK(hipStreamSynchronize(s->st));
    });
}

int mj_kernel_values_noalloc(mj_solver *s, int32_t n, const int32_t *lag, const int32_t *offset, double *out)
{
    if (!s) return MJ_EINVAL;
    if (n < 0 || (n > 0 && (!lag || !offset || !out))) return fail(s, MJ_EINVAL, "bad kernel value request");
    if (n > kNoAllocMax)
        return fail(s, MJ_EINVAL, "at most " + std::to_string(kNoAllocMax) + " requests per call (staging array size)");
    return guarded(s, [&] {
        for (int i = 0; i < n; i++) {
            if (lag[i] < 0 || lag[i] > s->ell) throw ArgError("lag out of range");
            if (std::abs(offset[3 * i]) >= s->U || std::abs(offset[3 * i + 1]) >= s->V ||
                std::abs(offset[3 * i + 2]) >= s->W)
                throw ArgError("offset out of range");
        }
        if (n == 0) return;
        int cur = -1;
        MJ_CHECK(hipGetDevice(&cur));
        if (cur != s->dev) throw ArgError("call with the solver's device current");
        unsigned char *base = scratch_ptr(cur);
        double *out_d = (double *)base;
        int32_t *lag_d = (int32_t *)(base + (size_t)kNoAllocMax * 6 * sizeof(double));
        int32_t *off_d = lag_d + kNoAllocMax;
        std::lock_guard<std::mutex> lk(g_noalloc_mu);
        MJ_CHECK(hipMemcpyAsync(lag_d, lag, sizeof(int32_t) * n, hipMemcpyHostToDevice, s->st));
        MJ_CHECK(hipMemcpyAsync(off_d, offset, sizeof(int32_t) * 3 * n, hipMemcpyHostToDevice, s->st));
        mj::gen_kernel_values(s->gen, n, lag_d, off_d, out_d, s->st);
        MJ_CHECK(hipMemcpyAsync(out, out_d, sizeof(double) * 6 * n, hipMemcpyDeviceToHost, s->st));
        MJ_CHECK(hipStreamSynchronize(s->st));
    });
}

int mj_stats(const mj_solver *s, double *out, int32_t n)
{
    if (!s || !out) return MJ_EINVAL;
    for (int i = 0; i < n && i < 21; i++) out[i] = s->stat[i];
    return MJ_OK;
}

int mj_fft_roundtrip(mj_solver *s, const double *x, double *X, double *yout)
{
    if (!s || !x) return MJ_EINVAL;
    return guarded(s, [&] {
        // the spectrum is held with row pitch Hp; the caller's X has rows of Hx
        double2 *Xd = s->Shat;
        mj::fft3d_forward(s->fft, x, Xd, 3, s->st);
        if (X)
            MJ_CHECK(hipMemcpy2DAsync(X, sizeof(double2) * s->Hx, Xd, sizeof(double2) * s->Hp, sizeof(double2) * s->Hx,
                                      (size_t)3 * s->Nz * s->Ny, hipMemcpyDeviceToDevice, s->st));
        if (yout) mj::fft3d_inverse(s->fft, Xd, yout, 3, s->st);
        MJ_CHECK(hipStreamSynchronize(s->st));
    });
}

}  // extern "C"
