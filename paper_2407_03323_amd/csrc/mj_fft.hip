// Padded 3-D FFTs of real vector fields (FP64), hand-written for gfx950.
//
// The history sum uses the circulant embedding of the three-level block-Toeplitz
// interaction matrices (Appendix A): fields on the U x V x W voxel box are
// zero-padded to an Nx x Ny x Nz grid with N >= 2U - 1 per axis, transformed,
// multiplied point-wise in the spectral domain and transformed back; only the
// box part of the inverse is kept.
//
// Lengths that split into two factors of at most 16 are transformed in registers with one exchange
// through LDS (k_fft2_*).  For the others, each 1-D pass loads a tile of pencils into LDS, runs a Stockham autosort FFT
// (decimation in time, natural-order output) stage by stage in place (each stage
// reads its butterflies into registers, synchronises, writes them back), and
// writes the tile back.  Pencils along y and z are strided in
// memory; a tile covers consecutive x-frequencies so every global access is a
// run of consecutive complex values.  The x pass packs two real rows into one
// complex pencil (real and imaginary part) and separates the two half-spectra
// afterwards (and the reverse for the inverse).  Zero padding is never stored:
// the forward passes read only the U (V, W) live inputs, the inverse passes
// write only the box outputs.
//
// Twiddles come from a table W_N^m computed on the host in long double and
// rounded once, so no recurrence error accumulates.

#include "mj_internal.h"

#include <algorithm>
#include <cmath>

namespace mj {

namespace {

constexpr int kThreads = 256;

// Division by a divisor that is the same in every lane (a tile or plan size), by one multiply:
// for x < 2^16 and 1 <= d <= 2^16, floor(x / d) = floor(x m / 2^32) with m = floor(2^32 / d) + 1,
// since x m / 2^32 exceeds x / d by less than 2^-16 and the fraction of x / d is at most
// 1 - 1/d.  Building m is scalar work (d is uniform); the per-element quotient replaces the
// reciprocal-and-correct sequence of a division by a run-time divisor, which dominated the
// integer work of the index arithmetic.  Every index divided here is below 2^16.
struct FastDiv {
    unsigned d;
    unsigned long long m;
    __device__ explicit FastDiv(unsigned dv) : d(dv), m((1ull << 32) / dv + 1) {}
    __device__ unsigned div(unsigned x) const { return (unsigned)(((unsigned long long)x * m) >> 32); }
    __device__ unsigned mod(unsigned x) const { return x - div(x) * d; }
};

__device__ inline double2 tw_at(const double2 *tw, int m, bool inv)
{
    double2 w = tw[m];
    return inv ? make_double2(w.x, -w.y) : w;
}

// cos(2 pi m / R) and sin(2 pi m / R), m = 1 .. (R-1)/2, of the odd radices, interleaved, from
// offset odd_base(R).  They are the same for every N, so they sit in constant memory, where the
// compiler keeps them in scalar registers.
__constant__ double c_odd_cs[2 * (1 + 2 + 3 + 5 + 6)];
constexpr int odd_base(int R) { return R == 3 ? 0 : R == 5 ? 2 : R == 7 ? 6 : R == 11 ? 12 : 22; }

// In-register R-point DFT, v[q] <- sum_t v[t] W_R^{q t} (W_R = exp(-+2 pi i / R)).
template <int R>
__device__ inline void dft_small(double2 *v, const double2 *tw, int N, bool inv)
{
    if constexpr (R == 2) {
        double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 4) {
        double2 a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3];
        double2 s02 = cadd(a0, a2), d02 = csub(a0, a2);
        double2 s13 = cadd(a1, a3), d13 = csub(a1, a3);
        // forward: -i * d13 ; inverse: +i * d13
        double2 r = inv ? make_double2(-d13.y, d13.x) : make_double2(d13.y, -d13.x);
        v[0] = cadd(s02, s13);
        v[2] = csub(s02, s13);
        v[1] = cadd(d02, r);
        v[3] = csub(d02, r);
    } else {
        // odd R: pair inputs t and R - t.  With a_t = v_t + v_{R-t}, b_t = v_t - v_{R-t},
        // c_m = cos(2 pi m / R), s_m = sin(2 pi m / R) and sg = -1 (forward) or +1 (inverse):
        //   out_q     = v_0 + sum_t a_t c_{qt} + i sg sum_t b_t s_{qt}
        //   out_{R-q} = v_0 + sum_t a_t c_{qt} - i sg sum_t b_t s_{qt}     (q, t = 1 .. (R-1)/2)
        static_assert(R % 2 == 1, "even radices other than 2 and 4 are not used");
        constexpr int H = (R - 1) / 2;
        double cm[H + 1], sm[H + 1];
#pragma unroll
        for (int m = 1; m <= H; m++) {
            cm[m] = c_odd_cs[odd_base(R) + 2 * (m - 1)];
            sm[m] = c_odd_cs[odd_base(R) + 2 * (m - 1) + 1];
        }
        double2 a[H + 1], b[H + 1];
        double2 sum = v[0];
#pragma unroll
        for (int t = 1; t <= H; t++) {
            a[t] = cadd(v[t], v[R - t]);
            b[t] = csub(v[t], v[R - t]);
            sum = cadd(sum, a[t]);
        }
        const double sg = inv ? 1.0 : -1.0;
        const double2 v0 = v[0];
        v[0] = sum;
#pragma unroll
        for (int q = 1; q <= H; q++) {
            double2 A = v0, B = make_double2(0.0, 0.0);
#pragma unroll
            for (int t = 1; t <= H; t++) {
                const int m = (q * t) % R;
                // cos is even and sin odd about R/2: fold m into 1 .. H
                const double c = m <= H ? cm[m] : cm[R - m];
                const double sn = m <= H ? sm[m] : -sm[R - m];
                A.x += a[t].x * c;
                A.y += a[t].y * c;
                B.x += b[t].x * sn;
                B.y += b[t].y * sn;
            }
            // i sg B = (-sg B.y, sg B.x)
            const double2 iB = make_double2(-sg * B.y, sg * B.x);
            v[q] = cadd(A, iB);
            v[R - q] = csub(A, iB);
        }
    }
}

// A tile holds at most kTileElems complex values (P pencils of length N, P * N <= kTileElems).
constexpr int kTileElems = 3072;
static_assert(kMaxFftN <= kTileElems, "one pencil must fit a tile");

// One Stockham stage, in place, on P pencils of length N stored with leading dimension ld.
// Every thread first reads and transforms all of its butterflies (at most BF of them), the
// block synchronises, and only then are the results written back over the inputs; the caller
// synchronises again before the next stage.
template <int R>
__device__ void stage(double2 *buf, int N, int Ns, int P, int ld, const double2 *tw, bool inv)
{
    constexpr int BF = (kTileElems / R + kThreads - 1) / kThreads;
    const int nb = N / R;
    const int step = N / (Ns * R);
    const int total = P * nb;
    const FastDiv fnb(nb), fns(Ns);
    double2 v[BF][R];
#pragma unroll
    for (int f = 0; f < BF; f++) {
        const int b = (int)threadIdx.x + f * kThreads;
        if (b < total) {
            const int p = fnb.div(b), j = b - p * nb, jm = fns.mod(j);
            const double2 *s = buf + p * ld;
#pragma unroll
            for (int r = 0; r < R; r++) v[f][r] = s[j + r * nb];
#pragma unroll
            for (int r = 1; r < R; r++) v[f][r] = cmul(v[f][r], tw_at(tw, jm * r * step, inv));
            dft_small<R>(v[f], tw, N, inv);
        }
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < BF; f++) {
        const int b = (int)threadIdx.x + f * kThreads;
        if (b < total) {
            const int p = fnb.div(b), j = b - p * nb, jq = fns.div(j), jm = j - jq * Ns;
            const int base = jq * Ns * R + jm;
            double2 *d = buf + p * ld;
#pragma unroll
            for (int r = 0; r < R; r++) d[base + r * Ns] = v[f][r];
        }
    }
}

struct PlanArg {
    int N, nst;
    int radix[kMaxStages];
};

// Radix sets: a kernel instantiated for set MASK holds code (and registers) only for the
// radices in it.  The generic instance kAll serves every plan.
constexpr int kR2 = 1, kR3 = 2, kR4 = 4, kR5 = 8, kR7 = 16, kR11 = 32, kR13 = 64, kAll = 127;

// Stage of radix R for a plan whose radices lie in MASK: tests the radices of MASK in turn;
// the last one is taken without a test (the plan guarantees R is in MASK).
constexpr int kRadixOfBit[7] = {2, 3, 4, 5, 7, 11, 13};
constexpr int lowest_bit(int m) { return (m & 1) ? 0 : 1 + lowest_bit(m >> 1); }

template <int MASK>
__device__ inline void stage_of(int R, double2 *buf, int N, int Ns, int P, int ld, const double2 *tw, bool inv)
{
    constexpr int b = lowest_bit(MASK);
    constexpr int RB = kRadixOfBit[b];
    constexpr int REST = MASK & ~(1 << b);
    if constexpr (REST == 0) {
        stage<RB>(buf, N, Ns, P, ld, tw, inv);
    } else {
        if (R == RB) stage<RB>(buf, N, Ns, P, ld, tw, inv);
        else stage_of<REST>(R, buf, N, Ns, P, ld, tw, inv);
    }
}

// Runs all stages in place on the tile in buf.
template <int MASK>
__device__ void lds_fft(double2 *buf, int P, int ld, const PlanArg &pl, const double2 *tw, bool inv)
{
    int Ns = 1;
    for (int s = 0; s < pl.nst; s++) {
        const int R = pl.radix[s];
        stage_of<MASK>(R, buf, pl.N, Ns, P, ld, tw, inv);
        __syncthreads();
        Ns *= R;
    }
}

__device__ inline void load_twiddles(double2 *tw_s, const double2 *tw, int N)
{
    for (int i = threadIdx.x; i < N; i += blockDim.x) tw_s[i] = tw[i];
}

// Moves a tile from global memory into LDS: every thread first issues kBatch independent
// loads (get(i) for items i = i0 + u * kThreads + tid), then stores them (put(i, v)), so
// that the loads of a thread overlap instead of each waiting out the memory latency.
constexpr int kBatch = 8;
template <typename T, class Get, class Put>
__device__ inline void gather_tile(int total, Get get, Put put)
{
    for (int i0 = 0; i0 < total; i0 += kThreads * kBatch) {
        T v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
            const int i = i0 + u * kThreads + (int)threadIdx.x;
            v[u] = i < total ? get(i) : T{};
        }
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
            const int i = i0 + u * kThreads + (int)threadIdx.x;
            if (i < total) put(i, v[u]);
        }
    }
}

// ---------------------------------------------------------------------------- x pass
// Forward: rows of U reals (row r at x + r*U), nrows rows; two rows per pencil.
// Output: rows of Hx complex at X + r*Hp.
template <int MASK>
__global__ void __launch_bounds__(kThreads) k_fft_x_fwd(const double *__restrict__ x, double2 *__restrict__ X,
                                                        int nrows, int U, int Hx, int Hp, PlanArg pl, const double2 *tw,
                                                        int P)
{
    extern __shared__ double2 sm[];
    const int N = pl.N, ld = N + 1;
    double2 *tw_s = sm;
    double2 *a = sm + N;
    load_twiddles(tw_s, tw, N);
    const int row0 = (int)xcd_block(blockIdx.x, gridDim.x) * (2 * P);
    const FastDiv fN(N), fU(U), fH(Hx);
    // load: pencil p takes rows row0 + 2p (real part) and row0 + 2p + 1 (imaginary part)
    for (int i = threadIdx.x; i < P * N; i += blockDim.x) {
        int p = fN.div(i), n = i - p * N;
        a[p * ld + n] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    gather_tile<double>(
        2 * P * U,
        [&](int i) {
            const int rr = fU.div(i), u = i - rr * U, row = row0 + rr;
            return row < nrows ? x[(size_t)row * U + u] : 0.0;
        },
        [&](int i, double v) {
            const int rr = fU.div(i), u = i - rr * U;
            double2 *slot = &a[(rr >> 1) * ld + u];
            if (rr & 1) slot->y = v; else slot->x = v;
        });
    __syncthreads();
    lds_fft<MASK>(a, P, ld, pl, tw_s, false);
    const double2 *res = a;
    // separate: Xa[k] = (Z[k] + conj Z[N-k]) / 2, Xb[k] = (Z[k] - conj Z[N-k]) / (2i)
    for (int i = threadIdx.x; i < 2 * P * Hx; i += blockDim.x) {
        int rr = fH.div(i), k = i - rr * Hx;
        int row = row0 + rr;
        if (row >= nrows) continue;
        const double2 *Z = res + (rr >> 1) * ld;
        double2 z1 = Z[k], z2 = Z[k == 0 ? 0 : N - k];
        double2 o;
        if (rr & 1) o = make_double2(0.5 * (z1.y + z2.y), -0.5 * (z1.x - z2.x));
        else o = make_double2(0.5 * (z1.x + z2.x), 0.5 * (z1.y - z2.y));
        X[(size_t)row * Hp + k] = o;
    }
}

// Inverse: rows of Hx complex half-spectra (pitch Hp) -> rows of U reals (unnormalised).
template <int MASK>
__global__ void __launch_bounds__(kThreads) k_fft_x_inv(const double2 *__restrict__ X, double *__restrict__ y,
                                                        int nrows, int U, int Hx, int Hp, PlanArg pl, const double2 *tw,
                                                        int P)
{
    extern __shared__ double2 sm[];
    const int N = pl.N, ld = N + 1;
    double2 *tw_s = sm;
    double2 *a = sm + N;
    load_twiddles(tw_s, tw, N);
    const int row0 = (int)xcd_block(blockIdx.x, gridDim.x) * (2 * P);
    const FastDiv fN(N), fU(U);
    // Z[k] = Xa[k] + i Xb[k] for k <= N/2, Z[N-k] = conj(Xa[k]) + i conj(Xb[k]) for 0 < k < N/2
    gather_tile<double4>(
        P * N,
        [&](int i) {
            const int p = fN.div(i), n = i - p * N;
            const int ra = row0 + 2 * p, rb = ra + 1;
            const int k = n <= N / 2 ? n : N - n;
            double2 xa = make_double2(0, 0), xb = make_double2(0, 0);
            if (ra < nrows) xa = X[(size_t)ra * Hp + k];
            if (rb < nrows) xb = X[(size_t)rb * Hp + k];
            return make_double4(xa.x, xa.y, xb.x, xb.y);
        },
        [&](int i, double4 v) {
            const int p = fN.div(i), n = i - p * N;
            double2 xa = make_double2(v.x, v.y), xb = make_double2(v.z, v.w);
            if (n > N / 2) {
                xa.y = -xa.y;
                xb.y = -xb.y;
            }
            a[p * ld + n] = make_double2(xa.x - xb.y, xa.y + xb.x);
        });
    __syncthreads();
    lds_fft<MASK>(a, P, ld, pl, tw_s, true);
    const double2 *res = a;
    for (int i = threadIdx.x; i < 2 * P * U; i += blockDim.x) {
        int rr = fU.div(i), u = i - rr * U;
        int row = row0 + rr;
        if (row >= nrows) continue;
        double2 z = res[(rr >> 1) * ld + u];
        y[(size_t)row * U + u] = (rr & 1) ? z.y : z.x;
    }
}

// ---------------------------------------------------------------------------- strided pass
// Pencil groups g = (c, q), c < ncomp, q < nq.  Group g holds Hx pencils (consecutive in
// memory, index kx) with elements at stride es.  Input base c*cs_in + q*qs_in, n_in live
// elements (the rest are zero); output base c*cs_out + q*qs_out, first n_out elements stored.
struct StridedArg {
    int nq, Hx;
    long cs_in, qs_in, es_in, cs_out, qs_out, es_out;
    int n_in, n_out;
};

template <int MASK>
__global__ void __launch_bounds__(kThreads) k_fft_strided(const double2 *__restrict__ in, double2 *__restrict__ out,
                                                          StridedArg g, PlanArg pl, const double2 *tw, int P,
                                                          int inv)
{
    extern __shared__ double2 sm[];
    const int N = pl.N, ld = N + 1;
    double2 *tw_s = sm;
    double2 *a = sm + N;
    load_twiddles(tw_s, tw, N);
    const int ntile = (g.Hx + P - 1) / P;
    const int lb = (int)xcd_block(blockIdx.x, gridDim.x);   // neighbouring tiles share row ends
    const int tile = lb % ntile;
    const int grp = lb / ntile;
    const int c = grp / g.nq, q = grp - c * g.nq;
    const int kx0 = tile * P;
    const int np = min(P, g.Hx - kx0);
    const FastDiv fP(P);
    const double2 *src = in + c * g.cs_in + q * g.qs_in + kx0;
    gather_tile<double2>(
        P * N,
        [&](int i) {
            const int n = fP.div(i), p = i - n * P;
            return (n < g.n_in && p < np) ? src[(long)n * g.es_in + p] : make_double2(0.0, 0.0);
        },
        [&](int i, double2 v) {
            const int n = fP.div(i), p = i - n * P;
            a[p * ld + n] = v;
        });
    __syncthreads();
    lds_fft<MASK>(a, P, ld, pl, tw_s, inv != 0);
    const double2 *res = a;
    double2 *dst = out + c * g.cs_out + q * g.qs_out + kx0;
    for (int i = threadIdx.x; i < P * g.n_out; i += blockDim.x) {
        int n = fP.div(i), p = i - n * P;
        if (p < np) dst[(long)n * g.es_out + p] = res[p * ld + n];
    }
}


// ---------------------------------------------------------------------------- two-radix strided pass
// The strided passes of a length N = R1 R2 with both factors at most 16 keep a butterfly of 16 points a thread
// in registers and exchange once: a thread loads the R1 points j + r R2 of its pencil straight from memory,
// transforms them, leaves them in LDS at j R1 + q, and after one barrier takes the R2 points j + r R1,
// twiddles, transforms and stores j + q R1.  The stage-by-stage kernel above moves every point through LDS
// once for the load, once per stage (three or four) and once for the store, with a barrier each time, and that,
// not its arithmetic, kept it at 3 TB/s.  Neighbouring lanes hold neighbouring pencils, so every
// access of memory and LDS is a run of the pencils' values.  The inverse is the forward transform with real
// and imaginary parts traded at the load and the store.
// Per pass, before and after: 104^3 77 -> 50 us, 64^3 26.3 -> 13.3, eight right-hand sides at 64^3 149 -> 90,
// 80^3 53 -> 24, 48^3 20.3 -> 8.6, 32^3 8.1 -> 4.8 (mean of the y and z passes, both directions).

// cos(2 pi m / R), sin(2 pi m / R)
template <int R>
struct Roots;
template <>
struct Roots<6> {
    static constexpr double c[6] = {
        1.0, 0.5, -0.5, -1.0, -0.5, 0.5};
    static constexpr double s[6] = {
        0.0, 0.8660254037844386, 0.8660254037844386, 0.0, -0.8660254037844386, -0.8660254037844386};
};
template <>
struct Roots<8> {
    static constexpr double c[8] = {
        1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476, 0.0,
        0.7071067811865476};
    static constexpr double s[8] = {
        0.0, 0.7071067811865476, 1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0,
        -0.7071067811865476};
};
template <>
struct Roots<9> {
    static constexpr double c[9] = {
        1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084, -0.9396926207859084,
        -0.5, 0.17364817766693036, 0.766044443118978};
    static constexpr double s[9] = {
        0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386, 0.3420201433256687,
        -0.3420201433256687, -0.8660254037844386, -0.984807753012208, -0.6427876096865394};
};
template <>
struct Roots<10> {
    static constexpr double c[10] = {
        1.0, 0.8090169943749475, 0.30901699437494745, -0.30901699437494745, -0.8090169943749475, -1.0,
        -0.8090169943749475, -0.30901699437494745, 0.30901699437494745, 0.8090169943749475};
    static constexpr double s[10] = {
        0.0, 0.5877852522924731, 0.9510565162951535, 0.9510565162951535, 0.5877852522924731, 0.0,
        -0.5877852522924731, -0.9510565162951535, -0.9510565162951535, -0.5877852522924731};
};
template <>
struct Roots<12> {
    static constexpr double c[12] = {
        1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0, -0.8660254037844386, -0.5,
        0.0, 0.5, 0.8660254037844386};
    static constexpr double s[12] = {
        0.0, 0.5, 0.8660254037844386, 1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386,
        -1.0, -0.8660254037844386, -0.5};
};
template <>
struct Roots<14> {
    static constexpr double c[14] = {
        1.0, 0.9009688679024191, 0.6234898018587335, 0.2225209339563144, -0.2225209339563144,
        -0.6234898018587335, -0.9009688679024191, -1.0, -0.9009688679024191, -0.6234898018587335,
        -0.2225209339563144, 0.2225209339563144, 0.6234898018587335, 0.9009688679024191};
    static constexpr double s[14] = {
        0.0, 0.4338837391175581, 0.7818314824680298, 0.9749279121818236, 0.9749279121818236,
        0.7818314824680298, 0.4338837391175581, 0.0, -0.4338837391175581, -0.7818314824680298,
        -0.9749279121818236, -0.9749279121818236, -0.7818314824680298, -0.4338837391175581};
};
template <>
struct Roots<15> {
    static constexpr double c[15] = {
        1.0, 0.9135454576426009, 0.6691306063588582, 0.30901699437494745, -0.10452846326765347, -0.5,
        -0.8090169943749475, -0.9781476007338057, -0.9781476007338057, -0.8090169943749475, -0.5,
        -0.10452846326765347, 0.30901699437494745, 0.6691306063588582, 0.9135454576426009};
    static constexpr double s[15] = {
        0.0, 0.4067366430758002, 0.7431448254773942, 0.9510565162951535, 0.9945218953682733,
        0.8660254037844386, 0.5877852522924731, 0.20791169081775934, -0.20791169081775934,
        -0.5877852522924731, -0.8660254037844386, -0.9945218953682733, -0.9510565162951535,
        -0.7431448254773942, -0.4067366430758002};
};
template <>
struct Roots<16> {
    static constexpr double c[16] = {
        1.0, 0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898,
        -0.7071067811865476, -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476,
        -0.3826834323650898, 0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867};
    static constexpr double s[16] = {
        0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867, 1.0, 0.9238795325112867,
        0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898, -0.7071067811865476,
        -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476, -0.3826834323650898};
};

constexpr bool fft_prime(int R) { return R == 2 || R == 3 || R == 4 || R == 5 || R == 7 || R == 11 || R == 13; }
constexpr int fft_split(int R)   // first factor of a composite register transform
{
    return R == 6 ? 2 : R == 8 ? 2 : R == 9 ? 3 : R == 10 ? 2 : R == 12 ? 4 : R == 14 ? 2 : R == 15 ? 3 : 4;
}

// In-register forward transform of R points (2 <= R <= 16), v[q] <- sum_t v[t] W_R^{q t}
template <int R>
__device__ __attribute__((always_inline)) inline void dft_reg(double2 (&v)[R])
{
    if constexpr (fft_prime(R)) {
        dft_small<R>(v, nullptr, R, false);
    } else {
        constexpr int A = fft_split(R), B = R / A;
        double2 u[R];
#pragma unroll
        for (int b = 0; b < B; b++) {
            double2 x[A];
#pragma unroll
            for (int a = 0; a < A; a++) x[a] = v[a * B + b];
            dft_reg<A>(x);
#pragma unroll
            for (int a = 0; a < A; a++) {
                const int m = a * b % R;
                u[a * B + b] = m == 0 ? x[a] : cmul(x[a], make_double2(Roots<R>::c[m], -Roots<R>::s[m]));
            }
        }
#pragma unroll
        for (int a = 0; a < A; a++) {
            double2 x[B];
#pragma unroll
            for (int b = 0; b < B; b++) x[b] = u[a * B + b];
            dft_reg<B>(x);
#pragma unroll
            for (int b = 0; b < B; b++) v[a + A * b] = x[b];
        }
    }
}

template <int R1, int R2>
__global__ void __launch_bounds__(kThreads) k_fft2_strided(const double2 *__restrict__ in, double2 *__restrict__ out,
                                                           StridedArg g, const double2 *tw, int P, int inv)
{
    constexpr int N = R1 * R2;
    extern __shared__ double2 sm[];
    double2 *tw_s = sm, *buf = sm + N;
    load_twiddles(tw_s, tw, N);
    const int ntile = (g.Hx + P - 1) / P;
    const int lb = (int)xcd_block(blockIdx.x, gridDim.x);   // neighbouring tiles share row ends
    const int tile = lb % ntile;
    const int grp = lb / ntile;
    const int c = grp / g.nq, qi = grp - c * g.nq;
    const int kx0 = tile * P;
    const FastDiv fP(P);
    const int b = threadIdx.x, j = fP.div(b), p = b - j * P;
    const bool live = kx0 + p < g.Hx;
    if (j < R2) {
        const double2 *src = in + c * g.cs_in + qi * g.qs_in + kx0 + p;
        double2 v[R1];
#pragma unroll
        for (int r = 0; r < R1; r++) {
            const int n = j + r * R2;
            v[r] = live && n < g.n_in ? src[(long)n * g.es_in] : make_double2(0.0, 0.0);
        }
        if (inv)
#pragma unroll
            for (int r = 0; r < R1; r++) v[r] = make_double2(v[r].y, v[r].x);
        dft_reg<R1>(v);
#pragma unroll
        for (int q = 0; q < R1; q++) buf[(j * R1 + q) * P + p] = v[q];
    }
    __syncthreads();
    if (j < R1) {
        double2 v[R2];
#pragma unroll
        for (int r = 0; r < R2; r++) v[r] = buf[b + r * (R1 * P)];   // point j + r R1
#pragma unroll
        for (int r = 1; r < R2; r++) v[r] = cmul(v[r], tw_s[j * r]);
        dft_reg<R2>(v);
        if (inv)
#pragma unroll
            for (int r = 0; r < R2; r++) v[r] = make_double2(v[r].y, v[r].x);
        double2 *dst = out + c * g.cs_out + qi * g.qs_out + kx0 + p;
#pragma unroll
        for (int q = 0; q < R2; q++) {
            const int n = j + q * R1;
            if (live && n < g.n_out) dst[(long)n * g.es_out] = v[q];
        }
    }
}

// The x passes in the same way, two real rows a pencil.  Neighbouring lanes hold neighbouring points of a
// row (runs of R2 reals at the load, of R1 at the inverse's store); in LDS a pencil's rows of R1 points are
// one value longer when R1 is even, so that the lanes' writes, R1 values apart, spread over the banks.
template <int R1, int R2>
struct XTile {
    static constexpr int N = R1 * R2, row = R1 + (R1 % 2 == 0 ? 1 : 0), ld = R2 * row;
};

template <int R1, int R2>
__global__ void __launch_bounds__(kThreads) k_fft2_x_fwd(const double *__restrict__ x, double2 *__restrict__ X,
                                                         int nrows, int U, int Hx, int Hp, const double2 *tw, int P)
{
    using T = XTile<R1, R2>;
    constexpr int N = T::N;
    extern __shared__ double2 sm[];
    double2 *tw_s = sm, *buf = sm + N;
    load_twiddles(tw_s, tw, N);
    const int row0 = (int)xcd_block(blockIdx.x, gridDim.x) * (2 * P);
    const int b = threadIdx.x;
    {
        const int p = b / R2, j = b % R2, ra = row0 + 2 * p;
        if (p < P) {
            const double *xa = x + (size_t)ra * U, *xb = xa + U;
            double2 v[R1];
#pragma unroll
            for (int r = 0; r < R1; r++) {
                const int n = j + r * R2;
                v[r] = make_double2(n < U && ra < nrows ? xa[n] : 0.0, n < U && ra + 1 < nrows ? xb[n] : 0.0);
            }
            dft_reg<R1>(v);
#pragma unroll
            for (int q = 0; q < R1; q++) buf[p * T::ld + j * T::row + q] = v[q];
        }
    }
    __syncthreads();
    const int p = b / R1, j = b % R1;
    double2 v[R2];
    if (p < P) {
#pragma unroll
        for (int r = 0; r < R2; r++) v[r] = buf[p * T::ld + r * T::row + j];   // point j + r R1
#pragma unroll
        for (int r = 1; r < R2; r++) v[r] = cmul(v[r], tw_s[j * r]);
        dft_reg<R2>(v);
    }
    __syncthreads();
    if (p < P)
#pragma unroll
        for (int q = 0; q < R2; q++) buf[p * T::ld + j + q * R1] = v[q];
    __syncthreads();
    // separate: Xa[k] = (Z[k] + conj Z[N-k]) / 2, Xb[k] = (Z[k] - conj Z[N-k]) / (2i)
    const FastDiv fH(Hx);
    for (int i = threadIdx.x; i < 2 * P * Hx; i += blockDim.x) {
        const int rr = fH.div(i), k = i - rr * Hx, row = row0 + rr;
        if (row >= nrows) continue;
        const double2 *Z = buf + (rr >> 1) * T::ld;
        const double2 z1 = Z[k], z2 = Z[k == 0 ? 0 : N - k];
        X[(size_t)row * Hp + k] = (rr & 1) ? make_double2(0.5 * (z1.y + z2.y), -0.5 * (z1.x - z2.x))
                                           : make_double2(0.5 * (z1.x + z2.x), 0.5 * (z1.y - z2.y));
    }
}

template <int R1, int R2>
__global__ void __launch_bounds__(kThreads) k_fft2_x_inv(const double2 *__restrict__ X, double *__restrict__ y,
                                                         int nrows, int U, int Hx, int Hp, const double2 *tw, int P)
{
    using T = XTile<R1, R2>;
    constexpr int N = T::N;
    extern __shared__ double2 sm[];
    double2 *tw_s = sm, *buf = sm + N;
    load_twiddles(tw_s, tw, N);
    const int row0 = (int)xcd_block(blockIdx.x, gridDim.x) * (2 * P);
    const int b = threadIdx.x;
    {
        const int p = b / R2, j = b % R2, ra = row0 + 2 * p;
        if (p < P) {
            const double2 *Xa = X + (size_t)ra * Hp, *Xb = Xa + Hp;
            double2 v[R1];
            // Z[k] = Xa[k] + i Xb[k] for k <= N/2, Z[N-k] = conj(Xa[k]) + i conj(Xb[k]) for 0 < k < N/2, with
            // real and imaginary parts traded
#pragma unroll
            for (int r = 0; r < R1; r++) {
                const int n = j + r * R2, k = n <= N / 2 ? n : N - n;
                const double2 xa = ra < nrows ? Xa[k] : make_double2(0.0, 0.0);
                const double2 xb = ra + 1 < nrows ? Xb[k] : make_double2(0.0, 0.0);
                const double sg = n <= N / 2 ? 1.0 : -1.0;
                v[r] = make_double2(fma(sg, xa.y, xb.x), fma(-sg, xb.y, xa.x));
            }
            dft_reg<R1>(v);
#pragma unroll
            for (int q = 0; q < R1; q++) buf[p * T::ld + j * T::row + q] = v[q];
        }
    }
    __syncthreads();
    const int p = b / R1, j = b % R1, ra = row0 + 2 * p;
    if (p < P) {
        double2 v[R2];
#pragma unroll
        for (int r = 0; r < R2; r++) v[r] = buf[p * T::ld + r * T::row + j];
#pragma unroll
        for (int r = 1; r < R2; r++) v[r] = cmul(v[r], tw_s[j * r]);
        dft_reg<R2>(v);
        double *ya = y + (size_t)ra * U, *yb = ya + U;
#pragma unroll
        for (int q = 0; q < R2; q++) {
            const int n = j + q * R1;
            if (n < U && ra < nrows) ya[n] = v[q].y;
            if (n < U && ra + 1 < nrows) yb[n] = v[q].x;
        }
    }
}

// The lengths with a two-radix pass: every even product of 2, 3, 5, 7, 11 and 13 from 8 to 256 that
// splits so, with the factors as near each other as they go, the larger one first.  (Also the shortest ones,
// where a pass has little to do: 18 and 26 points, strided, 9.3 us a pass with a stage per radix.)
#define MJ_FFT2_SIZES(X) \
    X(8, 4, 2) X(10, 5, 2) X(12, 4, 3) X(14, 7, 2) X(16, 4, 4) X(18, 6, 3) X(20, 5, 4) X(22, 11, 2) \
    X(24, 6, 4) X(26, 13, 2) X(28, 7, 4) X(30, 6, 5) \
    X(32, 8, 4) X(36, 6, 6) X(40, 8, 5) X(42, 7, 6) X(44, 11, 4) X(48, 8, 6) X(50, 10, 5) \
    X(52, 13, 4) X(54, 9, 6) X(56, 8, 7) X(60, 10, 6) X(64, 8, 8) X(66, 11, 6) X(70, 10, 7) \
    X(72, 9, 8) X(78, 13, 6) X(80, 10, 8) X(84, 12, 7) X(88, 11, 8) X(90, 10, 9) X(96, 12, 8) \
    X(98, 14, 7) X(100, 10, 10) X(104, 13, 8) X(108, 12, 9) X(110, 11, 10) X(112, 14, 8) X(120, 12, 10) \
    X(126, 14, 9) X(128, 16, 8) X(130, 13, 10) X(132, 12, 11) X(140, 14, 10) X(144, 12, 12) X(150, 15, 10) \
    X(154, 14, 11) X(156, 13, 12) X(160, 16, 10) X(168, 14, 12) X(176, 16, 11) X(180, 15, 12) X(182, 14, 13) \
    X(192, 16, 12) X(196, 14, 14) X(208, 16, 13) X(210, 15, 14) X(224, 16, 14) X(240, 16, 15) X(256, 16, 16)

PlanArg plan_arg(const FftPlan1D &p)
{
    PlanArg a{};
    a.N = p.N;
    a.nst = p.nst;
    for (int i = 0; i < p.nst; i++) a.radix[i] = p.radix[i];
    return a;
}

int pencils_per_block(int N) { return std::max(1, std::min(16, kTileElems / N)); }

size_t lds_bytes(int N, int P) { return sizeof(double2) * (size_t)(N + P * (N + 1)); }

// Radices of the stages, in order.  The first stage (Ns = 1) writes its R outputs with a stride
// of R complex values in LDS, so an odd radix goes first: a stride of 13 x 16 bytes spreads the
// lanes over every bank, where a stride of 4 x 16 bytes puts four lanes on each bank group.
// Later stages write runs of Ns consecutive values.  Then radix 4 as often as possible, and 2.
bool factor(int N, std::vector<int> &out)
{
    out.clear();
    int n = N;
    for (int r : {13, 11, 7, 5, 3})
        while (n % r == 0) { out.push_back(r); n /= r; }
    while (n % 4 == 0) { out.push_back(4); n /= 4; }
    while (n % 2 == 0) { out.push_back(2); n /= 2; }
    return n == 1 && (int)out.size() <= kMaxStages;
}

}  // namespace

bool fft_size_ok(int N)
{
    std::vector<int> f;
    return N >= 2 && N <= kMaxFftN && N % 2 == 0 && factor(N, f);
}

int fft_pick_size(int nmin)
{
    for (int N = nmin; N <= kMaxFftN; N++)
        if (fft_size_ok(N)) return N;
    throw ArgError("grid too large for the FFT (padded size above " + std::to_string(kMaxFftN) + ")");
}

void fft_plan_init(FftPlan1D &p, int N, const DevAlloc &da)
{
    std::vector<int> f;
    if (!fft_size_ok(N) || !factor(N, f)) throw ArgError("unsupported FFT size " + std::to_string(N));
    p.N = N;
    p.nst = (int)f.size();
    for (int i = 0; i < p.nst; i++) p.radix[i] = f[i];
    std::vector<double2> h(N);
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int m = 0; m < N; m++) {
        long double ang = -2.0L * pi * (long double)m / (long double)N;
        h[m] = make_double2((double)cosl(ang), (double)sinl(ang));
    }
    p.tw = (double2 *)da.get(sizeof(double2) * N, "FFT twiddles");
    MJ_CHECK(hipMemcpy(p.tw, h.data(), sizeof(double2) * N, hipMemcpyHostToDevice));
    // the odd-radix constants, rounded the same way (cheap; repeated for every plan so that
    // the device current at plan creation has them)
    double cs[2 * (1 + 2 + 3 + 5 + 6)];
    for (int R : {3, 5, 7, 11, 13})
        for (int m = 1; m <= (R - 1) / 2; m++) {
            long double ang = 2.0L * pi * (long double)m / (long double)R;
            cs[odd_base(R) + 2 * (m - 1)] = (double)cosl(ang);
            cs[odd_base(R) + 2 * (m - 1) + 1] = (double)sinl(ang);
        }
    MJ_CHECK(hipMemcpyToSymbol(HIP_SYMBOL(c_odd_cs), cs, sizeof(cs)));
}

void fft_plan_free(FftPlan1D &p, const DevAlloc &da)
{
    da.put(p.tw);
    p.tw = nullptr;
}

void fft3d_init(Fft3D &f, int U, int V, int W, int ncomp, int Nx, int Ny, int Nz, const DevAlloc &da)
{
    f.da = da;
    f.U = U; f.V = V; f.W = W;
    f.Nx = Nx; f.Ny = Ny; f.Nz = Nz;
    f.Hx = Nx / 2 + 1;
    f.Hp = spectrum_pitch(f.Hx);
    f.ncomp = ncomp;
    fft_plan_init(f.px, Nx, da);
    fft_plan_init(f.py, Ny, da);
    fft_plan_init(f.pz, Nz, da);
    fft3d_set_pencils(f, 1 << 30);
    size_t na = (size_t)ncomp * W * V * f.Hp, nb = (size_t)ncomp * W * Ny * f.Hp;
    f.bufA = (double2 *)da.get(sizeof(double2) * na, "FFT scratch A");
    f.bufB = (double2 *)da.get(sizeof(double2) * nb, "FFT scratch B");
}

void fft3d_free(Fft3D &f)
{
    fft_plan_free(f.px, f.da);
    fft_plan_free(f.py, f.da);
    fft_plan_free(f.pz, f.da);
    f.da.put(f.bufA);
    f.da.put(f.bufB);
    f.bufA = f.bufB = nullptr;
}

// Radix set of a plan, and the stage-by-stage kernel instance that serves it where no two-radix pass does
// (lengths 2 to 6 and above 256, and those that are no product of two radices of at most 16): powers of two and 3 2^k
// have their own instances, any other plan the generic one.
static int plan_mask(const FftPlan1D &p)
{
    int m = 0;
    for (int i = 0; i < p.nst; i++) {
        switch (p.radix[i]) {
        case 2: m |= kR2; break;
        case 3: m |= kR3; break;
        case 4: m |= kR4; break;
        case 5: m |= kR5; break;
        case 7: m |= kR7; break;
        case 11: m |= kR11; break;
        default: m |= kR13; break;
        }
    }
    return m;
}

#define MJ_FFT_DISPATCH(mask, KERNEL, ...)                                                        \
    do {                                                                                          \
        switch (mask) {                                                                           \
        case kR4: hipLaunchKernelGGL(KERNEL<kR4>, __VA_ARGS__); break;                            \
        case kR2 | kR4: hipLaunchKernelGGL(KERNEL<kR2 | kR4>, __VA_ARGS__); break;                \
        case kR3 | kR4: hipLaunchKernelGGL(KERNEL<kR3 | kR4>, __VA_ARGS__); break;                \
        case kR2 | kR3 | kR4: hipLaunchKernelGGL(KERNEL<kR2 | kR3 | kR4>, __VA_ARGS__); break;    \
        default: hipLaunchKernelGGL(KERNEL<kAll>, __VA_ARGS__); break;                            \
        }                                                                                         \
    } while (0)

// threads of a two-radix pass: P pencils (P <= 16) of at most 16 butterflies, in whole waves
static dim3 two_radix_threads(int P, int R1, int R2) { return dim3((unsigned)((P * std::max(R1, R2) + 63) / 64 * 64)); }

static void launch_strided(const double2 *in, double2 *out, const StridedArg &g, int ncomp, const FftPlan1D &p,
                           int P, bool inv, hipStream_t st)
{
    int ntile = (g.Hx + P - 1) / P;
    dim3 grid(ncomp * g.nq * ntile);
    const size_t lds2 = sizeof(double2) * (size_t)p.N * (P + 1);
    switch (p.N) {
#define X(N, R1, R2)                                                                                          \
    case N:                                                                                                   \
        hipLaunchKernelGGL((k_fft2_strided<R1, R2>), grid, two_radix_threads(P, R1, R2), lds2, st, in, out, g, \
                           p.tw, P, inv ? 1 : 0);                                                             \
        MJ_CHECK(hipGetLastError());                                                                          \
        return;
        MJ_FFT2_SIZES(X)
#undef X
    default: break;
    }
    MJ_FFT_DISPATCH(plan_mask(p), k_fft_strided, grid, dim3(kThreads), lds_bytes(p.N, P), st, in, out, g,
                    plan_arg(p), p.tw, P, inv ? 1 : 0);
    MJ_CHECK(hipGetLastError());
}

// The six passes; P is the number of pencils per block of the pass (x: 2P real rows).
// x pass forward: rows (c, w, v) of U reals -> A[c][w][v][kx]
static void pass_x_fwd(const Fft3D &f, int ncomp, const double *x, int P, hipStream_t st)
{
    const int nrows = ncomp * f.W * f.V;
    dim3 grid((nrows + 2 * P - 1) / (2 * P));
    switch (f.Nx) {
#define X(N, R1, R2)                                                                                          \
    case N:                                                                                                   \
        hipLaunchKernelGGL((k_fft2_x_fwd<R1, R2>), grid, two_radix_threads(P, R1, R2),                        \
                           sizeof(double2) * (N + P * XTile<R1, R2>::ld), st, x, f.bufA, nrows, f.U, f.Hx,     \
                           f.Hp, f.px.tw, P);                                                                 \
        MJ_CHECK(hipGetLastError());                                                                          \
        return;
        MJ_FFT2_SIZES(X)
#undef X
    default: break;
    }
    MJ_FFT_DISPATCH(plan_mask(f.px), k_fft_x_fwd, grid, dim3(kThreads), lds_bytes(f.Nx, P), st, x, f.bufA, nrows,
                    f.U, f.Hx, f.Hp, plan_arg(f.px), f.px.tw, P);
    MJ_CHECK(hipGetLastError());
}
// y pass forward: groups (c, w); A[c][w][v][kx] -> B[c][w][ky][kx]
static void pass_y_fwd(const Fft3D &f, int ncomp, int P, hipStream_t st)
{
    StridedArg g{};
    g.nq = f.W; g.Hx = f.Hx;
    g.cs_in = (long)f.W * f.V * f.Hp; g.qs_in = (long)f.V * f.Hp; g.es_in = f.Hp;
    g.cs_out = (long)f.W * f.Ny * f.Hp; g.qs_out = (long)f.Ny * f.Hp; g.es_out = f.Hp;
    g.n_in = f.V; g.n_out = f.Ny;
    launch_strided(f.bufA, f.bufB, g, ncomp, f.py, P, false, st);
}
// z pass forward: groups (c, ky); B[c][w][ky][kx] -> X[c][kz][ky][kx]
static void pass_z_fwd(const Fft3D &f, int ncomp, double2 *X, int P, hipStream_t st)
{
    StridedArg g{};
    g.nq = f.Ny; g.Hx = f.Hx;
    g.cs_in = (long)f.W * f.Ny * f.Hp; g.qs_in = f.Hp; g.es_in = (long)f.Ny * f.Hp;
    g.cs_out = (long)f.Nz * f.Ny * f.Hp; g.qs_out = f.Hp; g.es_out = (long)f.Ny * f.Hp;
    g.n_in = f.W; g.n_out = f.Nz;
    launch_strided(f.bufB, X, g, ncomp, f.pz, P, false, st);
}
// z pass inverse: X[c][kz][ky][kx] -> B[c][w][ky][kx], w < W
static void pass_z_inv(const Fft3D &f, int ncomp, const double2 *X, int P, hipStream_t st)
{
    StridedArg g{};
    g.nq = f.Ny; g.Hx = f.Hx;
    g.cs_in = (long)f.Nz * f.Ny * f.Hp; g.qs_in = f.Hp; g.es_in = (long)f.Ny * f.Hp;
    g.cs_out = (long)f.W * f.Ny * f.Hp; g.qs_out = f.Hp; g.es_out = (long)f.Ny * f.Hp;
    g.n_in = f.Nz; g.n_out = f.W;
    launch_strided(X, f.bufB, g, ncomp, f.pz, P, true, st);
}
// y pass inverse: B[c][w][ky][kx] -> A[c][w][v][kx], v < V
static void pass_y_inv(const Fft3D &f, int ncomp, int P, hipStream_t st)
{
    StridedArg g{};
    g.nq = f.W; g.Hx = f.Hx;
    g.cs_in = (long)f.W * f.Ny * f.Hp; g.qs_in = (long)f.Ny * f.Hp; g.es_in = f.Hp;
    g.cs_out = (long)f.W * f.V * f.Hp; g.qs_out = (long)f.V * f.Hp; g.es_out = f.Hp;
    g.n_in = f.Ny; g.n_out = f.V;
    launch_strided(f.bufB, f.bufA, g, ncomp, f.py, P, true, st);
}
// x pass inverse: rows (c, w, v) of Hx -> U reals
static void pass_x_inv(const Fft3D &f, int ncomp, double *y, int P, hipStream_t st)
{
    const int nrows = ncomp * f.W * f.V;
    dim3 grid((nrows + 2 * P - 1) / (2 * P));
    switch (f.Nx) {
#define X(N, R1, R2)                                                                                          \
    case N:                                                                                                   \
        hipLaunchKernelGGL((k_fft2_x_inv<R1, R2>), grid, two_radix_threads(P, R1, R2),                        \
                           sizeof(double2) * (N + P * XTile<R1, R2>::ld), st, f.bufA, y, nrows, f.U, f.Hx,     \
                           f.Hp, f.px.tw, P);                                                                 \
        MJ_CHECK(hipGetLastError());                                                                          \
        return;
        MJ_FFT2_SIZES(X)
#undef X
    default: break;
    }
    MJ_FFT_DISPATCH(plan_mask(f.px), k_fft_x_inv, grid, dim3(kThreads), lds_bytes(f.Nx, P), st, f.bufA, y, nrows,
                    f.U, f.Hx, f.Hp, plan_arg(f.px), f.px.tw, P);
    MJ_CHECK(hipGetLastError());
}

// ncomp <= the plan's ncomp (the scratch buffers are sized for that)
void fft3d_forward(Fft3D &f, const double *x, double2 *X, int ncomp, hipStream_t st)
{
    if (ncomp < 1 || ncomp > f.ncomp) throw std::logic_error("FFT batch larger than its plan");
    pass_x_fwd(f, ncomp, x, f.Px, st);
    pass_y_fwd(f, ncomp, f.Py, st);
    pass_z_fwd(f, ncomp, X, f.Pz, st);
}

void fft3d_inverse(Fft3D &f, const double2 *X, double *y, int ncomp, hipStream_t st)
{
    if (ncomp < 1 || ncomp > f.ncomp) throw std::logic_error("FFT batch larger than its plan");
    pass_z_inv(f, ncomp, X, f.Pz, st);
    pass_y_inv(f, ncomp, f.Py, st);
    pass_x_inv(f, ncomp, y, f.Px, st);
}

void fft3d_set_pencils(Fft3D &f, int cap)
{
    f.Px = std::max(1, std::min(cap, pencils_per_block(f.Nx)));
    f.Py = std::max(1, std::min(cap, pencils_per_block(f.Ny)));
    f.Pz = std::max(1, std::min(cap, pencils_per_block(f.Nz)));
}

// Picks the pencils per block of each axis pass by timing it.  A pencil's arithmetic does not
// depend on how many pencils share its block, so every choice gives bit-identical transforms;
// only the speed differs (row runs of the strided passes, blocks per compute unit).
// Candidates: the most a tile holds, and 3/4, 1/2 and 1/4 of that; each pass forward and
// inverse, best of three after one warm-up.
void fft3d_autotune(Fft3D &f, hipStream_t st)
{
    const size_t nX = (size_t)f.ncomp * f.Nz * f.Ny * f.Hp;
    double2 *X = (double2 *)f.da.get(sizeof(double2) * nX, "FFT autotune scratch");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    try {
        const size_t na = (size_t)f.ncomp * f.W * f.V * f.Hp, nb = (size_t)f.ncomp * f.W * f.Ny * f.Hp;
        MJ_CHECK(hipMemsetAsync(X, 0, sizeof(double2) * nX, st));
        MJ_CHECK(hipMemsetAsync(f.bufA, 0, sizeof(double2) * na, st));
        MJ_CHECK(hipMemsetAsync(f.bufB, 0, sizeof(double2) * nb, st));
        MJ_CHECK(hipEventCreate(&e0));
        MJ_CHECK(hipEventCreate(&e1));
        // bufB holds at least ncomp W V U reals: real input and output of the x pass
        double *xr = (double *)f.bufB;
        auto run = [&](int axis, int P) {
            if (axis == 0) {
                pass_x_fwd(f, f.ncomp, xr, P, st);
                pass_x_inv(f, f.ncomp, xr, P, st);
            } else if (axis == 1) {
                pass_y_fwd(f, f.ncomp, P, st);
                pass_y_inv(f, f.ncomp, P, st);
            } else {
                pass_z_fwd(f, f.ncomp, X, P, st);
                pass_z_inv(f, f.ncomp, X, P, st);
            }
        };
        const int Ns[3] = {f.Nx, f.Ny, f.Nz};
        int *Ps[3] = {&f.Px, &f.Py, &f.Pz};
        for (int axis = 0; axis < 3; axis++) {
            const int pmax = pencils_per_block(Ns[axis]);
            int cand[4] = {pmax, (3 * pmax) / 4, pmax / 2, pmax / 4};
            float best = 0.0f;
            int bestP = pmax;
            for (int ci = 0; ci < 4; ci++) {
                const int P = cand[ci];
                if (P < 1 || (ci > 0 && std::find(cand, cand + ci, P) != cand + ci)) continue;
                run(axis, P);
                float tmin = 0.0f;
                for (int rep = 0; rep < 3; rep++) {
                    MJ_CHECK(hipEventRecord(e0, st));
                    run(axis, P);
                    MJ_CHECK(hipEventRecord(e1, st));
                    MJ_CHECK(hipEventSynchronize(e1));
                    float ms = 0.0f;
                    MJ_CHECK(hipEventElapsedTime(&ms, e0, e1));
                    if (rep == 0 || ms < tmin) tmin = ms;
                }
                if (ci == 0 || tmin < best) {
                    best = tmin;
                    bestP = P;
                }
            }
            *Ps[axis] = bestP;
        }
    } catch (...) {
        (void)hipStreamSynchronize(st);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        f.da.put(X);
        throw;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    f.da.put(X);
}

}  // namespace mj
