// Space-time interaction kernels of the MOT-JVIE on the device (FP64).
//
// For test voxel m, source voxel m', lag k = n - n' and D = r_m - r_m' (lengths in units of
// the x edge: voxel edges h = (1, hy, hz), c dt = r <= min h), eq:Z with the
// piecewise-constant spatial basis (eq:SpatialBasis),
// the voxel-average Dirac-in-time test (eq:TestOperator) and the quadratic-spline
// temporal basis T(t) = B(t/dt + 1) (B the uniform quadratic B-spline on [0,3]) gives
//
//   Z^{ba}_k(m, m') = d_ab d_mm' T(k dt) / eps_m - chi_m K^{ba}_k(D),
//   K^{ba}_k(D) = Int g_k(d) d_a d_b Lam(d - D) dd - d_ab Int gbar_k(d) Lam(d - D) dd,
//   g_k = B(k + 1 - |d|/r) / (4 pi |d|),  gbar_k = B''(k + 1 - |d|/r) / (4 pi r^2 |d|),
//   Lam(x) = prod_i (1 - |x_i| / h_i)_+ ,
//
// the derivatives of Lam taken in the distributional sense (a == b gives the second
// difference across the planes d_a = D_a - h_a, D_a, D_a + h_a, divided by h_a).
//
// Factorisation used here.  On the shell a r <= |d| < (a + 1) r each B-spline piece is
// a quadratic in v = |d|/r - a, so every lag is a fixed combination of the lag-free
// shell moments
//   plane_a,j : sum_s w_s Int_{plane s, shell} lam lam v^j / |d| dS    (a = x, y, z; j = 0..2)
//   cube_ab,j : Int_{shell} d_a d_b Lam v^j / |d| dV                    (ab = xy, xz, yz)
//   gbar      : Int_{shell} Lam / |d| dV
// of the three shells a = k, k - 1, k - 2 (K_k = 0 unless one of them meets the
// distance range of the voxel pair: the causal / Huygens support).
//
// Quadrature.  A volume moment over a sub-box (where Lam and its derivatives are
// polynomials) is turned into face integrals by the divergence theorem with the radial
// field y Psi(y) / |y|^3, Psi(y) = Int_{a r}^{min(|y|, (a+1) r)} P(u yhat) v^j u du (div = P v^j/|y|
// on the shell); Psi is a polynomial in u of degree <= 4 and is integrated exactly by
// 3-point Gauss-Legendre.  Every face or plane integral is taken over a unit square as
// four signed triangles with apex at the foot of the perpendicular from the origin,
// parametrised by (s along the edge, tau along the ray), split where the shell's two
// spheres cut the plane and graded towards the foot where the integrand does not vanish
// there; nq x nq Gauss-Legendre on every cell.  Only the octant D >= 0 is computed; the
// other octants follow from the parity of each component, and along axes of equal voxel edges only one
// order of |D_x|, |D_y|, |D_z| is, the others being its permutations (a cubic grid computes one
// offset in six).
//
// A foot that lies outside the square by two of its edges or more starts the rays at its distance from
// the square instead of 0: what lies inside cancels between the four triangles.  That leaves only short
// cells away from the foot, where few points do (see order_class, and grazed for the exception).
//
// One wave takes one offset.  It is bound by FP64 work, about 250 operations a node, so the edges of the
// squares are cut first, a lane each, and the intervals that contribute go into a list in LDS whose s-nodes
// the lanes then share evenly (lanes bound to an interval slot of a square idled for most of them).
// Together: 48^3 grid kernels 12.2 ms (428 ms with 16 x 16 points everywhere, all offsets and bound
// lanes); 82 944 off-grid pairs of a 24^3 block 36 ms (318 ms), where only the orders, the start of the
// rays and the list can help.

#include "mj_internal.h"

#include <cmath>

namespace mj {

namespace {

constexpr int kGenThreads = 64;
constexpr int kMaxQ = 24;
constexpr double kInvFourPi = 0.07957747154594766788;

// Points per cell (along an edge, along a ray) by the gap between the two voxels in units of the longest
// edge.  With quad_order 0 the orders fall where the integrands get smoother.  They were chosen
// on the CPU in extended precision against 20 x 20 points, over every sorted offset up to 12, 1500
// log-uniform real offsets out to 80 and 400 with edges 1 x 0.7 x 1.3: in the distance classes the cells'
// error stays below 1e-14 of the largest |K_k| of its offset, where rounding alone leaves 1e-14 to
// 1e-13 with 16 points and, having fewer nodes to add, not more with these.  Where a sphere cuts a plane in a
// circle smaller than the voxels they are 16 again (see grazed), and 16 points have their own limit there: 3e-7
// of the kernel at D = (1.096, 34.9998, 0.5048) with edges 1 x 0.6 x 1.4 and c dt = 0.6, a circle of 0.07.
constexpr int kOrderClasses = 5;
constexpr double kClassGap[kOrderClasses] = {0.0, 3.5, 6.0, 12.0, 24.0};
constexpr int kClassS[kOrderClasses] = {16, 14, 12, 11, 10}, kClassT[kOrderClasses] = {16, 12, 11, 9, 8};

// The Gauss-Legendre rules in use: those of the classes, or the caller's order in every class.
struct GenRules {
    int ns[kOrderClasses], nt[kOrderClasses];      // points
    int rs[kOrderClasses], rt[kOrderClasses];      // rows of x, w
    double x[2 * kOrderClasses][kMaxQ], w[2 * kOrderClasses][kMaxQ];   // on [-1, 1]
    double g3x[3], g3w[3];                         // 3-point rule on [-1, 1]
};

struct GenArg {
    int Uo, Vo, Wo;
    int nq;
    int ms;                          // shells stored per offset
    double r;                        // c dt
    double hv[3], ih[3];             // voxel edges and their inverses
    double glx[kMaxQ], glw[kMaxQ];   // nq-point rule on [-1, 1] (host checks)
    double g3x[3], g3w[3];           // 3-point rule on [-1, 1]
    const GenRules *rules;           // on the device
};

// Order class of the offset |D| (voxel steps, real): see above.
__host__ __device__ inline int order_class(double dx, double dy, double dz, const double hv[3])
{
    const double d[3] = {dx, dy, dz};
    double g2 = 0.0, hm = 0.0;
    for (int i = 0; i < 3; i++) {
        const double e = d[i] > 1.0 ? (d[i] - 1.0) * hv[i] : 0.0;
        g2 += e * e;
        hm = hv[i] > hm ? hv[i] : hm;
    }
    int c = 0;
    for (int i = 1; i < kOrderClasses; i++) c = g2 >= kClassGap[i] * kClassGap[i] * hm * hm ? i : c;
    return c;
}

// Whether a sphere of shell [Ra, Rb) cuts a plane of the offset D (lengths) in a circle about as small as the
// voxels, next to the squares in that plane.  The rays to an edge then start or end at rho / L, where L, the
// distance to the foot, bends over an edge that is nearer than its own length, and the few points of a far
// offset do not follow: at D = (13.6, 1.04, 0.29) with edges 1 x 0.7 x 1.3 and r = 0.7, where the sphere 18 r
// = 12.6 cuts the plane 12.5958 in a circle of 0.33, 11 points a side gave 3e-8 of the kernel where 16 give
// 2e-10.  Such a shell takes the points of voxels in contact, whatever its distance.  From 1.5 edges away the
// bend's nearest singularity leaves 10 points below 1e-15; circles of 3 edges and more pass the squares that
// are nearer than that.
__host__ __device__ inline bool grazed(const double D[3], double Ra, double Rb, const double hv[3])
{
    const double hm = fmax(hv[0], fmax(hv[1], hv[2])), rho2 = 9.0 * hm * hm;
    bool g = false;
    for (int ax = 0; ax < 3; ax++) {
        const int b1 = (ax + 1) % 3, b2 = (ax + 2) % 3;
        const double n1 = fmax(0.0, fabs(D[b1]) - hv[b1]), n2 = fmax(0.0, fabs(D[b2]) - hv[b2]);
        if (n1 * n1 + n2 * n2 >= 2.25 * hm * hm) continue;
        for (int t = -1; t <= 1; t++) {
            const double c = D[ax] + t * hv[ax], a2 = Ra * Ra - c * c, b2_ = Rb * Rb - c * c;
            g = g || (a2 > 0.0 && a2 < rho2) || (b2_ > 0.0 && b2_ < rho2);
        }
    }
    return g;
}

// Shells a r <= |d| < (a + 1) r, a in [a_lo, a_lo + nsh), that meet the distance range
// [R_min, R_max] of two voxels: a_lo = floor(R_min / r), a_lo + nsh = ceil(R_max / r).  With
// r = 1 the squared radii are integers and the bounds are exact.
__host__ __device__ inline void shell_bounds(double rmin2, double rmax2, double r, int &a_lo, int &nsh)
{
    const double Rmin = sqrt(rmin2), Rmax = sqrt(rmax2);
    int lo = (int)floor(Rmin / r);
    while ((lo + 1) * r <= Rmin) lo++;
    while (lo > 0 && lo * r > Rmin) lo--;
    int hi = (int)ceil(Rmax / r);
    while (hi - 1 > lo && (hi - 1) * r >= Rmax) hi--;
    while (hi * r < Rmax) hi++;
    a_lo = lo;
    nsh = hi - lo;
}

__host__ __device__ inline void shell_range(int dx, int dy, int dz, const double hv[3], double r, int &a_lo,
                                            int &nsh)
{
    const int ex = dx > 0 ? dx - 1 : 0, ey = dy > 0 ? dy - 1 : 0, ez = dz > 0 ? dz - 1 : 0;
    const double rmin2 = (ex * hv[0]) * (ex * hv[0]) + (ey * hv[1]) * (ey * hv[1]) + (ez * hv[2]) * (ez * hv[2]);
    const double rmax2 = ((dx + 1) * hv[0]) * ((dx + 1) * hv[0]) + ((dy + 1) * hv[1]) * ((dy + 1) * hv[1]) +
                         ((dz + 1) * hv[2]) * ((dz + 1) * hv[2]);
    shell_bounds(rmin2, rmax2, r, a_lo, nsh);
}

// Upper bound on the shells of one voxel pair: R_max - R_min <= 2 |h|, plus one shell cut at
// each end and one for rounding.
__host__ __device__ inline int shells_per_offset(double r, const double hv[3])
{
    return (int)(2.0 * sqrt(hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2]) / r) + 3;
}

// Fixed-size ascending sort with compile-time indices only (values stay in registers).
template <int N>
__host__ __device__ inline void sort_fixed(double *a)
{
#pragma unroll
    for (int i = 0; i < N - 1; i++)
#pragma unroll
        for (int j = 0; j < N - 1 - i; j++) {
            double lo = fmin(a[j], a[j + 1]), hi = fmax(a[j], a[j + 1]);
            a[j] = lo;
            a[j + 1] = hi;
        }
}

// Contribution of one face node y (weight wgt = dA * quadrature weight) on the square of
// plane y_AX = c = D[AX] + s h_AX with sub-square signs (s1, s2) along the in-plane axes.
// Every array index is a compile-time constant.
// ANI = false compiles the cubic-voxel case, where every edge factor is 1.
template <int AX, bool ANI>
__host__ __device__ inline void node_contrib(double m[kMoments], const double y[3], double ny, double wgt, int s,
                                             int s1, int s2, const double D[3], double Ra, double Rb, double inv_r,
                                             const double *ih, const double *g3x, const double *g3w)
{
    constexpr int A1 = (AX + 1) % 3, A2 = (AX + 2) % 3;
    const double c = y[AX];
    const double inv_ny = 1.0 / ny;
    // plane term of component AX: w_s lam lam v^j / |y| on the shell
    if (ny >= Ra && ny < Rb) {
        const double ws = ANI ? ((s == 0) ? -2.0 : 1.0) * ih[AX] : ((s == 0) ? -2.0 : 1.0);
        const double l1 = ANI ? 1.0 - s1 * (y[A1] - D[A1]) * ih[A1] : 1.0 - s1 * (y[A1] - D[A1]);
        const double l2 = ANI ? 1.0 - s2 * (y[A2] - D[A2]) * ih[A2] : 1.0 - s2 * (y[A2] - D[A2]);
        const double v = (ny - Ra) * inv_r;
        const double f = wgt * ws * l1 * l2 * inv_ny;
        m[3 * AX + 0] += f;
        m[3 * AX + 1] += f * v;
        m[3 * AX + 2] += f * v * v;
    }
    if (c == 0.0 || ny <= Ra) return;
    // cone fluxes of the adjacent sub-boxes
    const double hi = ny < Rb ? ny : Rb;
    const double hm = 0.5 * (hi - Ra), hc = 0.5 * (hi + Ra);
    const double yh[3] = {y[0] * inv_ny, y[1] * inv_ny, y[2] * inv_ny};
    const double flux_scale = wgt * inv_ny * inv_ny * inv_ny * hm;
#pragma unroll
    for (int side = 0; side < 2; side++) {
        // s = -1: box sb_AX = -1, lower face (y.n = -c); s = +1: box +1, upper face (y.n = c);
        // s = 0: box -1 upper face (y.n = c) and box +1 lower face (y.n = -c)
        int sbax;
        double ydotn;
        if (s == 0) {
            sbax = side == 0 ? -1 : 1;
            ydotn = side == 0 ? c : -c;
        } else {
            if (side == 1) break;
            sbax = s;
            ydotn = s < 0 ? -c : c;
        }
        int sb[3];
        sb[AX] = sbax;
        sb[A1] = s1;
        sb[A2] = s2;
        double lamI = 0.0, cb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
        for (int q = 0; q < 3; q++) {
            const double u = hc + hm * g3x[q];
            const double wq = g3w[q] * u;
            const double l0 = ANI ? 1.0 - sb[0] * (u * yh[0] - D[0]) * ih[0] : 1.0 - sb[0] * (u * yh[0] - D[0]);
            const double l1 = ANI ? 1.0 - sb[1] * (u * yh[1] - D[1]) * ih[1] : 1.0 - sb[1] * (u * yh[1] - D[1]);
            const double l2 = ANI ? 1.0 - sb[2] * (u * yh[2] - D[2]) * ih[2] : 1.0 - sb[2] * (u * yh[2] - D[2]);
            const double v = (u - Ra) * inv_r;
            lamI += wq * l0 * l1 * l2;
            const double w0 = wq, w1 = wq * v, w2 = wq * v * v;
            const double pxy = ANI ? sb[0] * sb[1] * l2 * (ih[0] * ih[1]) : sb[0] * sb[1] * l2;
            const double pxz = ANI ? sb[0] * sb[2] * l1 * (ih[0] * ih[2]) : sb[0] * sb[2] * l1;
            const double pyz = ANI ? sb[1] * sb[2] * l0 * (ih[1] * ih[2]) : sb[1] * sb[2] * l0;
            cb[0][0] += w0 * pxy; cb[0][1] += w1 * pxy; cb[0][2] += w2 * pxy;
            cb[1][0] += w0 * pxz; cb[1][1] += w1 * pxz; cb[1][2] += w2 * pxz;
            cb[2][0] += w0 * pyz; cb[2][1] += w1 * pyz; cb[2][2] += w2 * pyz;
        }
        const double f = flux_scale * ydotn;
        m[18] += f * lamI;
#pragma unroll
        for (int pr = 0; pr < 3; pr++)
#pragma unroll
            for (int j = 0; j < 3; j++) m[9 + 3 * pr + j] += f * cb[pr][j];
    }
}

constexpr double kSentinel = 1e300;
constexpr int kMaxGrade = 6;   // graded tau points towards the foot (ratio 3)

// The edge E of a face or plane square (plane y_AX = c = D[AX] + s h_AX, sub-square signs s1, s2) seen from
// the foot of the perpendicular from the origin:
// E = 0: y_A2 = lo2 (s along A1); 1: y_A1 = hi1 (s along A2); 2: y_A2 = hi2; 3: y_A1 = lo1.
struct FaceEdge {
    double c;        // distance of the plane
    double p;        // signed distance of the edge's line from the foot
    double fixed;    // its in-plane coordinate
    double rho0;     // rays start here: inside the inner sphere nothing contributes, and what lies
                     // nearer to the foot than the square cancels between its edges
    double rhoB;     // in-plane radius of the outer sphere (0: it does not reach the plane)
    double grade;    // |c| if the rays are graded towards the foot, else 0
};

// Cuts edge E for the shell [Ra, Rb): its geometry, and in sp the six ascending split points of the edge
// coordinate (kSentinel where there are fewer).  False if nothing on it contributes.
template <int AX, bool ANI>
__host__ __device__ inline bool face_edge(int E, const double D[3], double Ra, double Rb, const double *hv, int s, int s1,
                                          int s2, FaceEdge &g, double sp[6])
{
    constexpr int A1 = (AX + 1) % 3, A2 = (AX + 2) % 3;
    const double e0_ = ANI ? hv[AX] : 1.0, e1_ = ANI ? hv[A1] : 1.0, e2_ = ANI ? hv[A2] : 1.0;
    const double c = D[AX] + s * e0_;
    const double lo1 = s1 > 0 ? D[A1] : D[A1] - e1_, lo2 = s2 > 0 ? D[A2] : D[A2] - e2_;
    const double hi1 = lo1 + e1_, hi2 = lo2 + e2_;
    // range [e0, e1] of the edge coordinate
    const bool along2 = E & 1, upper = E == 1 || E == 2;
    const double fixed = along2 ? (upper ? hi1 : lo1) : (upper ? hi2 : lo2);
    const double p = upper ? fixed : -fixed;
    const double e0 = along2 ? lo2 : lo1, e1 = along2 ? hi2 : hi1;
    if (p == 0.0) return false;
    const double ap = fabs(p), c2 = c * c;
    // nothing contributes where |y| <= a: skip edges whose farthest point is inside the shell
    const double Lmax2 = p * p + fmax(e0 * e0, e1 * e1);
    if (c2 + Lmax2 <= Ra * Ra) return false;
    // in-plane radii of the two spheres (0 when the sphere does not reach the plane)
    const bool haveA = Ra > fabs(c), haveB = Rb > fabs(c);
    const double rhoA = haveA ? sqrt(Ra * Ra - c2) : 0.0;
    const double rhoB = haveB ? sqrt(Rb * Rb - c2) : 0.0;
    // distance of the square from the foot, used from twice its longer edge on (nearer, the start radius
    // over the ray's length would bend more over the edge than the rays from 0 do)
    const double n1 = fmax(0.0, fmax(lo1, -hi1)), n2 = fmax(0.0, fmax(lo2, -hi2)), rn = sqrt(n1 * n1 + n2 * n2);
    g.c = c;
    g.p = p;
    g.fixed = fixed;
    g.rho0 = fmax(rhoA, rn >= 2.0 * fmax(e1_, e2_) ? rn : 0.0);
    g.rhoB = rhoB;
    g.grade = haveA ? 0.0 : fabs(c);
    // split points of the edge coordinate where the spheres cross the edge
    sp[0] = e0;
    sp[1] = sp[2] = sp[3] = sp[4] = kSentinel;
    sp[5] = e1;
    if (haveA && rhoA > ap) {
        const double t = sqrt(rhoA * rhoA - p * p);
        if (t > e0 && t < e1) sp[1] = t;
        if (-t > e0 && -t < e1) sp[2] = -t;
    }
    if (haveB && rhoB > ap) {
        const double t = sqrt(rhoB * rhoB - p * p);
        if (t > e0 && t < e1) sp[3] = t;
        if (-t > e0 && -t < e1) sp[4] = -t;
    }
    sort_fixed<6>(sp);
    return true;
}

// Whether the interval [sa, sb] of the edge holds anything: rays to its middle reach rho0 (the splits put
// either all of an interval or nothing of it outside the inner sphere, and no point of an edge is nearer to
// the foot than the square; where the middle is the nearest point, both sides are the same number).
__host__ __device__ inline bool edge_interval(const FaceEdge &g, double sa, double sb)
{
    if (!(sb > sa) || sb >= kSentinel) return false;
    const double sm = 0.5 * (sa + sb);
    return g.p * g.p + sm * sm >= g.rho0 * g.rho0;
}

// One s-node (gx, gw on [-1, 1]) of the interval [sa, sb] of an edge: the ray to it, cut at the outer sphere
// and graded (ratio 3) towards the foot where the integrand does not vanish there, nt points a cell.
template <int AX, bool ANI>
__host__ __device__ inline void edge_node(const FaceEdge &g, bool along2, double sa, double sb, double gx, double gw,
                                          int nt, const double *tx, const double *tw, const double *g3x,
                                          const double *g3w, const double D[3], double Ra, double Rb, double inv_r,
                                          const double *ih, int s, int s1, int s2, double m[kMoments])
{
    constexpr int A1 = (AX + 1) % 3, A2 = (AX + 2) % 3;
    const double shm = 0.5 * (sb - sa), shc = 0.5 * (sb + sa);
    const double sn = shc + shm * gx;
    const double L = sqrt(g.p * g.p + sn * sn);
    const double ey1 = along2 ? g.fixed : sn, ey2 = along2 ? sn : g.fixed;
    const double wsn = gw * shm * g.p;
    const double c2 = g.c * g.c, tB = g.rhoB > 0.0 ? g.rhoB / L : 2.0;
    double ta = g.rho0 / L, tg = g.grade > 0.0 ? g.grade / L : 2.0;
    int left = kMaxGrade;
    while (ta < 1.0) {
        while (tg <= ta && left > 0) {
            tg *= 3.0;
            left--;
        }
        double tb = 1.0;
        if (left > 0 && tg < tb) tb = tg;
        if (tB > ta && tB < tb) tb = tB;
        const double thm = 0.5 * (tb - ta), thc = 0.5 * (tb + ta);
        for (int q = 0; q < nt; q++) {
            const double tau = thc + thm * tx[q];
            double y[3];
            y[AX] = g.c;
            y[A1] = tau * ey1;
            y[A2] = tau * ey2;
            const double ny = sqrt(c2 + tau * tau * L * L);
            const double wgt = wsn * thm * tw[q] * tau;
            node_contrib<AX, ANI>(m, y, ny, wgt, s, s1, s2, D, Ra, Rb, inv_r, ih, g3x, g3w);
        }
        ta = tb;
    }
}

// s-interval iv, s-node iq of the four edges of a square, serially (host checks)
template <int AX, bool ANI>
__host__ __device__ inline void gen_square(int nq, const double *glx, const double *glw, const double *g3x,
                                           const double *g3w, const double D[3], double Ra, double Rb, double inv_r,
                                           const double *hv, const double *ih, int s, int s1, int s2, int iv, int iq,
                                           double m[kMoments])
{
    for (int E = 0; E < 4; E++) {
        FaceEdge g;
        double sp[6];
        if (!face_edge<AX, ANI>(E, D, Ra, Rb, hv, s, s1, s2, g, sp) || !edge_interval(g, sp[iv], sp[iv + 1])) continue;
        edge_node<AX, ANI>(g, E & 1, sp[iv], sp[iv + 1], glx[iq], glw[iq], nq, glx, glw, g3x, g3w, D, Ra, Rb, inv_r, ih,
                           s, s1, s2, m);
    }
}

// Number of work items per (offset, shell): 36 unit squares x 5 s-intervals x nq s-nodes.
__host__ __device__ inline int gen_items(int nq) { return 36 * 5 * nq; }

// Item index -> (unit square, s-interval, s-node); the four edges of the square are
// handled inside the item.
template <bool ANI>
__host__ __device__ inline void gen_item(int nq, const double *glx, const double *glw, const double *g3x,
                                         const double *g3w, const double D[3], int a, double r, const double *hv,
                                         const double *ih, int it, double m[kMoments])
{
    const double Ra = a * r, Rb = (a + 1) * r, inv_r = 1.0 / r;
    const int iq = it % nq;
    const int rest = it / nq;
    const int iv = rest % 5;
    const int sq = rest / 5;
    const int ax = sq / 12, rem = sq % 12;
    const int s = rem / 4 - 1;
    const int s1 = (rem & 1) ? 1 : -1, s2 = (rem & 2) ? 1 : -1;
    if (ax == 0) gen_square<0, ANI>(nq, glx, glw, g3x, g3w, D, Ra, Rb, inv_r, hv, ih, s, s1, s2, iv, iq, m);
    else if (ax == 1) gen_square<1, ANI>(nq, glx, glw, g3x, g3w, D, Ra, Rb, inv_r, hv, ih, s, s1, s2, iv, iq, m);
    else gen_square<2, ANI>(nq, glx, glw, g3x, g3w, D, Ra, Rb, inv_r, hv, ih, s, s1, s2, iv, iq, m);
}

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Scratch of one wave: the rules of its offset, the 48 edges of one plane axis and the list of their
// contributing intervals (at most 5 an edge).
struct GenLds {
    double sx[kMaxQ], sw[kMaxQ], tx[kMaxQ], tw[kMaxQ], g3x[3], g3w[3];
    FaceEdge edge[48];
    double ia[240], ib[240];
    unsigned char ie[240];
};

__device__ inline void load_rules(GenLds &l, const GenRules &R, int cls)
{
    for (int i = threadIdx.x; i < kMaxQ; i += kGenThreads) {
        l.sx[i] = R.x[R.rs[cls]][i];
        l.sw[i] = R.w[R.rs[cls]][i];
        l.tx[i] = R.x[R.rt[cls]][i];
        l.tw[i] = R.w[R.rt[cls]][i];
    }
    if (threadIdx.x < 3) {
        l.g3x[threadIdx.x] = R.g3x[threadIdx.x];
        l.g3w[threadIdx.x] = R.g3w[threadIdx.x];
    }
    __syncthreads();
}

// The rules of one shell of an offset of order class `far`, loaded unless they are there (cls: the class that is)
__device__ inline void shell_rules(GenLds &l, const GenRules &R, int far, const double D[3], double Ra, double Rb,
                                   const double *hv, int &cls)
{
    const int want = far > 0 && grazed(D, Ra, Rb, hv) ? 0 : far;
    if (want == cls) return;
    __syncthreads();
    load_rules(l, R, want);
    cls = want;
}

// The planes of axis AX, shell [Ra, Rb): each lane's share of the moments (every lane of the wave calls it)
template <int AX, bool ANI>
__device__ __attribute__((always_inline)) inline void axis_moments(GenLds &l, int ns, int nt, const double D[3],
                                                                   double Ra, double Rb, double inv_r,
                                                                   const double *hv, const double *ih,
                                                                   double (&m)[kMoments])
{
    const int lane = threadIdx.x;
    // lane e + 4 sq: edge e of square sq = (s1 > 0) + 2 (s2 > 0) + 4 (s + 1)
    double sp[6];
    unsigned keep = 0;   // its contributing intervals
    if (lane < 48) {
        const int sq = lane >> 2;
        FaceEdge g;
        if (face_edge<AX, ANI>(lane & 3, D, Ra, Rb, hv, (sq >> 2) - 1, (sq & 1) ? 1 : -1, (sq & 2) ? 1 : -1, g, sp)) {
#pragma unroll
            for (int j = 0; j < 5; j++)
                if (edge_interval(g, sp[j], sp[j + 1])) keep |= 1u << j;
            l.edge[lane] = g;
        }
    }
    int at = __popc(keep);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(at, off);
        if (lane >= off) at += v;
    }
    const int total = __shfl(at, 63);
    at -= __popc(keep);
#pragma unroll
    for (int j = 0; j < 5; j++)
        if (keep & (1u << j)) {
            l.ia[at] = sp[j];
            l.ib[at] = sp[j + 1];
            l.ie[at] = (unsigned char)lane;
            at++;
        }
    __syncthreads();
    for (int it = lane; it < total * ns; it += kGenThreads) {
        const int e = it / ns, iq = it - e * ns;
        const int id = l.ie[e], sq = id >> 2;
        const FaceEdge g = l.edge[id];
        edge_node<AX, ANI>(g, id & 1, l.ia[e], l.ib[e], l.sx[iq], l.sw[iq], nt, l.tx, l.tw, l.g3x, l.g3w, D, Ra, Rb,
                           inv_r, ih, (sq >> 2) - 1, (sq & 1) ? 1 : -1, (sq & 2) ? 1 : -1, m);
    }
    __syncthreads();
}

// The 19 moments of shell a, in lane 0 (every lane of the wave calls it)
template <bool ANI>
__device__ __attribute__((always_inline)) inline void shell_moments(GenLds &l, int ns, int nt, const double D[3], int a,
                                                                    double r, const double *hv, const double *ih,
                                                                    double (&m)[kMoments])
{
    const double Ra = a * r, Rb = (a + 1) * r, inv_r = 1.0 / r;
#pragma unroll
    for (int i = 0; i < kMoments; i++) m[i] = 0.0;
    axis_moments<0, ANI>(l, ns, nt, D, Ra, Rb, inv_r, hv, ih, m);
    axis_moments<1, ANI>(l, ns, nt, D, Ra, Rb, inv_r, hv, ih, m);
    axis_moments<2, ANI>(l, ns, nt, D, Ra, Rb, inv_r, hv, ih, m);
#pragma unroll
    for (int i = 0; i < kMoments; i++) m[i] = wave_sum(m[i]);
}

// Which stored offset stands for |D|: axes of equal voxel edges may trade their components, and the larger
// component goes to the axis with more voxels (so it stays on the grid), the lower axis among equals.
// d becomes that offset; pos[a] is the axis where the component of axis a went.
__host__ __device__ inline void stored_offset(int d[3], int pos[3], const int n[3], const double hv[3])
{
    pos[0] = 0;
    pos[1] = 1;
    pos[2] = 2;
    // three passes of conditional exchanges sort three axes; axes of unequal edges never trade
    for (int pass = 0; pass < 3; pass++)
        for (int i = 0; i < 2; i++)
            for (int j = i + 1; j < 3; j++) {
                if (hv[i] != hv[j]) continue;
                const bool first = n[i] >= n[j];   // axis i takes the larger component
                if (first ? d[i] < d[j] : d[i] > d[j]) {
                    const int t = d[i];
                    d[i] = d[j];
                    d[j] = t;
                    for (int a = 0; a < 3; a++) pos[a] = pos[a] == i ? j : pos[a] == j ? i : pos[a];
                }
            }
}

// Held to two waves per SIMD, here and for the off-grid table: with a rule per shell the compiler otherwise takes
// 22 more registers and leaves one (new 48^3 solver 35.6 against 32.4 ms, 24^3 job 74.5 against 64.6).
template <bool ANI>
__global__ void __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(2))) k_gen_moments(double *__restrict__ mom, GenArg ga)
{
    __shared__ GenLds lds;
    const int idx = blockIdx.x;
    const int d0[3] = {idx % ga.Uo, (idx / ga.Uo) % ga.Vo, idx / (ga.Uo * ga.Vo)}, n[3] = {ga.Uo, ga.Vo, ga.Wo};
    int d[3] = {d0[0], d0[1], d0[2]}, pos[3];
    stored_offset(d, pos, n, ga.hv);
    if (d[0] != d0[0] || d[1] != d0[1] || d[2] != d0[2]) return;   // another offset stands for this one
    const double D[3] = {d[0] * ga.hv[0], d[1] * ga.hv[1], d[2] * ga.hv[2]};
    int a_lo, nsh;
    shell_range(d[0], d[1], d[2], ga.hv, ga.r, a_lo, nsh);
    const int far = order_class(d[0], d[1], d[2], ga.hv);
    int cls = -1;
    double *out = mom + (size_t)idx * ga.ms * kMoments;
    for (int sh = 0; sh < min(nsh, ga.ms); sh++) {   // the others stay zero
        shell_rules(lds, *ga.rules, far, D, (a_lo + sh) * ga.r, (a_lo + sh + 1) * ga.r, ga.hv, cls);
        const int ns = ga.rules->ns[cls], nt = ga.rules->nt[cls];
        double m[kMoments];
        shell_moments<ANI>(lds, ns, nt, D, a_lo + sh, ga.r, ga.hv, ga.ih, m);
        if (threadIdx.x == 0)
#pragma unroll
            for (int i = 0; i < kMoments; i++) out[sh * kMoments + i] = m[i];
    }
}

// K_k at an octant offset >= 0 from the moments of its shells a_lo .. a_lo + nsh - 1.
__host__ __device__ inline void kernel_from_shells(const double *mom_d, int a_lo, int nsh, int k, double r,
                                                   double K[6])
{
    for (int i = 0; i < 6; i++) K[i] = 0.0;
    // B(k+1-|d|/r) on shell k-p as a quadratic in v = |d|/r - a:  p=0: (1-v)^2/2, p=1: (1+2v-2v^2)/2,
    // p=2: v^2/2; the time derivatives bring B'' / r^2
    const double cg[3][3] = {{0.5, -1.0, 0.5}, {0.5, 1.0, -1.0}, {0.0, 0.0, 0.5}};
    const double ir2 = 1.0 / (r * r);
    const double cb[3] = {ir2, -2.0 * ir2, ir2};  // B'' on the three pieces
    for (int p = 0; p < 3; p++) {
        int sh = k - p - a_lo;
        if (sh < 0 || sh >= nsh) continue;
        const double *m = mom_d + sh * kMoments;
        for (int al = 0; al < 3; al++)
            K[al] += cg[p][0] * m[3 * al] + cg[p][1] * m[3 * al + 1] + cg[p][2] * m[3 * al + 2] - cb[p] * m[18];
        for (int pr = 0; pr < 3; pr++)
            K[3 + pr] += cg[p][0] * m[9 + 3 * pr] + cg[p][1] * m[9 + 3 * pr + 1] + cg[p][2] * m[9 + 3 * pr + 2];
    }
    for (int i = 0; i < 6; i++) K[i] *= kInvFourPi;
}

// K_k at integer octant offset (dx,dy,dz) >= 0 from the shell moments.
__host__ __device__ inline void kernel_from_moments(const double *mom_d, int dx, int dy, int dz, int k, double r,
                                                    const double hv[3], double K[6])
{
    int a_lo, nsh;
    shell_range(dx, dy, dz, hv, r, a_lo, nsh);
    kernel_from_shells(mom_d, a_lo, nsh, k, r, K);
    // exact zeros of the odd components on their symmetry planes
    if (dx == 0 || dy == 0) K[3] = 0.0;
    if (dx == 0 || dz == 0) K[4] = 0.0;
    if (dy == 0 || dz == 0) K[5] = 0.0;
}

struct MomView {
    const double *mom;   // [Wo][Vo][Uo][ms][kMoments]
    int Uo, Vo, Wo, ms;
    double r;
    double hv[3];
};

__device__ inline void kernel_at(const MomView &g, int k, int Dx, int Dy, int Dz, double K[6])
{
    int d[3] = {Dx < 0 ? -Dx : Dx, Dy < 0 ? -Dy : Dy, Dz < 0 ? -Dz : Dz}, pos[3];
    const int n[3] = {g.Uo, g.Vo, g.Wo};
    stored_offset(d, pos, n, g.hv);
    const double *md = g.mom + ((size_t)(d[2] * g.Vo + d[1]) * g.Uo + d[0]) * g.ms * kMoments;
    double Ks[6];
    kernel_from_moments(md, d[0], d[1], d[2], k, g.r, g.hv, Ks);
    // component ab of K is component pos[a] pos[b] of the stored offset's
    for (int a = 0; a < 3; a++) K[a] = pos[a] == 0 ? Ks[0] : pos[a] == 1 ? Ks[1] : Ks[2];
    auto off = [&](int i) { return i == 1 ? Ks[3] : i == 2 ? Ks[4] : Ks[5]; };   // by the sum of the two axes
    K[3] = off(pos[0] + pos[1]);
    K[4] = off(pos[0] + pos[2]);
    K[5] = off(pos[1] + pos[2]);
    double sx = Dx < 0 ? -1.0 : 1.0, sy = Dy < 0 ? -1.0 : 1.0, sz = Dz < 0 ? -1.0 : 1.0;
    K[3] *= sx * sy;
    K[4] *= sx * sz;
    K[5] *= sy * sz;
}

// Periodic embedding on the Nx x Ny x Nz grid: index i holds offset i (i < U) or i - N
// (i > N - U); the remaining indices are zero (Appendix A, first column of the circulant).
__global__ void k_kernel_grid(MomView g, int k, int Nx, int Ny, int Nz, double *__restrict__ grid)
{
    const int Uo = g.Uo, Vo = g.Vo, Wo = g.Wo;
    size_t n = (size_t)Nx * Ny * Nz;
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int ix = (int)(i % Nx), iy = (int)((i / Nx) % Ny), iz = (int)(i / ((size_t)Nx * Ny));
    int Dx = ix < Uo ? ix : (ix > Nx - Uo ? ix - Nx : INT32_MAX);
    int Dy = iy < Vo ? iy : (iy > Ny - Vo ? iy - Ny : INT32_MAX);
    int Dz = iz < Wo ? iz : (iz > Nz - Wo ? iz - Nz : INT32_MAX);
    double K[6] = {0, 0, 0, 0, 0, 0};
    if (Dx != INT32_MAX && Dy != INT32_MAX && Dz != INT32_MAX) kernel_at(g, k, Dx, Dy, Dz, K);
    for (int c = 0; c < 6; c++) grid[c * n + i] = K[c];
}

__global__ void k_kernel_values(MomView g, int n, const int *__restrict__ lag, const int *__restrict__ off,
                                double *__restrict__ out)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double K[6];
    kernel_at(g, lag[i], off[3 * i], off[3 * i + 1], off[3 * i + 2], K);
    for (int c = 0; c < 6; c++) out[6 * i + c] = K[c];
}

// ---------------------------------------------------------------------------- off-grid offsets
// Shell range for a real octant offset D >= 0 (the distances between points of the two
// voxels lie in [|max(D - 1, 0)|, |D + 1|]).
// D in voxel steps per axis; edges hv.
__host__ __device__ inline void shell_range_real(const double D[3], const double hv[3], double r, int &a_lo,
                                                 int &nsh)
{
    double a2 = 0.0, b2 = 0.0;
    for (int i = 0; i < 3; i++) {
        const double e = D[i] > 1.0 ? (D[i] - 1.0) * hv[i] : 0.0;
        a2 += e * e;
        b2 += ((D[i] + 1.0) * hv[i]) * ((D[i] + 1.0) * hv[i]);
    }
    shell_bounds(a2, b2, r, a_lo, nsh);
    if (nsh > kShellCap) nsh = kShellCap;   // cannot happen for r >= kMinCdtOverH
}

// K_k for k = kmin .. kmin + nw - 1 at the signed real offset Ds, serially (host checks and
// reference): fold to the octant, quadrature of every shell, parity signs.
__host__ __device__ inline void fold_offset(const double Ds[3], double D[3], double sg[3])
{
    for (int i = 0; i < 3; i++) {
        D[i] = Ds[i] < 0.0 ? -Ds[i] : Ds[i];
        sg[i] = Ds[i] < 0.0 ? -1.0 : 1.0;
    }
}

__host__ __device__ inline void finish_offgrid(const double D[3], const double sg[3], double K[6])
{
    if (D[0] == 0.0 || D[1] == 0.0) K[3] = 0.0;
    if (D[0] == 0.0 || D[2] == 0.0) K[4] = 0.0;
    if (D[1] == 0.0 || D[2] == 0.0) K[5] = 0.0;
    K[3] *= sg[0] * sg[1];
    K[4] *= sg[0] * sg[2];
    K[5] *= sg[1] * sg[2];
}

struct OffgridArg {
    const double *pos;        // [np][3] test-voxel centres, voxel steps per axis from the grid corner
    const int *pair_probe;    // [npairs]
    const int *pair_vox;      // [npairs] source voxel, linear index u + U (v + V w)
    const int *pair_kmin;     // [npairs] first lag of the window
    int U, V;
    double r;                 // c dt
    double hv[3], ih[3];      // voxel edges and their inverses
    int nw;                   // lags per pair
    int kmax;                 // lags above kmax are stored as zero
    long npairs;
    double *out;              // [nw][npairs][6]: for one window slot, consecutive pairs are adjacent
};

// One 64-lane block per (test voxel, source voxel) pair: shell moments by the same face
// quadrature as the grid kernels, then the pair's window of lags.
template <bool ANI>
__global__ void __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(2))) k_offgrid_table(OffgridArg oa, GenArg ga)
{
    const long i = blockIdx.x;
    const int p = oa.pair_probe[i], vox = oa.pair_vox[i];
    const int u = vox % oa.U, v = (vox / oa.U) % oa.V, w = vox / (oa.U * oa.V);
    const double Ds[3] = {oa.pos[3 * p] - (u + 0.5), oa.pos[3 * p + 1] - (v + 0.5), oa.pos[3 * p + 2] - (w + 0.5)};
    double Dv[3], sg[3];
    fold_offset(Ds, Dv, sg);
    int a_lo, nsh;
    shell_range_real(Dv, oa.hv, oa.r, a_lo, nsh);
    const double D[3] = {Dv[0] * oa.hv[0], Dv[1] * oa.hv[1], Dv[2] * oa.hv[2]};
    __shared__ GenLds lds;
    __shared__ double mom[kShellCap * kMoments];
    const int far = order_class(Dv[0], Dv[1], Dv[2], oa.hv);
    int cls = -1;
    for (int sh = 0; sh < nsh; sh++) {
        shell_rules(lds, *ga.rules, far, D, (a_lo + sh) * oa.r, (a_lo + sh + 1) * oa.r, oa.hv, cls);
        const int ns = ga.rules->ns[cls], nt = ga.rules->nt[cls];
        double m[kMoments];
        shell_moments<ANI>(lds, ns, nt, D, a_lo + sh, oa.r, oa.hv, oa.ih, m);
        if (threadIdx.x == 0)
#pragma unroll
            for (int t = 0; t < kMoments; t++) mom[sh * kMoments + t] = m[t];
    }
    __syncthreads();
    for (int wl = threadIdx.x; wl < oa.nw; wl += kGenThreads) {
        const int k = oa.pair_kmin[i] + wl;
        double K[6] = {0, 0, 0, 0, 0, 0};
        if (k <= oa.kmax) {
            kernel_from_shells(mom, a_lo, nsh, k, oa.r, K);
            finish_offgrid(D, sg, K);
        }
        double *o = oa.out + ((long)wl * oa.npairs + i) * 6;
        for (int c = 0; c < 6; c++) o[c] = K[c];
    }
}

// Gauss-Legendre rule on [-1, 1]: roots of P_n by Newton's method from Tricomi's initial
// guesses, in long double; weights 2 / ((1 - x^2) P_n'(x)^2).
void legendre_rule(int n, double *x, double *w)
{
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int i = 0; i < n; i++) {
        long double th = pi * (4.0L * (i + 1) - 1.0L) / (4.0L * n + 2.0L);
        long double z = (1.0L - (n - 1.0L) / (8.0L * n * n * n)) * cosl(th);
        long double dp = 0.0L;
        for (int iter = 0; iter < 60; iter++) {
            long double pm = 1.0L, pc = z;  // P_0, P_1
            for (int j = 1; j < n; j++) {
                long double pn = ((2.0L * j + 1.0L) * z * pc - j * pm) / (j + 1.0L);
                pm = pc;
                pc = pn;
            }
            dp = n * (pm - z * pc) / (1.0L - z * z);
            long double dz = pc / dp;
            z -= dz;
            if (fabsl(dz) <= 1e-19L * fabsl(z) + 1e-30L) break;
        }
        long double pm = 1.0L, pc = z;
        for (int j = 1; j < n; j++) {
            long double pn = ((2.0L * j + 1.0L) * z * pc - j * pm) / (j + 1.0L);
            pm = pc;
            pc = pn;
        }
        dp = n * (pm - z * pc) / (1.0L - z * z);
        x[n - 1 - i] = (double)z;   // ascending order
        w[n - 1 - i] = (double)(2.0L / ((1.0L - z * z) * dp * dp));
    }
}

}  // namespace

// The rules for quad_order (0: by class), on the device for as long as the object lives.
namespace {
struct RulesOnDevice {
    DevTemp tmp;
    hipStream_t st;
    RulesOnDevice(int quad_order, const DevAlloc &da, hipStream_t s) : tmp(da, sizeof(GenRules), "quadrature rules"), st(s)
    {
        if (quad_order != 0 && (quad_order < 4 || quad_order > kMaxQ)) throw ArgError("quad_order must be in [4, 24]");
        GenRules R{};
        for (int c = 0; c < kOrderClasses; c++) {
            R.ns[c] = quad_order ? quad_order : kClassS[c];
            R.nt[c] = quad_order ? quad_order : kClassT[c];
            R.rs[c] = 2 * c;
            R.rt[c] = 2 * c + 1;
            legendre_rule(R.ns[c], R.x[2 * c], R.w[2 * c]);
            legendre_rule(R.nt[c], R.x[2 * c + 1], R.w[2 * c + 1]);
        }
        legendre_rule(3, R.g3x, R.g3w);
        MJ_CHECK(hipMemcpyAsync(tmp.p, &R, sizeof R, hipMemcpyHostToDevice, st));
        MJ_CHECK(hipStreamSynchronize(st));
    }
    ~RulesOnDevice() { (void)hipStreamSynchronize(st); }   // the kernel that reads them has ended
    const GenRules *get() const { return tmp.as<GenRules>(); }
};
}  // namespace

static void check_geometry(double r, const double hv[3])
{
    const double hmin = fmin(hv[0], fmin(hv[1], hv[2])), hmax = fmax(hv[0], fmax(hv[1], hv[2]));
    if (!(hmin > 0.0) || !(r <= hmin * (1.0 + 1e-12)) || !(r >= kMinCdtOverH * hmax))
        throw ArgError("c dt must lie in [0.3 max(h), min(h)]");
    if (shells_per_offset(r, hv) > kShellCap) throw ArgError("too many kernel shells per voxel pair");
}

void gen_moments(GenResult &g, int U, int V, int W, double r, const double hv[3], int nquad, const DevAlloc &da,
                 hipStream_t st)
{
    const RulesOnDevice rules(nquad, da, st);
    check_geometry(r, hv);
    GenArg ga{};
    ga.rules = rules.get();
    ga.Uo = U;
    ga.Vo = V;
    ga.Wo = W;
    ga.r = r;
    for (int i = 0; i < 3; i++) {
        ga.hv[i] = hv[i];
        ga.ih[i] = 1.0 / hv[i];
        g.hv[i] = hv[i];
    }
    ga.ms = shells_per_offset(r, hv);
    g.Uo = U;
    g.Vo = V;
    g.Wo = W;
    g.ms = ga.ms;
    g.r = r;
    size_t noff = (size_t)U * V * W;
    size_t bytes = noff * g.ms * kMoments * sizeof(double);
    g.moments = (double *)da.get(bytes, "kernel moments");
    MJ_CHECK(hipMemsetAsync(g.moments, 0, bytes, st));
    if (hv[1] != 1.0 || hv[2] != 1.0)
        hipLaunchKernelGGL(k_gen_moments<true>, dim3((unsigned)noff), dim3(kGenThreads), 0, st, g.moments, ga);
    else
        hipLaunchKernelGGL(k_gen_moments<false>, dim3((unsigned)noff), dim3(kGenThreads), 0, st, g.moments, ga);
    MJ_CHECK(hipGetLastError());
}

void gen_kernel_grid(const GenResult &g, int k, int Nx, int Ny, int Nz, double *grid, hipStream_t st)
{
    size_t n = (size_t)Nx * Ny * Nz;
    dim3 blk(256), grd((unsigned)((n + 255) / 256));
    const MomView mv{g.moments, g.Uo, g.Vo, g.Wo, g.ms, g.r, {g.hv[0], g.hv[1], g.hv[2]}};
    hipLaunchKernelGGL(k_kernel_grid, grd, blk, 0, st, mv, k, Nx, Ny, Nz, grid);
    MJ_CHECK(hipGetLastError());
}

void gen_kernel_values(const GenResult &g, int n, const int *lag_dev, const int *off_dev, double *out_dev,
                       hipStream_t st)
{
    if (n <= 0) return;
    const MomView mv{g.moments, g.Uo, g.Vo, g.Wo, g.ms, g.r, {g.hv[0], g.hv[1], g.hv[2]}};
    hipLaunchKernelGGL(k_kernel_values, dim3((n + 127) / 128), dim3(128), 0, st, mv, n, lag_dev, off_dev, out_dev);
    MJ_CHECK(hipGetLastError());
}

void gen_offgrid_table(const double *pos_dev, const int *pair_probe_dev, const int *pair_vox_dev,
                       const int *pair_kmin_dev, long npairs, int U, int V, double r, const double hv[3], int nw,
                       int kmax, int nquad, double *out_dev, const DevAlloc &da, hipStream_t st)
{
    if (npairs <= 0) return;
    check_geometry(r, hv);
    if (npairs > 0x7fffffffL) throw ArgError("too many probe pairs");
    const RulesOnDevice rules(nquad, da, st);
    GenArg ga{};
    ga.rules = rules.get();
    OffgridArg oa{};
    oa.pos = pos_dev;
    oa.pair_probe = pair_probe_dev;
    oa.pair_vox = pair_vox_dev;
    oa.pair_kmin = pair_kmin_dev;
    oa.U = U;
    oa.V = V;
    oa.r = r;
    for (int i = 0; i < 3; i++) {
        oa.hv[i] = hv[i];
        oa.ih[i] = 1.0 / hv[i];
    }
    oa.nw = nw;
    oa.kmax = kmax;
    oa.npairs = npairs;
    oa.out = out_dev;
    if (hv[1] != 1.0 || hv[2] != 1.0)
        hipLaunchKernelGGL(k_offgrid_table<true>, dim3((unsigned)npairs), dim3(kGenThreads), 0, st, oa, ga);
    else
        hipLaunchKernelGGL(k_offgrid_table<false>, dim3((unsigned)npairs), dim3(kGenThreads), 0, st, oa, ga);
    MJ_CHECK(hipGetLastError());
}

}  // namespace mj
