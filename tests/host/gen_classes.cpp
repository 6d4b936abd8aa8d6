// Test harness: the orders that the kernel generator takes by distance (order_class, grazed) and the offsets
// that stand for their permutations (stored_offset), as the device's kernels use them, serially on the host.
// Built by tests/test_generator_classes_host.py.
#include "../../paper_2407_03323_amd/csrc/mj_gen.hip"

namespace mj {
template <int AX, bool ANI>
static void axis_serial(int ns, int nt, const double (&x)[2][kMaxQ], const double (&w)[2][kMaxQ], const double *g3x,
                        const double *g3w, const double D[3], double Ra, double Rb, double r, const double *hv,
                        const double *ih, double *m)
{
    for (int sq = 0; sq < 12; sq++)
        for (int E = 0; E < 4; E++) {
            const int s = (sq >> 2) - 1, s1 = (sq & 1) ? 1 : -1, s2 = (sq & 2) ? 1 : -1;
            FaceEdge g;
            double sp[6];
            if (!face_edge<AX, ANI>(E, D, Ra, Rb, hv, s, s1, s2, g, sp)) continue;
            for (int j = 0; j < 5; j++)
                if (edge_interval(g, sp[j], sp[j + 1]))
                    for (int q = 0; q < ns; q++)
                        edge_node<AX, ANI>(g, E & 1, sp[j], sp[j + 1], x[0][q], w[0][q], nt, x[1], w[1], g3x, g3w, D, Ra,
                                           Rb, 1.0 / r, ih, s, s1, s2, m);
        }
}

// K_k(D), k = 0..kmax, with `order` points a side, or, with 0, by distance.  Returns the order class of D.
extern "C" int host_class_kernels(const double *Ds, double r, double hy, double hz, int order, int kmax, double *out)
{
    const double hv[3] = {1.0, hy, hz}, ih[3] = {1.0, 1.0 / hy, 1.0 / hz};
    double Dv[3], sg[3], g3x[3], g3w[3];
    legendre_rule(3, g3x, g3w);
    fold_offset(Ds, Dv, sg);
    int a_lo, nsh;
    shell_range_real(Dv, hv, r, a_lo, nsh);
    const double D[3] = {Dv[0] * hv[0], Dv[1] * hv[1], Dv[2] * hv[2]};
    const int far = order_class(Dv[0], Dv[1], Dv[2], hv);
    double mom[kShellCap * kMoments] = {0};
    for (int sh = 0; sh < nsh; sh++) {
        const double Ra = (a_lo + sh) * r, Rb = (a_lo + sh + 1) * r;
        const int cls = far > 0 && grazed(D, Ra, Rb, hv) ? 0 : far;
        const int ns = order ? order : kClassS[cls], nt = order ? order : kClassT[cls];
        double x[2][kMaxQ], w[2][kMaxQ], *m = mom + sh * kMoments;
        legendre_rule(ns, x[0], w[0]);
        legendre_rule(nt, x[1], w[1]);
        if (hy != 1.0 || hz != 1.0) {
            axis_serial<0, true>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
            axis_serial<1, true>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
            axis_serial<2, true>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
        } else {
            axis_serial<0, false>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
            axis_serial<1, false>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
            axis_serial<2, false>(ns, nt, x, w, g3x, g3w, D, Ra, Rb, r, hv, ih, m);
        }
    }
    for (int k = 0; k <= kmax; k++) {
        kernel_from_shells(mom, a_lo, nsh, k, r, out + 6 * k);
        finish_offgrid(D, sg, out + 6 * k);
    }
    return far;
}

// The stored offset of d (replaced) on an n[0] x n[1] x n[2] grid of voxels with edges hv; pos as in stored_offset
extern "C" void host_stored_offset(int *d, int *pos, const int *n, const double *hv) { stored_offset(d, pos, n, hv); }
}  // namespace mj
