// One step of a linearly implicit scheme (Eq:IMEX_DAE) of a 1D state of 128 to 4096
// points by one workgroup, after the step's right-hand side: the thirteen launches it
// stands for (transform of U, three passes of G, the mode-wise update, the way back, the
// two combinations and the copies of the level ring) each took 2 to 21 us for a line
// that one compute unit holds.
#pragma once
#include "sgn_device.h"

namespace sgn {

// Against the general path, us per step with its right-hand side: 62 -> 19 at 128 points,
// 63 -> 23 at 512, 74 -> 43 at 2048, 93 -> 66 at 4096; at 8192, where the four vectors of
// a thread no longer fit its registers, 133 -> 149, so that length keeps the general path.
constexpr int LINIMP_NMIN = 128, LINIMP_NMAX = 4096;
constexpr int LINIMP_TERMS = 6;
struct LinimpLine {
    double L, sig, alp;            // A = sig I - alp dxx
    const double* hx;
    double *eta, *U, *u;           // the state: the current level in, the new one out
    double *eta_to, *U_to;         // the oldest level's places, which take the current one
    // eta, U of the new level: (sum_k w_k f_k) / div, in this order
    const double *fe[LINIMP_TERMS], *fU[LINIMP_TERMS];
    double w[LINIMP_TERMS], div;
    int nterms;
    // u_hat of the new level: A^{-1} (sum_j b_j R_j - sum_{j<s} c_j A u_hat_j) inv_cs; the
    // current level's R = A u_hat - G u_hat + U_hat (j = s - 1) is formed here and stored
    int s;
    const cpx<double>* Rj[2];
    const cpx<double>* uhj[3];
    double b[3], c[3], inv_cs;
    cpx<double>*R, *uh_new;        // uh_new may be uhj[0]
};

hipError_t launch_linimp_line(int n, hipStream_t stream, const LinimpLine& P, const cpx<double>* tw);

}  // namespace sgn
