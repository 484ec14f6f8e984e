// The one-workgroup linearly implicit step of 1D states (sgn_linimp.h): kernel and launch.
#include "sgn_batch.h"
#include "sgn_linimp.h"

namespace sgn {

// Half-spectrum entries of pair e in a mode array X[0 .. M] and back: pair 0 holds
// (X_0, X_M) as one complex entry.
template <int M>
__device__ __forceinline__ void pair_read(const cpx<double>* X, int tau, cpx<double>& a, cpx<double>& b) {
    a = X[tau];
    b = X[tau == 0 ? M / 2 : M - tau];
    if (tau == 0) a = C<double>(a.re, X[M].re);
}
template <int M>
__device__ __forceinline__ void pair_write(cpx<double>* X, int tau, cpx<double> a, cpx<double> b) {
    X[tau] = tau == 0 ? C<double>(a.re, 0.0) : a;
    X[tau == 0 ? M / 2 : M - tau] = b;
    if (tau == 0) X[M] = C<double>(a.im, 0.0);
}

template <int M>
__device__ __noinline__ void line_linimp(const LinimpLine& P, const cpx<double>* __restrict__ tw, void* lds,
                                         double* red) {
    using Geo = LineGeo<double, M>;
    constexpr int E = Geo::E, G = Geo::G, NP = Geo::NP;
    Line<double, M> L(lds, red, tw);
    const LinePairs<double, M> K(L, 6.283185307179586476925286766559 / P.L);
    cpx<double> v[E], Uh[NP][2], p[NP][2];
#pragma unroll
    for (int s = 0; s < E; ++s) v[s] = C<double>(0, 0);
#pragma unroll
    for (int e = 0; e < NP; ++e) Uh[e][0] = Uh[e][1] = p[e][0] = p[e][1] = C<double>(0, 0);
    if (L.act && L.fld == 0) {
#pragma unroll
        for (int s = 0; s < E; ++s) v[s] = ld2(P.U, L.t + s * G);
    }
    L.sync_all();   // the twiddle table
    line_to_pairs<double, M>(L, K, v, [&](int e, cpx<double> x0, cpx<double> x1, cpx<double>, cpx<double>) {
        Uh[e][0] = x0;
        Uh[e][1] = x1;
    });
    if (L.act) {
        const int q = L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) pair_read<M>(P.uhj[P.s - 1], K.tau(q, e), p[e][0], p[e][1]);
    }
    L.sync_all();
    // R = A u_hat - G u_hat + U_hat, into Uh
    double pq;
    const LineCoefFly<double, M> fly{P.eta, P.hx, L.fld};
    line_apply<double, M>(L, K, p, fly, pq, [&](int e, cpx<double> q0, cpx<double> q1) {
        const int q = L.thread();
        const double k0 = K.k0(q, e), k1 = K.k1(q, e);
        Uh[e][0] = ((P.sig + P.alp * k0 * k0) * p[e][0] - q0) + Uh[e][0];
        Uh[e][1] = ((P.sig + P.alp * k1 * k1) * p[e][1] - q1) + Uh[e][1];
    });
    // the new u_hat, into p, every level read before one is written
    if (L.act) {
        const int q = L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const int tau = K.tau(q, e);
            const double k0 = K.k0(q, e), k1 = K.k1(q, e);
            const double A0 = P.sig + P.alp * k0 * k0, A1 = P.sig + P.alp * k1 * k1;
            cpx<double> r0 = C<double>(0, 0), r1 = C<double>(0, 0);
            for (int j = 0; j < P.s; ++j) {
                cpx<double> R0 = Uh[e][0], R1 = Uh[e][1];
                if (j < P.s - 1) pair_read<M>(P.Rj[j], tau, R0, R1);
                r0 = r0 + P.b[j] * R0;
                r1 = r1 + P.b[j] * R1;
                if (P.c[j] != 0.0) {
                    cpx<double> u0, u1;
                    pair_read<M>(P.uhj[j], tau, u0, u1);
                    r0 = r0 - (P.c[j] * A0) * u0;
                    r1 = r1 - (P.c[j] * A1) * u1;
                }
            }
            p[e][0] = (P.inv_cs / A0) * r0;
            p[e][1] = (P.inv_cs / A1) * r1;
            pair_write<M>(P.R, tau, Uh[e][0], Uh[e][1]);
            pair_write<M>(P.uh_new, tau, p[e][0], p[e][1]);
        }
    }
    L.sync_all();   // every thread is done with eta, U and the exchange buffers
    // eta (field 0's threads) and U (field 1's) of the new level, the ring's shift
    if (L.act) {
        double* x = L.fld ? P.U : P.eta;
        double* to = L.fld ? P.U_to : P.eta_to;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int k = 0; k < LINIMP_TERMS; ++k) {
                if (k >= P.nterms) break;
                const cpx<double> f = ld2(L.fld ? P.fU[k] : P.fe[k], j);
                s0 += P.w[k] * f.re;
                s1 += P.w[k] * f.im;
            }
            const cpx<double> now = ld2(x, j);
            if (P.div != 1.0) {
                s0 /= P.div;
                s1 /= P.div;
            }
            st2(to, j, now);
            st2(x, j, C<double>(s0, s1));
        }
    }
    // u of the new level, by field 0; the other field carries zeros along
    L.turn_all();
    if (L.act) {
        cpx<double>*fa = L.field(0), *fb = L.field(1);
        const double invN = 1.0 / (double)Geo::N;
        const int q = L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            cpx<double> q0, q1;
            pair_c2r(invN * p[e][0], invN * p[e][1], K.w(q, e), K.tau(q, e) == 0, q0, q1);
            fa[i0] = q0;
            fa[i1] = q1;
            fb[i0] = fb[i1] = C<double>(0, 0);
        }
    }
    L.sync_all();
    if (L.act) line_load<double, M>(L, L.field(L.fld), v);
    line_transform<double, M, true>(L, v);
    if (L.act && L.fld == 0) {
#pragma unroll
        for (int s = 0; s < E; ++s) st2(P.u, L.t + s * G, v[s]);
    }
}

__global__ void __launch_bounds__(BATCH_THREADS) k_linimp_line(int n, LinimpLine P, const cpx<double>* __restrict__ tw) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[RED_DOUBLES];
    line_dispatch(n, [&](auto m) __attribute__((always_inline)) {
        if constexpr (2 * decltype(m)::value <= LINIMP_NMAX) line_linimp<decltype(m)::value>(P, tw, smem_raw, red);
    });
}

hipError_t launch_linimp_line(int n, hipStream_t stream, const LinimpLine& P, const cpx<double>* tw) {
    const size_t lds = batch_lds_bytes(n);
    int grid = 1;
    const hipError_t e = batch_grid(k_linimp_line, batch_threads_for(n), lds, 1, 1, grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_linimp_line, dim3(1), dim3(batch_threads_for(n)), lds, stream, n, P, tw);
    return hipGetLastError();
}

}  // namespace sgn
