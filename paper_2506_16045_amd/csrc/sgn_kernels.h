// Kernels of the SGN hot path.  Templated on the working precision T (double
// or float) and on the dimension D (1 or 2); reductions always accumulate in
// double.  Layouts: physical fields [ny][nx]; "H" and "S" spectral fields
// [kx][y] / [kx][ky] with kx = 0..nx/2 (see sgn_device.h).
#pragma once
#include "sgn_device.h"

namespace sgn {

// Device-side scalars of one Krylov solve (one instance per solve in flight).
// Protocol (no device-scope fences or atomics): a reducing kernel writes one
// partial sum per block; the next kernel in the stream reduces those partials
// in every block, in a fixed order, and block 0 publishes the scalars.
struct SolveScal {
    double rho;        // r.z of the current search direction
    double rho_prev;   // r.z used by the last x, r update
    double alpha, beta, bb, rr, pq, tol2, relres;
    double sig, alp, kap;     // preconditioner A = sig I - alp grad div, bound kappa_ub
    double inv_n;             // 1 / (nx ny)
    double red[8];            // results of the last generic reduction
    int iter, max_iter, done, converged, flat, status;
    int first;                // 1 until the first update (beta = 0)
    int init_bb;              // 1: ||b|| is the norm of the initial residual
    int outer;                // refinement steps taken (mixed precision)
};

// Waves per SIMD the column kernels leave room for: three, so that three blocks of
// a column each fit a compute unit (1024-point columns: 513 blocks, which two per
// compute unit would take in two rounds); the columns of 2048 take two.
template <int EPC>
constexpr int COL_WAVES = EPC <= 4 ? 3 : 2;
constexpr int PARTIALS_MAX = 4096;  // blocks of a reducing launch
// regions of the partials buffer (doubles)
constexpr int PART_C2 = 0;                       // p.Gp of the row pass (one per row block)
constexpr int PART_C3 = 4096;                    // (r.z, r.r) of the update pass (two per column block)
constexpr int PART_GEN = 4096 + 2 * 4096;        // one-off reductions (up to 5 per block)
constexpr int PART_TOTAL = PART_GEN + 5 * PARTIALS_MAX;

template <typename T, int N>
struct PtrList {
    T* p[N];
    int n;
};
constexpr int MAXF = 12;

// z = A^{-1} r in Fourier space (Def:A, section 6.1): the symbol of A is
//   1D: sig + alp k^2;   2D: sig I + alp k k^T.
// In 2D the inverse splits r into its parts along k and across k,
//   z = r_perp / sig + r_par / (sig + alp |k|^2),  r_par = k (k.r) / |k|^2,
// which keeps full relative accuracy in both parts (the equivalent
// Sherman-Morrison form r/sig - alp k (k.r)/(sig (sig + alp |k|^2)) cancels
// digits along k when alp |k|^2 >> sig).
template <typename T, int D>
__device__ __forceinline__ void precond_mode(T kx, T ky, T sig, T alp, const cpx<T> (&r)[D],
                                             cpx<T> (&z)[D]) {
    if (D == 1) {
        const T s = (T)1 / (sig + alp * kx * kx);
        z[0] = s * r[0];
    } else {
        const T k2 = kx * kx + ky * ky;
        const T is = (T)1 / sig;
        if (k2 == (T)0) {
            z[0] = is * r[0];
            z[1 % D] = is * r[1 % D];
        } else {
            const cpx<T> kr = ((T)1 / k2) * (kx * r[0] + ky * r[1 % D]);   // (k.r) / |k|^2
            const cpx<T> px = kx * kr, py = ky * kr;                       // r_par
            const T ip = (T)1 / (sig + alp * k2);
            z[0] = is * (r[0] - px) + ip * px;
            z[1 % D] = is * (r[1 % D] - py) + ip * py;
        }
    }
}

// ---------------------------------------------------------------------------
// Generic FFT passes
// ---------------------------------------------------------------------------

// Fields f >= first of a forward row pass are read as src + (c1 a + c2 b): an
// extrapolated initial guess formed from its base and two recorded offsets as
// it is loaded (b may be null; first < 0: no field is combined).
template <typename Tin>
struct RowCombo {
    const Tin* a[4];
    const Tin* b[4];
    double c1, c2;
    int first;
};

// Forward row transforms of n physical fields (Tin = double or T) into H fields.  A
// block takes its rows of one field (blocks [f nblocks, (f + 1) nblocks): field f):
// small grids fill more of the chip than with a block's fields in lockstep, and a
// field's registers leave room for twice the waves (256 x 128, three fields: forward
// 14.8 -> 6.6 us, inverse 8.2 -> 5.0; 512 x 512, inverse: 11.5 -> 7.8).  In blocks of 1024
// threads 64 registers, so that two fit a compute unit (2048 x 2048: 60 -> 51 us) though a
// few values go to scratch; blocks of 256 take the 69 they need and none, since a launch
// of a kernel that uses scratch costs the small calls, which wait for it, more than an
// eighth wave gives (grad h of a closed 64 x 64 basin 85 -> 78 us, of 1024 points 82 -> 78).
template <typename T, typename Tin, int EPC, int MAXT>
__global__ void __launch_bounds__(MAXT, EPC > 4 ? 4 : MAXT <= 256 ? 7 : 8) k_rows_fwd(RowGeom g, PtrList<const Tin, MAXF> src,
                                                   PtrList<cpx<T>, MAXF> dst,
                                                   const cpx<T>* __restrict__ tw, T scale, RowCombo<Tin> cmb) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.M);
    const int f = (int)blockIdx.x / g.nblocks;
    const RowThread<T> rt = row_thread_at<T>(g, lds, (int)blockIdx.x - f * g.nblocks, threadIdx.x);
    const Tin* in = src.p[f];
    const int k = f - cmb.first;
    const bool comb = cmb.first >= 0 && k >= 0;
    cpx<T> z[1][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        z[0][e] = C<T>(0, 0);
        if (j < g.M && rt.valid) {
            const unsigned o = rt.y * g.nx + 2 * j;
            if (comb) {
                double v[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    double t = cmb.c1 * (double)cmb.a[k][o + s];
                    if (cmb.b[k]) t += cmb.c2 * (double)cmb.b[k][o + s];
                    v[s] = (double)at32(in, o + s) + t;
                }
                z[0][e] = C<T>((T)v[0], (T)v[1]);
            } else {
                z[0][e] = C<T>((T)at32(in, o), (T)at32(in, o + 1));
            }
        }
    }
    cpx<T>* H[1] = {dst.p[f]};
    row_forward<T, EPC, 1>(g, rt, z, H, tw, twm, scale);
}

// Inverse row transforms of n H fields into physical fields (Tout), blocks as in
// k_rows_fwd: dst = acc * dst + scale * value  (acc = 0 overwrites).  With offs.n > 0,
// offs_f = new - old value of dst_f is written too (the offset of a solve's
// result from its base, recorded for the next extrapolated guess); with
// oacc != 0 it is added to offs_f instead (a result stored a second time).
template <typename T, typename Tout, int EPC, int MAXT>
__global__ void __launch_bounds__(MAXT) k_rows_inv(RowGeom g, PtrList<const cpx<T>, MAXF> src,
                                                   PtrList<Tout, MAXF> dst,
                                                   const cpx<T>* __restrict__ tw, T scale, T acc,
                                                   PtrList<Tout, MAXF> offs, int oacc) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.M);
    const int f = (int)blockIdx.x / g.nblocks;
    const RowThread<T> rt = row_thread_at<T>(g, lds, (int)blockIdx.x - f * g.nblocks, threadIdx.x);
    cpx<T> z[1][EPC];
    const cpx<T>* H[1] = {src.p[f]};
    row_inverse<T, EPC, 1>(g, rt, H, tw, twm, z);
    Tout* d = dst.p[f];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        if (j < g.M && rt.valid) {
            const unsigned o = rt.y * g.nx + 2 * j;
            T v0 = scale * z[0][e].re, v1 = scale * z[0][e].im;
            if (acc != (T)0) {
                v0 += acc * (T)d[o];
                v1 += acc * (T)d[o + 1];
            }
            if (offs.n > 0) {
                Tout* od = offs.p[f];
                const Tout d0 = (Tout)v0 - d[o], d1 = (Tout)v1 - d[o + 1];
                od[o] = oacc ? od[o] + d0 : d0;
                od[o + 1] = oacc ? od[o + 1] + d1 : d1;
            }
            d[o] = (Tout)v0;
            d[o + 1] = (Tout)v1;
        }
    }
}

// ---------------------------------------------------------------------------
// Right-hand side row passes (Eq:DSWEcf, Def:bigF, Eq:DAE_DSWE), fused with
// their pointwise stages.
// ---------------------------------------------------------------------------

// Source field i of the right-hand side's forward transforms at one point:
// [u_c (D), eta u_c (D), eta, -eta u_1 u_D, beta = grad h . u].  The momentum
// flux enters negated: its divergence is later summed with grad S in the
// spectral domain, so both reach U_t through one pair of inverse transforms.
// In 2D only the mixed flux -eta u_x u_y is transformed here: the diagonal
// terms reach U_t only through d_x (eta u_x^2) and d_y (eta u_y^2), so the
// inverse pass folds them into S_x = S - eta u_x^2 and S_y = S - eta u_y^2, and
// (U_t)_x gains d_x S_x - d_y (eta u_x u_y), (U_t)_y gains d_y S_y - d_x (eta u_x u_y).
template <int D>
__device__ __forceinline__ double rhs_source(int i, double e, const double (&uc)[D], const double (&hc)[D]) {
    if (i < D) return uc[i];
    if (i < 2 * D) return e * uc[i - D];
    if (i == 2 * D) return e;
    if (i == 2 * D + 1) return -(e * uc[0] * uc[D - 1]);
    double b = hc[0] * uc[0];
    if (D == 2) b += hc[1 % D] * uc[1 % D];
    return b;
}

// Products and forward row transforms of the right-hand side's source fields
// (rhs_source order) in groups of NFG fields; dst.p[i] receives field i.  Each
// block does every group in turn (running the groups side by side in separate
// blocks was measured slower: every group then reloads its inputs).  With
// 256-thread blocks eta, u and beta = grad h . u are read once per point into
// registers before the first group, so each input crosses HBM once; larger
// blocks, whose register budget is smaller, read them again for every group.
// MAXT bounds the workgroup size (256 lets the compiler use more registers).
template <int D, int EPC, int NFG, int MAXT>
__global__ void __launch_bounds__(MAXT, MAXT <= 256 ? 2 : 1) k_rhs_rows_fwd(RowGeom g, const double* __restrict__ eta,
                                                       const double* __restrict__ u, const double* __restrict__ gh,
                                                       PtrList<cpx<double>, MAXF> dst,
                                                       const cpx<double>* __restrict__ tw) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<double>* lds = reinterpret_cast<cpx<double>*>(smem_raw);
    const cpx<double>* twm = tw_size(tw, g.M);
    const RowThread<double> rt = row_thread<double>(g, lds);
    const size_t npts = (size_t)g.nx * g.ny;
    constexpr int NFLD = 2 * D + 3;
    // the inputs of this thread's points: eta, u_c and beta (the last field)
    constexpr bool KEEP = MAXT <= 256;
    constexpr int EK = KEEP ? EPC : 1;
    double ie[EK][2], iu[D][EK][2], ib[EK][2];
    auto load = [&](int e, int s, double& et, double (&uc)[D], double (&hc)[D]) {
        const int j = rt.t + g.TPR * e;
        const bool ok = j < g.M && rt.valid;
        const unsigned o = ok ? rt.y * g.nx + 2 * j : 0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            uc[c] = ok ? at32(u + c * npts, o + s) : 0.0;
            hc[c] = ok ? at32(gh + c * npts, o + s) : 0.0;
        }
        et = ok ? at32(eta, o + s) : 0.0;
    };
    if (KEEP) {
#pragma unroll
        for (int e = 0; e < EK; ++e) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                double uc[D], hc[D];
                load(e, s, ie[e][s], uc, hc);
#pragma unroll
                for (int c = 0; c < D; ++c) iu[c][e][s] = uc[c];
                ib[e][s] = rhs_source<D>(NFLD - 1, ie[e][s], uc, hc);
            }
        }
    }
#pragma unroll
    for (int f0 = 0; f0 < NFLD; f0 += NFG) {
        cpx<double> z[NFG][EPC];
        cpx<double>* H[NFG];
#pragma unroll
        for (int k = 0; k < NFG; ++k) H[k] = (f0 + k < NFLD) ? dst.p[f0 + k] : dst.p[f0];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = rt.t + g.TPR * e;
#pragma unroll
            for (int k = 0; k < NFG; ++k) z[k][e] = C<double>(0, 0);
            if (j < g.M && rt.valid) {
                double v[NFG][2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    double et, uc[D], hc[D];
                    if (KEEP) {
                        const int ek = KEEP ? e : 0;
                        et = ie[ek][s];
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            uc[c] = iu[c][ek][s];
                            hc[c] = 0.0;
                        }
                    } else {
                        load(e, s, et, uc, hc);
                    }
#pragma unroll
                    for (int k = 0; k < NFG; ++k)
                        v[k][s] = KEEP && f0 + k == NFLD - 1 ? ib[KEEP ? e : 0][s] : rhs_source<D>(f0 + k, et, uc, hc);
                }
#pragma unroll
                for (int k = 0; k < NFG; ++k) z[k][e] = C<double>(v[k][0], v[k][1]);
            }
        }
        if (f0 + NFG <= NFLD) {
            row_forward<double, EPC, NFG>(g, rt, z, H, tw, twm, 1.0);
        } else {
            // the last group holds fewer fields: transform them one by one
            for (int k = 0; f0 + k < NFLD; ++k) {
                cpx<double> z1[1][EPC];
                cpx<double>* H1[1] = {H[k]};
#pragma unroll
                for (int e = 0; e < EPC; ++e) z1[0][e] = z[k][e];
                row_forward<double, EPC, 1>(g, rt, z1, H1, tw, twm, 1.0);
            }
        }
    }
}

// The same, a block's rows of one field (blocks [f nblocks, (f + 1) nblocks): field f),
// for launches of less than 512 blocks, which leave most of the chip idle with a row's
// seven fields on the same threads: 256 x 128 13.3 -> 5.9 us, 512 x 512 18.1 -> 12.4.
__global__ void __launch_bounds__(256, 4) k_rhs_rows_fwd_f(RowGeom g, const double* __restrict__ eta,
                                                           const double* __restrict__ u,
                                                           const double* __restrict__ gh,
                                                           PtrList<cpx<double>, MAXF> dst,
                                                           const cpx<double>* __restrict__ tw) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<double>* lds = reinterpret_cast<cpx<double>*>(smem_raw);
    constexpr int EPC = 4;
    const int f = (int)blockIdx.x / g.nblocks;
    const RowThread<double> rt = row_thread_at<double>(g, lds, (int)blockIdx.x - f * g.nblocks, threadIdx.x);
    const size_t npts = (size_t)g.nx * g.ny;
    const bool use_e = f >= 2 && f < 6, use_h = f == 6;
    cpx<double> z[1][EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) {
        const int j = rt.t + g.TPR * i;
        const bool ok = j < g.M && rt.valid;
        const unsigned o = ok ? rt.y * g.nx + 2 * j : 0u;
        double v[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const double e = use_e ? at32(eta, o + s) : 0.0;
            double uc[2] = {0.0, 0.0}, hc[2] = {0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (f != 4) uc[c] = at32(u + c * npts, o + s);
                if (use_h) hc[c] = at32(gh + c * npts, o + s);
            }
            v[s] = ok ? rhs_source<2>(f, e, uc, hc) : 0.0;
        }
        z[0][i] = C<double>(v[0], v[1]);
    }
    cpx<double>* H[1] = {dst.p[f]};
    row_forward<double, EPC, 1>(g, rt, z, H, tw, tw_size(tw, g.M), 1.0);
}

// x-derivatives formed by an inverse row pass: a nonzero f[i] means that field i
// is given as another spectrum (delta's column output, f = 1, or a forward row
// transform, f = 1/nx, the column pass's scale of 1/(nx ny) times the ny of its y
// round trip) whose entry kx is multiplied by i k_x f before the transform (the
// Nyquist entry has no wavenumber), so the column pass writes three outputs fewer.
struct RowDx {
    double f[8];
};

// Inverse row transforms of the derivative fields Q, in the order m =
// div(eta u), delta = div u, d_c delta, d_c beta, d_c eta, one at a time (the next
// one's loads in flight), consumed into the pointwise right-hand side as they arrive: eta_t = -m,
// U_t = -eta grad(eta - h) - T grad h (grad S - div(eta u (x) u) is added later),
// and S, T of Def:bigF accumulated as S = e^3/3 P + e^2 m delta + e m beta +
// e^2/2 Q, T = e^2/2 P + e m delta + m beta + e Q with P = u.grad(delta) -
// delta^2 and Q = u.grad(beta) (the reading u.grad(u.grad h)), so that at most
// four values per point are live.  S's forward row transform goes to Sdst
// (grad S is added to U_t later); in 2D S_x = S - eta u_x^2 goes to Sdst and
// S_y = S - eta u_y^2 to Sydst (see rhs_source).
// dx: fields with dx.f[i] != 0 are given as row spectra (or another field's column
// output) whose x-derivative is wanted (see RowDx).
// The line of 16384 points (D = 1) is one block of 1024 threads of 128 registers, 64 of
// which the accumulated state of 16 points takes: nothing is held or loaded ahead across
// its transforms, where 541 spilled registers cost more than the loads' latency (367 ->
// 207 us).
template <int D, int EPC, int MAXT>
__global__ void __launch_bounds__(MAXT, MAXT <= 256 ? 2 : 1) k_rhs_rows_inv(RowGeom g, PtrList<const cpx<double>, MAXF> src,
                                                       const double* __restrict__ eta, const double* __restrict__ u,
                                                       const double* __restrict__ gh, double* __restrict__ eta_t,
                                                       double* __restrict__ U_t, cpx<double>* __restrict__ Sdst,
                                                       cpx<double>* __restrict__ Sydst,
                                                       const cpx<double>* __restrict__ tw, double scale, RowDx dx,
                                                       double tpx) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<double>* lds = reinterpret_cast<cpx<double>*>(smem_raw);
    const cpx<double>* twm = tw_size(tw, g.M);
    const RowThread<double> rt = row_thread<double>(g, lds);
    const size_t npts = (size_t)g.nx * g.ny;
    constexpr int NQ = 3 * D + 2;
    // live state per point: eta and (m, delta, P) while the first 2 + D fields arrive,
    // then (S, T), in 2D (S_x, S_y, T) once d_c beta is in; d_c eta comes last, when T is
    // complete, so U_t goes straight out
    // (LEAN: (m, delta), then (S, T), and nothing else held or in flight across a
    // transform, see above)
    constexpr bool LEAN = D == 1;
    double A0[EPC][2], A1[EPC][2], A2[LEAN ? 1 : EPC][2], e0[LEAN ? 1 : EPC][2];
    // (the index is opaque: addresses are formed where they are used)
    auto point = [&](int e, bool& ok) -> unsigned {
        int t = rt.t;
        asm volatile("" : "+v"(t));
        const int j = t + g.TPR * e;
        ok = j < g.M && rt.valid;
        return ok ? (unsigned)(rt.y * g.nx + 2 * j) : 0u;
    };
    RowPairs<double, EPC> X;
    if (!LEAN) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            bool ok;
            const unsigned o = point(e, ok);
            e0[LEAN ? 0 : e][0] = at32(eta, o);
            e0[LEAN ? 0 : e][1] = at32(eta, o + 1);
        }
        row_fetch<double, EPC>(g, rt, src.p[0], X);
    }
#pragma unroll 1
    for (int i = 0; i < NQ; ++i) {
        if (LEAN) row_fetch<double, EPC>(g, rt, src.p[i], X);
        row_join<double, EPC>(g, rt, X, rt.lds, tw, dx.f[i], tpx);
        // in flight across the transform: the next field's entries, and the factor
        // this field is consumed with (u_c for d_c delta and d_c beta, (grad h)_c for
        // d_c eta)
        const int c = i < 2 ? 0 : (i - 2) % D;
        if (!LEAN && i + 1 < NQ) row_fetch<double, EPC>(g, rt, src.p[i + 1], X);
        const double* fac = i < 2 ? eta : (i <= 1 + 2 * D ? u : gh) + c * npts;
        double fv[LEAN ? 1 : EPC][2];
        if (!LEAN) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                bool ok;
                const unsigned o = point(e, ok);
                fv[LEAN ? 0 : e][0] = at32(fac, o);
                fv[LEAN ? 0 : e][1] = at32(fac, o + 1);
            }
        }
        auto factor = [&](int e, int s, unsigned o) { return LEAN ? at32(fac, o) : fv[LEAN ? 0 : e][s]; };
        block_lds_barrier();
        cpx<double> z[1][EPC];
        row_inverse_lds<double, EPC, 1>(g, rt, twm, z);
        block_lds_barrier();
        // eta, opaque: its powers are formed where they are used, not held across the
        // loop over the fields
        auto depth = [&](int e, int s, unsigned o) {
            if (LEAN) return at32(eta, o);
            double v = e0[LEAN ? 0 : e][s];
            asm volatile("" : "+v"(v));
            return v;
        };
        // f(e, s, q, o, ok): value q of point e, component s
        auto each = [&](auto&& f) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                __builtin_amdgcn_sched_barrier(0);   // one entry's loads at a time
                bool ok;
                const unsigned o = point(e, ok);
#pragma unroll
                for (int s = 0; s < 2; ++s) f(e, s, scale * (s ? z[0][e].im : z[0][e].re), o + s, ok);
            }
        };
        if (i == 0) {                       // m
            each([&](int e, int s, double q, unsigned o, bool ok) {
                A0[e][s] = q;
                if (ok) at32(eta_t, o) = -q;
            });
        } else if (i == 1) {                // delta
            each([&](int e, int s, double q, unsigned, bool) {
                A1[e][s] = q;
                if (!LEAN) A2[LEAN ? 0 : e][s] = -q * q;
            });
        } else if (i <= 1 + D) {            // d_c delta: P += u_c d_c delta
            if (!LEAN) each([&](int e, int s, double q, unsigned o, bool) { A2[LEAN ? 0 : e][s] += factor(e, s, o) * q; });
            if (i == 1 + D) {               // P complete: fold into S, T
                each([&](int e, int s, double q, unsigned o, bool) {
                    const double et = depth(e, s, o);
                    double bt = 0.0;
#pragma unroll
                    for (int cc = 0; cc < D; ++cc) bt += at32(gh + cc * npts, o) * at32(u + cc * npts, o);
                    const double e2 = et * et, mm = A0[e][s], d0 = A1[e][s];
                    const double pp = LEAN ? -d0 * d0 + factor(e, s, o) * q : A2[LEAN ? 0 : e][s];
                    A0[e][s] = e2 * et / 3.0 * pp + e2 * mm * d0 + et * mm * bt;   // S
                    A1[e][s] = e2 / 2.0 * pp + et * mm * d0 + mm * bt;            // T
                });
            }
        } else if (i <= 1 + 2 * D) {        // d_c beta: Q += u_c d_c beta
            each([&](int e, int s, double q, unsigned o, bool) {
                const double et = depth(e, s, o), t = factor(e, s, o) * q;
                A0[e][s] += et * et / 2.0 * t;
                A1[e][s] += et * t;
            });
            if (D == 2 && i == 1 + 2 * D) {   // S_x, S_y, while u is whole: U_t may be written over it
                each([&](int e, int s, double, unsigned o, bool) {
                    const double et = depth(e, s, o), u0 = at32(u, o), u1 = factor(e, s, o), S = A0[e][s];
                    A0[e][s] = S - et * u0 * u0;
                    A2[LEAN ? 0 : e][s] = S - et * u1 * u1;
                });
            }
        } else {                            // d_c eta: U_t less the flux and grad S
            each([&](int e, int s, double q, unsigned o, bool ok) {
                const double et = LEAN ? at32(eta, o) : e0[LEAN ? 0 : e][s], hx = factor(e, s, o);
                if (ok) at32(U_t + c * npts, o) = -et * (q - hx) - hx * A1[e][s];
            });
        }
    }
    // S (2D: S_x, S_y) forward-transformed, one field at a time (the launch's LDS holds one)
#pragma unroll
    for (int c = 0; c < D; ++c) {
        cpx<double> z1[1][EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const bool ok = rt.t + g.TPR * e < g.M && rt.valid;
            z1[0][e] = !ok ? C<double>(0, 0) : c == 0 ? C<double>(A0[e][0], A0[e][1])
                                           : C<double>(A2[LEAN ? 0 : e][0], A2[LEAN ? 0 : e][1]);
        }
        cpx<double>* H1[1] = {c == 0 ? Sdst : Sydst};
        row_forward<double, EPC, 1>(g, rt, z1, H1, tw, twm, 1.0);
    }
}

// The inverse row pass of the right-hand side (see k_rhs_rows_inv) on 2D grids with rows
// of up to 1024 points, the fields side by side (order m, delta, grad delta, grad eta,
// grad beta): each of eight groups of R TPR threads transforms a field into LDS, then
// every thread forms the right-hand side at one point from the eight values there, and
// the first two groups transform S_x and S_y forward.
// The eight fields one after another on the same threads, with the accumulated state of
// eight points each, took 27 us at 256 x 128 and 32 at 512 x 512; here 8.2 and 15.
// Longer rows (eight entries per thread, one row per block, two batches of four fields
// at 2048 pairs) were slower than one field after another: 514 against 293 us at
// 2048 x 2048, 536 against 367 at 4096 x 1024.
__global__ void __launch_bounds__(1024) k_rhs_rows_inv_f(RowGeom g, PtrList<const cpx<double>, MAXF> src,
                                                         const double* __restrict__ eta, const double* __restrict__ u,
                                                         const double* __restrict__ gh, double* __restrict__ eta_t,
                                                         double* __restrict__ U_t, cpx<double>* __restrict__ Sdst,
                                                         cpx<double>* __restrict__ Sydst,
                                                         const cpx<double>* __restrict__ tw, double scale, RowDx dx,
                                                         double tpx) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<double>* lds = reinterpret_cast<cpx<double>*>(smem_raw);
    constexpr int EPC = 4;   // 8 groups of R M / 4 threads: as many as points
    const cpx<double>* twm = tw_size(tw, g.M);
    const int lgG = g.lgR + g.lgT, G = 1 << lgG, M = g.M;
    const int f = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> lgG);
    const int fs = g.R * (M + 1);
    const RowThread<double> rt = row_thread_at<double>(g, lds + f * fs, blockIdx.x, threadIdx.x & (G - 1));
    RowPairs<double, EPC> X;
    row_fetch<double, EPC>(g, rt, src.p[f], X);
    // this thread's point: value s of pair j of row r, its place in a field's LDS and
    // the inputs there, in flight across the transform
    const size_t npts = (size_t)g.nx * g.ny;
    const int pr = (int)threadIdx.x >> 1, s = threadIdx.x & 1, r = pr >> ilog2(M), j = pr & (M - 1);
    const bool ok = r < g.R && rt.row0 + r < g.ny;
    const unsigned o = ok ? (rt.row0 + r) * g.nx + 2 * j + s : 0u, at = r < g.R ? 2 * (r * (M + 1) + j) + s : 0u;
    const double e = at32(eta, o);
    double uc[2], hc[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        uc[c] = at32(u + c * npts, o);
        hc[c] = at32(gh + c * npts, o);
    }
    row_join<double, EPC>(g, rt, X, rt.lds, tw, dx.f[f], tpx);
    fft_sync(G);
    cpx<double> z[1][EPC];
    row_inverse_lds<double, EPC, 1>(g, rt, twm, z);
    fft_sync(g.TPR);
    cpx<double>* rowb = rt.lds + rt.r * (M + 1);
#pragma unroll
    for (int i = 0; i < EPC; ++i) {
        const int jj = rt.t + g.TPR * i;
        if (jj < M) rowb[jj] = z[0][i];
    }
    block_lds_barrier();
    double q[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = scale * reinterpret_cast<const double*>(lds + k * fs)[at];
    if (ok) {
        const double e2 = e * e, m = q[0], dl = q[1];
        const double bt = hc[0] * uc[0] + hc[1] * uc[1];
        const double P = -dl * dl + uc[0] * q[2] + uc[1] * q[3];   // u.grad(delta) - delta^2
        const double Q = uc[0] * q[6] + uc[1] * q[7];              // u.grad(beta)
        const double S = e2 * e / 3.0 * P + e2 * m * dl + e * m * bt + e2 / 2.0 * Q;
        const double T = e2 / 2.0 * P + e * m * dl + m * bt + e * Q;
        at32(eta_t, o) = -m;
#pragma unroll
        for (int c = 0; c < 2; ++c) at32(U_t + c * npts, o) = -e * (q[4 + c] - hc[c]) - hc[c] * T;
        // this place of the first two fields is read by this thread only
        reinterpret_cast<double*>(lds)[at] = S - e * uc[0] * uc[0];
        reinterpret_cast<double*>(lds + fs)[at] = S - e * uc[1] * uc[1];
    }
    block_lds_barrier();
    if (f < 2) {
#pragma unroll
        for (int i = 0; i < EPC; ++i) {
            const int jj = rt.t + g.TPR * i;
            z[0][i] = jj < M ? rowb[jj] : C<double>(0, 0);
        }
        cpx<double>* H[1] = {f == 0 ? Sdst : Sydst};
        row_forward<double, EPC, 1>(g, rt, z, H, tw, twm, 1.0);
    } else {
        row_forward_idle<EPC>(g);
    }
}

// Linear spectral operators on columns: out_o = sum_i c(code[o][i], k) in_i, with
// y-FFT of the inputs and y-IFFT of the outputs.  Codes: 0 none, 1 identity,
// 2 i kx, 3 i ky, 4 (i kx)^2, 5 (i kx)(i ky), 6 (i ky)^2; every value is also
// multiplied by `scale`.
constexpr int LIN_MAXO = 6;
constexpr int LIN_MAXI = 5;
struct LinCodes {
    int code[LIN_MAXO][LIN_MAXI];
    int no;
};

template <typename T>
__device__ __forceinline__ cpx<T> lin_coef(int code, T kx, T ky) {
    switch (code) {
        case 1: return C<T>(1, 0);
        case 2: return C<T>(0, kx);
        case 3: return C<T>(0, ky);
        case 4: return C<T>(-kx * kx, 0);
        case 5: return C<T>(-kx * ky, 0);
        case 6: return C<T>(-ky * ky, 0);
        default: return C<T>(0, 0);
    }
}

// Inputs loaded (and y-transformed) G fields at a time in lockstep; outputs
// formed and inverse-transformed G at a time.
template <typename T, int EPC, int G>
__device__ __forceinline__ void cols_lin_load(const ColGeom& g, const ColThread<T>& ct,
                                              const PtrList<const cpx<T>, MAXF>& src, int i0,
                                              const cpx<T>* twm, cpx<T> (&vi)[G][EPC]) {
    const cpx<T>* srcs[G];
#pragma unroll
    for (int k = 0; k < G; ++k) srcs[k] = src.p[i0 + k];
    col_load<T, EPC, G>(g, ct, srcs, true, twm, vi);
}

template <typename T, int EPC, int G, int NI>
__device__ __forceinline__ void cols_lin_store(const ColGeom& g, const ColThread<T>& ct,
                                               const PtrList<cpx<T>, MAXF>& dst, const LinCodes& lc, int o0,
                                               const cpx<T> (&in)[NI][EPC], T kx, T tpy, T scale,
                                               const cpx<T>* twm) {
    cpx<T> v[G][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
        const T ky = (g.ny > 1) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
#pragma unroll
        for (int k = 0; k < G; ++k) {
            cpx<T> s = C<T>(0, 0);
#pragma unroll
            for (int i = 0; i < NI; ++i) s = s + lin_coef<T>(lc.code[o0 + k][i], kx, ky) * in[i][e];
            v[k][e] = scale * s;
        }
    }
    cpx<T>* dsts[G];
#pragma unroll
    for (int k = 0; k < G; ++k) dsts[k] = dst.p[o0 + k];
    col_store<T, EPC, G>(g, ct, v, dsts, true, twm);
}

template <typename T, int EPC, int NI, int G>
__global__ void __launch_bounds__(256) k_cols_lin(ColGeom g, PtrList<const cpx<T>, MAXF> src,
                                                   PtrList<cpx<T>, MAXF> dst, LinCodes lc,
                                                   const cpx<T>* __restrict__ tw, T tpx, T tpy,
                                                   T scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    cpx<T> in[NI][EPC];
#pragma unroll
    for (int i0 = 0; i0 < NI; i0 += G) {
        if (i0 + G <= NI) {
            cpx<T> vi[G][EPC];
            cols_lin_load<T, EPC, G>(g, ct, src, i0, twm, vi);
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int e = 0; e < EPC; ++e) in[(i0 + k) % NI][e] = vi[k][e];
        } else {
#pragma unroll
            for (int i = i0; i < NI; ++i) {
                cpx<T> vi[1][EPC];
                cols_lin_load<T, EPC, 1>(g, ct, src, i, twm, vi);
#pragma unroll
                for (int e = 0; e < EPC; ++e) in[i][e] = vi[0][e];
            }
        }
    }
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    int o0 = 0;
    for (; o0 + G <= lc.no; o0 += G) cols_lin_store<T, EPC, G, NI>(g, ct, dst, lc, o0, in, kx, tpy, scale, twm);
    for (; o0 < lc.no; ++o0) cols_lin_store<T, EPC, 1, NI>(g, ct, dst, lc, o0, in, kx, tpy, scale, twm);
}

// Several independent linear column operators in one launch: job k takes
// blocks [k nblocks, (k+1) nblocks).  Each block first issues the loads of all
// its inputs (so their latencies overlap), then transforms them along y one by
// one, forms each output and inverse-transforms and stores it.  The jobs of the
// 2D right-hand side run side by side this way instead of in four launches,
// which keeps four times as many columns in flight.
constexpr int LINJ_MAXI = 4;
constexpr int LINJ_MAXO = 3;
constexpr int LINJ_MAXJ = 4;
template <typename T>
struct LinJob {
    const cpx<T>* src[LINJ_MAXI];
    cpx<T>* dst[LINJ_MAXO];
    int ni, no;
    int code[LINJ_MAXO][LINJ_MAXI];
    int kin[LINJ_MAXI], kout[LINJ_MAXO];   // series kinds of a wall job (bit 0: sine along x, bit 1: along y)
};
template <typename T>
struct LinJobs {
    LinJob<T> j[LINJ_MAXJ];
    int n;
};

// NF register columns of a block through one y-FFT in lockstep (shared barriers).
template <typename T, int EPC, int NF>
__device__ __forceinline__ void col_fft_group(const ColGeom& g, const ColThread<T>& ct, const cpx<T>* twm,
                                              cpx<T> (*v)[EPC], bool inverse) {
    reg_fft<T, EPC, NF>(v, ct.buf, ct.fstride, g.ny, ct.t, g.TPC, twm, inverse);
    fft_sync(g.TPC);
}

// The first nf (1..3) register columns of v through one lockstep y-FFT.
template <typename T, int EPC, int NMAX>
__device__ __forceinline__ void col_fft_first(const ColGeom& g, const ColThread<T>& ct, const cpx<T>* twm,
                                              cpx<T> (&v)[NMAX][EPC], int nf, bool inverse) {
    if (nf == 1) col_fft_group<T, EPC, 1>(g, ct, twm, v, inverse);
    else if (nf == 2 || NMAX < 3) col_fft_group<T, EPC, (NMAX < 2 ? NMAX : 2)>(g, ct, twm, v, inverse);
    else col_fft_group<T, EPC, (NMAX < 3 ? NMAX : 3)>(g, ct, twm, v, inverse);
}

// LK: columns per lockstep transform, 3 (LDS holds three columns per block) or 1
// (one at a time, for columns of 2048 where three would leave one block per CU).
template <typename T, int EPC, int NI, int LK>
__global__ void __launch_bounds__(256, COL_WAVES<EPC>) k_cols_lin_jobs(ColGeom g, LinJobs<T> jobs, const cpx<T>* __restrict__ tw,
                                                        T tpx, T tpy, T scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const int jb = blockIdx.x / g.nblocks;
    if (jb >= jobs.n) return;
    const LinJob<T>& J = jobs.j[jb];
    constexpr int NL = LK == 1 ? 1 : (NI < 3 ? NI : 3);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread_at<T>(g, lds, (int)blockIdx.x - jb * g.nblocks);
    const int ny = g.ny;
    cpx<T> in[NI][EPC];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
            in[i][e] = (i < J.ni && ct.valid && j < ny) ? at32(J.src[i], ct.kx * ny + j) : C<T>(0, 0);
        }
    }
    if (ny > 1 && LK == 1) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (i < J.ni) col_fft_group<T, EPC, 1>(g, ct, twm, in + i, false);
    } else if (ny > 1) {
        // the inputs in groups of up to three sharing their transform's barriers
        if (NI <= 3 || J.ni <= 3) {
            col_fft_first<T, EPC, NI>(g, ct, twm, in, J.ni, false);
        } else {
            col_fft_first<T, EPC, NI>(g, ct, twm, in, 3, false);
            col_fft_group<T, EPC, 1>(g, ct, twm, in + 3, false);
        }
    }
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    cpx<T> out[LINJ_MAXO][EPC];
#pragma unroll
    for (int o = 0; o < LINJ_MAXO; ++o) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
            const T ky = (ny > 1) ? wavenumber<T>(j, ny, tpy) : (T)0;
            cpx<T> s = C<T>(0, 0);
            if (o < J.no) {
#pragma unroll
                for (int i = 0; i < NI; ++i) s = s + lin_coef<T>(J.code[o][i], kx, ky) * in[i][e];
            }
            out[o][e] = scale * s;
        }
    }
    if (ny > 1 && LK == 1) {
#pragma unroll
        for (int o = 0; o < LINJ_MAXO; ++o)
            if (o < J.no) col_fft_group<T, EPC, 1>(g, ct, twm, out + o, true);
    } else if (ny > 1) {
        col_fft_first<T, EPC, LINJ_MAXO>(g, ct, twm, out, J.no, true);
    }
    if (ct.valid) {
#pragma unroll
        for (int o = 0; o < LINJ_MAXO; ++o) {
            if (o >= J.no) break;
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const int j = ct.t + g.TPC * e;
                if (j < ny) at32(J.dst[o], ct.kx * ny + j) = out[o][e];
            }
        }
    }
}

// A^{-1} on D spectral columns: y-FFT, per-mode A^{-1} (times scale), y-IFFT.
template <typename T, int EPC, int D>
__global__ void __launch_bounds__(256) k_cols_precond(ColGeom g, PtrList<const cpx<T>, MAXF> src,
                                                       PtrList<cpx<T>, MAXF> dst,
                                                       const cpx<T>* __restrict__ tw, T tpx, T tpy,
                                                       T sig, T alp, T scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    cpx<T> in[D][EPC];
    const cpx<T>* srcs[D];
    cpx<T>* dsts[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        srcs[c] = src.p[c];
        dsts[c] = dst.p[c];
    }
    col_load<T, EPC, D>(g, ct, srcs, true, twm, in);
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    cpx<T> out[D][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
        const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
        cpx<T> r[D], z[D];
#pragma unroll
        for (int c = 0; c < D; ++c) r[c] = in[c][e];
        precond_mode<T, D>(kx, ky, sig, alp, r, z);
#pragma unroll
        for (int c = 0; c < D; ++c) out[c][e] = scale * z[c];
    }
    col_store<T, EPC, D>(g, ct, out, dsts, true, twm);
}

// ---------------------------------------------------------------------------
// Krylov solve kernels (PCG of section 3.2 with the state x, r, p, q kept in
// the S layout; dot products by Parseval over the half spectrum, in FP64).
// One iteration is C1 -> R1 -> C2:
//   C1: reduce the previous update's (r.z, r.r) -> stop test, beta;
//       z = A^{-1} r, p = z + beta p; emits (p, div p) / (nx ny) and the y-IFFT
//   R1: x-IFFT -> pointwise  a = eta p + grad h (eta^2/2 div p + eta grad h.p),
//                            w = eta^3/3 div p + eta^2/2 grad h.p  -> x-FFT;
//       partial p.Gp as the grid sum of the weak form B[p, p] (section 3.1),
//       sum_x (p, div p)^T M(x) (p, div p) with M of Appendix A
//   C2: reduce p.Gp -> alpha; y-FFT; q = a - i k w (= G p, Def:G);
//       x += alpha p, r -= alpha q, z = A^{-1} r; partial r.z, r.r
// p.Gp equals B[p, p] exactly for the spectral D (real antisymmetric), so the
// curvature is known before q is formed and the update needs no extra pass.
// Every kernel returns at once when the solve is done.
// ---------------------------------------------------------------------------

// The scalars a column pass reads, in one batch of scalar loads.
struct PcgScal {
    double rho, rho_prev, bb, tol2, sig, alp, inv_n;
    int iter, max_iter, done, first, init_bb;
};
__device__ __forceinline__ PcgScal pcg_scalars(const SolveScal* sc) {
    return PcgScal{sc->rho,  sc->rho_prev, sc->bb,   sc->tol2,  sc->sig,    sc->alp,
                   sc->inv_n, sc->iter,     sc->max_iter, sc->done, sc->first, sc->init_bb};
}

// Stop test and beta from the sums (r.z, r.r) of the last update pass (or of the
// initial residual).  Identical in every block; block 0 publishes.  Returns done.
__device__ __forceinline__ bool pcg_iterate_state(SolveScal* __restrict__ sc, const PcgScal& s, const double (&tot)[2],
                                                  double& beta_out) {
    const double rz = tot[0] * s.inv_n;
    const double rr = tot[1] * s.inv_n;
    // init_bb: ||b||^2 is the first r.r seen (r_0 = b); taken once, while bb is unset
    const double bb = (s.init_bb && s.first && s.iter == 0 && s.bb == 0.0) ? rr : s.bb;
    const bool bad = !(rr == rr) || !(rz == rz) || !(rr <= 1.0e300);
    const bool conv = !bad && (bb == 0.0 || rr <= s.tol2 * bb);
    const bool done = bad || conv || s.iter >= s.max_iter;
    const double beta = s.first ? 0.0 : rz / s.rho_prev;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->rr = rr;
        sc->bb = bb;
        sc->relres = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        sc->rho = rz;
        sc->beta = beta;
        sc->converged = conv ? 1 : 0;
        if (bad) sc->status = -2;
        sc->done = done ? 1 : 0;
    }
    beta_out = beta;
    return done;
}

// C1_UPDATE: the PCG step (p = z + beta p); C1_COPY: p = xsrc (apply G to a
// given field); C1_ACCUM: x += dx (FP32 correction of a refinement step,
// x in ph) and p = x, so the pass that starts the FP64 residual also applies
// the correction.
enum { C1_UPDATE = 0, C1_COPY = 1, C1_ACCUM = 2 };

// FEW: blocks of 128 threads (see k_pcg_c2).
template <typename T, int EPC, int D, int MODE, bool FEW = false>
__global__ void __launch_bounds__(256, FEW ? 2 : COL_WAVES<EPC>) k_pcg_c1(ColGeom g, const cpx<T>* __restrict__ tw,
                                                 SolveScal* __restrict__ sc, const double* __restrict__ part,
                                                 int nb3, const cpx<T>* __restrict__ rh, cpx<T>* __restrict__ ph,
                                                 const cpx<T>* __restrict__ xsrc, cpx<T>* __restrict__ H,
                                                 size_t NS, T tpx, T tpy, const cpx<float>* __restrict__ dx) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    __shared__ double red[32];
    const PcgScal s0 = pcg_scalars(sc);
    if (s0.done) return;
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    // the partials, r and the last p, in flight across the reduction
    constexpr int V = FEW ? 2 : 1;
    double pb[PF_K * V][2];
    cpx<T> in[D][EPC], last[D][EPC];
    if (MODE == C1_UPDATE) {
        partials_fetch<2, V>(part + PART_C3, nb3, pb);
        __builtin_amdgcn_sched_barrier(0);
    }
    const cpx<T>* src = MODE == C1_UPDATE ? rh : MODE == C1_COPY ? xsrc : ph;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        bool ok;
        const unsigned idx = col_index(g, ct, ct.t + g.TPC * e, ok);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            in[c][e] = at32(src + c * NS, idx);
            if (MODE == C1_UPDATE) last[c][e] = at32(ph + c * NS, idx);
            if (MODE == C1_ACCUM) {
                const cpx<float> x = at32(dx + c * NS, idx);
                last[c][e] = C<T>((T)x.re, (T)x.im);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    double beta_d = 0.0;
    if (MODE == C1_UPDATE) {
        double tot[2];
        partials_sum<2, V>(part + PART_C3, nb3, pb, tot, red);
        if (pcg_iterate_state(sc, s0, tot, beta_d)) return;
    }
    const T beta = (T)beta_d, sig = (T)s0.sig, alp = (T)s0.alp, inv_n = (T)s0.inv_n;
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    cpx<T> o[D + 1][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
        const bool ok = ct.valid && j < g.ny;
        const unsigned idx = ok ? (unsigned)(ct.kx * g.ny + j) : 0u;
        const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
        cpx<T> p[D];
        if (MODE == C1_UPDATE) {
            cpx<T> r[D], z[D];
#pragma unroll
            for (int c = 0; c < D; ++c) r[c] = in[c][e];
            precond_mode<T, D>(kx, ky, sig, alp, r, z);
            // beta = 0 on the first iteration: p = z, the unset direction is not used
#pragma unroll
            for (int c = 0; c < D; ++c) p[c] = (beta != (T)0) ? z[c] + beta * last[c][e] : z[c];
        } else {
#pragma unroll
            for (int c = 0; c < D; ++c) p[c] = MODE == C1_ACCUM ? in[c][e] + last[c][e] : in[c][e];
        }
        if (MODE != C1_COPY && ok) {
#pragma unroll
            for (int c = 0; c < D; ++c) at32(ph + c * NS, idx) = p[c];
        }
        cpx<T> dv = ik(kx, p[0]);
        if (D == 2) dv = dv + ik(ky, p[1 % D]);
#pragma unroll
        for (int c = 0; c < D; ++c) o[c][e] = inv_n * p[c];
        o[D][e] = inv_n * dv;
    }
    cpx<T>* dsts[D + 1];
#pragma unroll
    for (int c = 0; c <= D; ++c) dsts[c] = H + c * NS;
    col_store<T, EPC, D + 1>(g, ct, o, dsts, true, twm);
}

// Stop test only (one block): closes a chunk of iterations so the host can
// read the done flag.  Idempotent with the C1 that follows.  With pub set,
// thread 0 then publishes the loop flags as k_publish_flags does.
__device__ __forceinline__ void publish_flags(const SolveScal* sc, int* d, int seq) {
    const int v[8] = {sc->iter, sc->max_iter, sc->done, sc->converged, sc->flat, sc->status, seq, sc->outer};
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i != 6) __hip_atomic_store(d + i, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the values are there before seq
    __hip_atomic_store(d + 6, v[6], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void inner_close(SolveScal* s, const SolveScal* d);
// With inner set (the FP32 inner solve of a refinement step that has just
// ended), thread 0 first adds that step to the counters (see inner_close).
__global__ void __launch_bounds__(256) k_pcg_check(SolveScal* __restrict__ sc, const double* __restrict__ part,
                                                   int nb3, int* pub, int seq, const SolveScal* __restrict__ inner) {
    if (inner) {
        if (threadIdx.x == 0) inner_close(sc, inner);
        __syncthreads();
    }
    const PcgScal s0 = pcg_scalars(sc);
    if (!s0.done) {
        __shared__ double red[32];
        double beta, pb[PF_K][2], tot[2];
        partials_fetch<2>(part + PART_C3, nb3, pb);
        partials_sum<2>(part + PART_C3, nb3, pb, tot, red);
        pcg_iterate_state(sc, s0, tot, beta);
    }
    // block 0 thread 0 wrote the scalars above and reads them back here
    if (pub && blockIdx.x == 0 && threadIdx.x == 0) publish_flags(sc, pub, seq);
}

// Publish iter, max_iter, done, converged, flat, status of a solve into host
// memory (d: device address of a host-coherent pinned buffer), then the
// sequence number seq in d[6].  System-scope stores: the values go out together, and
// seq once all of them have completed, so a host that sees seq also sees the values
// (no cache-wide fence needed for one thread's stores; one completed store after
// another made the check kernel take 7.1 us, 4.0 so).
__global__ void k_publish_flags(const SolveScal* __restrict__ sc, int* d, int seq) {
    if (threadIdx.x == 0 && blockIdx.x == 0) publish_flags(sc, d, seq);
}

// Row pass R1 on rows above 1024 points: a block's fields one after another, the next
// one's loads in flight meanwhile (three fields of LDS do not fit).
template <typename T, int EPC, int D, int MAXT>
__global__ void __launch_bounds__(MAXT) k_pcg_r1(RowGeom g, const cpx<T>* __restrict__ tw,
                                                 SolveScal* __restrict__ sc, cpx<T>* H, size_t NS,
                                                 const T* __restrict__ eta, const T* __restrict__ gh,
                                                 double* __restrict__ part) {
    if (sc->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    __shared__ double red[16];
    const cpx<T>* twm = tw_size(tw, g.M);
    const RowThread<T> rt = row_thread<T>(g, lds);
    double acc[1] = {0.0};
    cpx<T> v[D + 1][EPC];
    RowPairs<T, EPC> X;
    row_fetch<T, EPC>(g, rt, H, X);
#pragma unroll
    for (int c = 0; c <= D; ++c) {
        row_join<T, EPC>(g, rt, X, rt.lds, tw);
        if (c < D) row_fetch<T, EPC>(g, rt, H + (c + 1) * NS, X);
        block_lds_barrier();
        row_inverse_lds<T, EPC, 1>(g, rt, twm, v + c);
        block_lds_barrier();
    }
    const size_t npts = (size_t)g.nx * g.ny;
    const T third = (T)1 / (T)3, half = (T)0.5;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        if (j < g.M && rt.valid) {
            const unsigned o = rt.y * g.nx + 2 * j;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const T et = at32(eta, o + s);
                T hc[D], pc[D];
                T bt = 0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    hc[c] = at32(gh + c * npts, o + s);
                    pc[c] = s ? v[c][e].im : v[c][e].re;
                    bt += hc[c] * pc[c];
                }
                const T dl = s ? v[D][e].im : v[D][e].re;
                const T e2 = et * et;
                const T w1 = third * e2 * et * dl + half * e2 * bt;
                const T w2 = half * e2 * dl + et * bt;
                // B-density: eta |p|^2 + eta^3/3 dl^2 + eta^2 dl bt + eta bt^2 = p.a + dl w1
                double pp = 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) pp += (double)pc[c] * (double)pc[c];
                acc[0] += (double)et * pp + (double)dl * (double)w1 + (double)bt * (double)w2;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T a = et * pc[c] + hc[c] * w2;
                    if (s) v[c][e].im = a; else v[c][e].re = a;
                }
                if (s) v[D][e].im = w1; else v[D][e].re = w1;
            }
        }
    }
#pragma unroll
    for (int c = 0; c <= D; ++c) {
        cpx<T>* Hc[1] = {H + c * NS};
        cpx<T> vc[1][EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) vc[0][e] = v[c][e];
        row_forward<T, EPC, 1>(g, rt, vc, Hc, tw, twm, (T)1);
    }
    if (part) {
        block_sum<1>(acc, red);
        if (threadIdx.x == 0) part[PART_C2 + blockIdx.x] = acc[0];
    }
}

// Row pass R1 on shorter rows: each of the D + 1 fields has R TPR threads of its own
// (whole waves), which transform it, exchange the values with the other fields'
// through LDS and form that field's row of M(x).  Against all fields in lockstep on
// the same threads, three times the waves on a third of the serial work each
// (FP64 256 x 128 12.0 -> 8.0 us, 512 x 512 15.2 -> 13.7, FP32 512 x 512 7.4 -> 6.5).
template <typename T, int D>
__global__ void __launch_bounds__((D + 1) * 256) k_pcg_r1f(RowGeom g, const cpx<T>* __restrict__ tw,
                                                           SolveScal* __restrict__ sc, cpx<T>* H, size_t NS,
                                                           const T* __restrict__ eta, const T* __restrict__ gh,
                                                           double* __restrict__ part) {
    if (sc->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    __shared__ double red[16];
    constexpr int EPC = 4;
    const cpx<T>* twm = tw_size(tw, g.M);
    const int lgG = g.lgR + g.lgT, G = 1 << lgG;
    const int f = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> lgG);
    const int fs = g.R * (g.M + 1);
    const RowThread<T> rt = row_thread_at<T>(g, lds + f * fs, blockIdx.x, threadIdx.x & (G - 1));
    cpx<T>* Hf = H + f * NS;
    RowPairs<T, EPC> X;
    row_fetch<T, EPC>(g, rt, Hf, X);
    // eta and grad h at this thread's points, in flight across the transform
    const size_t npts = (size_t)g.nx * g.ny;
    cpx<T> et2[EPC], hc2[D][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        const unsigned o = (j < g.M && rt.valid) ? rt.y * g.nx + 2 * j : 0u;
        et2[e] = C<T>(at32(eta, o), at32(eta, o + 1));
#pragma unroll
        for (int c = 0; c < D; ++c) hc2[c][e] = C<T>(at32(gh + c * npts, o), at32(gh + c * npts, o + 1));
    }
    row_join<T, EPC>(g, rt, X, rt.lds, tw);
    fft_sync(G);
    cpx<T> z[1][EPC];
    row_inverse_lds<T, EPC, 1>(g, rt, twm, z);
    fft_sync(g.TPR);
    cpx<T>* rowb = lds + rt.r * (g.M + 1);   // this row of field 0
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        if (j < g.M) rowb[f * fs + j] = z[0][e];
    }
    block_lds_barrier();
    double acc[1] = {0.0};
    const T third = (T)1 / (T)3, half = (T)0.5;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = rt.t + g.TPR * e;
        if (j < g.M && rt.valid) {
            cpx<T> p[D + 1];
#pragma unroll
            for (int c = 0; c <= D; ++c) p[c] = rowb[c * fs + j];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const T et = s ? et2[e].im : et2[e].re;
                T hf = 0, pf = 0, bt = 0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T hc = s ? hc2[c][e].im : hc2[c][e].re, pc = s ? p[c].im : p[c].re;
                    bt += hc * pc;
                    if (c == f) {
                        hf = hc;
                        pf = pc;
                    }
                }
                const T dl = s ? p[D].im : p[D].re;
                const T e2 = et * et;
                const T w1 = third * e2 * et * dl + half * e2 * bt;
                const T w2 = half * e2 * dl + et * bt;
                // B-density: eta |p|^2 + eta^3/3 dl^2 + eta^2 dl bt + eta bt^2 = p.a + dl w1
                acc[0] += f < D ? (double)et * ((double)pf * (double)pf)
                                : (double)dl * (double)w1 + (double)bt * (double)w2;
                const T out = f < D ? et * pf + hf * w2 : w1;
                if (s) z[0][e].im = out; else z[0][e].re = out;
            }
        }
    }
    block_lds_barrier();   // the other fields' threads have read this field's values
    cpx<T>* Hc[1] = {Hf};
    row_forward<T, EPC, 1>(g, rt, z, Hc, tw, twm, (T)1);
    if (part) {
        block_sum<1>(acc, red);
        if (threadIdx.x == 0) part[PART_C2 + blockIdx.x] = acc[0];
    }
}

// Row pass R1 of the line of 16384 points (M = 8192 = 64 x 128), which fits one
// workgroup only with its registers spilled and keeps one compute unit busy (88 us
// against 11.6 for these three launches): in place over 64 waves, as 64-point transforms of the columns
// k = 128 a + b of the spectrum (k_pcg_long_cols<true>: real split, then over a), the
// 128-point transforms of the rows c (k_pcg_long_rows, with the pointwise operator) at
// the pairs j = c + 64 d, and the way back (k_pcg_long_cols<false>).
//   z_{c + 64 d} = sum_b W_128^{-db} W_M^{-cb} sum_a Z_{128 a + b} W_64^{-ac}.
// A block of one wave takes both fields of column b and of the column of its mirrored
// entries, 128 - b (0 and 64 together), 16 threads each.
constexpr int LONG_M = 8192, LONG_A = 64, LONG_B = 128;
template <typename T, bool INV>
__global__ void __launch_bounds__(64) k_pcg_long_cols(const cpx<T>* __restrict__ tw,
                                                      const SolveScal* __restrict__ sc, cpx<T>* H, size_t NS) {
    if (sc->done) return;
    __shared__ cpx<T> lds[4 * LONG_A];
    const int col = threadIdx.x >> 4, t = threadIdx.x & 15, s = col & 1, u = blockIdx.x;
    const int b = s == 0 ? u : (u == 0 ? LONG_B / 2 : LONG_B - u);
    cpx<T>* Hf = H + (col >> 1) * NS;
    const cpx<T>* tw2 = tw_size(tw, 2 * LONG_M);
    const cpx<T>* twM = tw_size(tw, LONG_M);
    const cpx<T>* twA = tw_size(tw, LONG_A);
    cpx<T>* buf = lds + col * LONG_A;
    cpx<T> v[1][4], w[4], wc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        w[e] = tw2[LONG_B * (t + 16 * e) + b];
        wc[e] = twM[(t + 16 * e) * b];
    }
    if (INV) {
        cpx<T> xm[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = LONG_B * (t + 16 * e) + b;
            v[0][e] = Hf[k];
            xm[e] = Hf[LONG_M - k];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const cpx<T> xk = v[0][e];
            if (e == 0 && t == 0 && b == 0) {
                v[0][e] = C<T>(xk.re + xm[e].re, xk.re - xm[e].re);
            } else {
                cpx<T> zm;
                split_join(xk, xm[e], w[e], v[0][e], zm);
            }
        }
        reg_fft<T, 4, 1>(v, buf, 0, LONG_A, t, 16, twA, true);
#pragma unroll
        for (int e = 0; e < 4; ++e) Hf[LONG_B * (t + 16 * e) + b] = v[0][e] * cj(wc[e]);
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[0][e] = Hf[LONG_B * (t + 16 * e) + b] * wc[e];
    reg_fft<T, 4, 1>(v, buf, 0, LONG_A, t, 16, twA, false);
    fft_sync(16);
#pragma unroll
    for (int e = 0; e < 4; ++e) buf[t + 16 * e] = v[0][e];
    fft_sync(16);
    const cpx<T>* mir = u == 0 ? buf : lds + (col ^ 1) * LONG_A;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int a = t + 16 * e, k = LONG_B * a + b;
        const cpx<T> zk = v[0][e];
        if (k == 0) {
            Hf[0] = C<T>(zk.re + zk.im, 0);
            Hf[LONG_M] = C<T>(zk.re - zk.im, 0);
        } else {
            cpx<T> xk, xm;
            split_part(zk, mir[b == 0 ? LONG_A - a : LONG_A - 1 - a], w[e], xk, xm);
            Hf[k] = xk;
        }
    }
}
// Rows c of the line of 16384 points: one wave per row, 32 threads per field; the
// pointwise operator as in k_pcg_r1f.
template <typename T>
__global__ void __launch_bounds__(64) k_pcg_long_rows(const cpx<T>* __restrict__ tw,
                                                      const SolveScal* __restrict__ sc, cpx<T>* H, size_t NS,
                                                      const T* __restrict__ eta, const T* __restrict__ gh,
                                                      double* __restrict__ part) {
    if (sc->done) return;
    __shared__ cpx<T> lds[2 * LONG_B];
    __shared__ double red[16];
    const int f = threadIdx.x >> 5, t = threadIdx.x & 31, c = blockIdx.x;
    cpx<T>* row = H + f * NS + LONG_B * c;
    const cpx<T>* twB = tw_size(tw, LONG_B);
    cpx<T> v[1][4], et2[4], h2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[0][e] = row[t + 32 * e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int o = 2 * (c + LONG_A * (t + 32 * e));
        et2[e] = C<T>(eta[o], eta[o + 1]);
        h2[e] = C<T>(gh[o], gh[o + 1]);
    }
    cpx<T>* buf = lds + f * LONG_B;
    reg_fft<T, 4, 1>(v, buf, 0, LONG_B, t, 32, twB, true);
    fft_sync(32);
#pragma unroll
    for (int e = 0; e < 4; ++e) buf[t + 32 * e] = v[0][e];
    fft_sync(32);
    double acc[1] = {0.0};
    const T third = (T)1 / (T)3, half = (T)0.5;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const cpx<T> p2 = lds[t + 32 * e], d2 = lds[LONG_B + t + 32 * e];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const T et = s ? et2[e].im : et2[e].re, h = s ? h2[e].im : h2[e].re;
            const T p = s ? p2.im : p2.re, dl = s ? d2.im : d2.re;
            const T bt = h * p, e2 = et * et;
            const T w1 = third * e2 * et * dl + half * e2 * bt;
            const T w2 = half * e2 * dl + et * bt;
            acc[0] += f == 0 ? (double)et * ((double)p * (double)p) : (double)dl * (double)w1 + (double)bt * (double)w2;
            const T out = f == 0 ? et * p + h * w2 : w1;
            if (s) v[0][e].im = out; else v[0][e].re = out;
        }
    }
    reg_fft<T, 4, 1>(v, buf, 0, LONG_B, t, 32, twB, false);
#pragma unroll
    for (int e = 0; e < 4; ++e) row[t + 32 * e] = v[0][e];
    if (part) {
        block_sum<1>(acc, red);
        if (threadIdx.x == 0) part[PART_C2 + c] = acc[0];
    }
}

// The iteration on that line with the column passes fused in (three launches instead of
// five): k_pcg_long_c1 is k_pcg_c1's update (mode C1_UPDATE) and k_pcg_long_cols<true>,
// k_pcg_long_c2 is k_pcg_long_cols<false> and k_pcg_c2's update (C2_UPDATE).  A mode's
// two fields are in one wave, so what the passes exchanged through memory goes through
// LDS.  20 -> 15.4 us per iteration.
struct LongCol {
    int col, t, s, f, u, b;
    bool edge;   // the thread of modes 0 and M
};
__device__ __forceinline__ LongCol long_col(int lane, int u) {
    LongCol c;
    c.col = lane >> 4;
    c.t = lane & 15;
    c.s = c.col & 1;
    c.f = c.col >> 1;
    c.u = u;
    c.b = c.s == 0 ? u : (u == 0 ? LONG_B / 2 : LONG_B - u);
    c.edge = u == 0 && c.s == 0 && c.t == 0;
    return c;
}
template <typename T>
__global__ void __launch_bounds__(64) k_pcg_long_c1(const cpx<T>* __restrict__ tw, SolveScal* __restrict__ sc,
                                                    const double* __restrict__ part, int nb3,
                                                    const cpx<T>* __restrict__ rh, cpx<T>* __restrict__ ph,
                                                    cpx<T>* __restrict__ H, size_t NS, T tpx) {
    __shared__ cpx<T> lds[4 * LONG_A];
    __shared__ double red[32];
    const PcgScal s0 = pcg_scalars(sc);
    if (s0.done) return;
    const LongCol c = long_col(threadIdx.x, blockIdx.x);
    constexpr int NX = 2 * LONG_M;
    const cpx<T>* tw2 = tw_size(tw, NX);
    const cpx<T>* twM = tw_size(tw, LONG_M);
    double pb[PF_K][2], tot[2], beta_d;
    partials_fetch<2>(part + PART_C3, nb3, pb);
    __builtin_amdgcn_sched_barrier(0);
    cpx<T> r[5], last[5], w[4], wc[4];   // modes 128 a + b, a = t + 16 e; entry 4: mode M
#pragma unroll
    for (int e = 0; e < 5; ++e) {
        const int k = e < 4 ? LONG_B * (c.t + 16 * e) + c.b : (c.edge ? LONG_M : 0);
        r[e] = rh[k];
        last[e] = ph[k];
        if (e < 4) {
            w[e] = tw2[k];
            wc[e] = twM[(c.t + 16 * e) * c.b];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    partials_sum<2>(part + PART_C3, nb3, pb, tot, red);
    if (pcg_iterate_state(sc, s0, tot, beta_d)) return;
    const T beta = (T)beta_d, sig = (T)s0.sig, alp = (T)s0.alp, inv_n = (T)s0.inv_n;
    cpx<T>* buf = lds + c.col * LONG_A;
    cpx<T> p[5], v[1][4];
#pragma unroll
    for (int e = 0; e < 5; ++e) {
        const int k = e < 4 ? LONG_B * (c.t + 16 * e) + c.b : LONG_M;
        const cpx<T> ri[1] = {r[e]};
        cpx<T> z[1];
        precond_mode<T, 1>(wavenumber<T>(k, NX, tpx), (T)0, sig, alp, ri, z);
        // beta = 0 on the first iteration: p = z, the unset direction is not used
        p[e] = (beta != (T)0) ? z[0] + beta * last[e] : z[0];
        if (c.f == 0 && (e < 4 || c.edge)) ph[k] = p[e];
        if (e < 4) buf[c.t + 16 * e] = p[e];
    }
    fft_sync(16);
    const cpx<T>* mir = c.u == 0 ? buf : lds + (c.col ^ 1) * LONG_A;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int a = c.t + 16 * e, k = LONG_B * a + c.b;
        const bool zero = k == 0;
        cpx<T> xk = inv_n * p[e];
        cpx<T> pm = mir[c.b == 0 ? (LONG_A - a) & (LONG_A - 1) : LONG_A - 1 - a];
        pm.re = zero ? p[4].re : pm.re;
        pm.im = zero ? p[4].im : pm.im;
        cpx<T> xm = inv_n * pm;
        if (c.f) {   // div p
            xk = ik(wavenumber<T>(k, NX, tpx), xk);
            xm = ik(wavenumber<T>(LONG_M - k, NX, tpx), xm);
        }
        cpx<T> zm;
        split_join(xk, xm, w[e], v[0][e], zm);
        if (zero) v[0][e] = C<T>(xk.re + xm.re, xk.re - xm.re);
    }
    reg_fft<T, 4, 1>(v, buf, 0, LONG_A, c.t, 16, tw_size(tw, LONG_A), true);
    cpx<T>* Hf = H + c.f * NS;
#pragma unroll
    for (int e = 0; e < 4; ++e) Hf[LONG_B * (c.t + 16 * e) + c.b] = v[0][e] * cj(wc[e]);
}
// 32 blocks of two waves: as many partials as the column launches of this line write
// less one, whose place the first block clears.
template <typename T>
__global__ void __launch_bounds__(128) k_pcg_long_c2(const cpx<T>* __restrict__ tw, SolveScal* __restrict__ sc,
                                                     const cpx<T>* __restrict__ H, size_t NS,
                                                     const cpx<T>* __restrict__ ph, cpx<T>* __restrict__ xh,
                                                     cpx<T>* __restrict__ rh, double* __restrict__ part, int nb_r1,
                                                     int nb3, T tpx) {
    __shared__ cpx<T> ldsb[2][4 * LONG_A];
    __shared__ double red[64];
    const PcgScal s0 = pcg_scalars(sc);
    if (s0.done) return;
    const int wv = threadIdx.x >> 6;
    const LongCol c = long_col(threadIdx.x & 63, 2 * blockIdx.x + wv);
    constexpr int NX = 2 * LONG_M;
    const cpx<T>* tw2 = tw_size(tw, NX);
    const cpx<T>* twM = tw_size(tw, LONG_M);
    const cpx<T>* Hf = H + c.f * NS;
    double pb[PF_K][1], tot[1];
    partials_fetch<1>(part + PART_C2, nb_r1, pb);
    __builtin_amdgcn_sched_barrier(0);
    cpx<T> v[1][4], w[4], wc[4], x[5], p[5], r[5];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = LONG_B * (c.t + 16 * e) + c.b;
        v[0][e] = Hf[k];
        wc[e] = twM[(c.t + 16 * e) * c.b];
        w[e] = tw2[k];
    }
#pragma unroll
    for (int e = 0; e < 5; ++e) {
        const int k = e < 4 ? LONG_B * (c.t + 16 * e) + c.b : (c.edge ? LONG_M : 0);
        x[e] = xh[k];
        p[e] = ph[k];
        r[e] = rh[k];
    }
    __builtin_amdgcn_sched_barrier(0);
    partials_sum<1>(part + PART_C2, nb_r1, pb, tot, red);
    const double a_d = s0.rho / tot[0];
    const T alpha = (T)a_d, sig = (T)s0.sig, alp = (T)s0.alp;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->pq = tot[0];
        sc->alpha = a_d;
        sc->rho_prev = s0.rho;
        sc->iter = s0.iter + 1;
        sc->first = 0;
    }
    cpx<T>* lds = ldsb[wv];
    cpx<T>* buf = lds + c.col * LONG_A;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[0][e] = v[0][e] * wc[e];
    reg_fft<T, 4, 1>(v, buf, 0, LONG_A, c.t, 16, tw_size(tw, LONG_A), false);
    fft_sync(16);
#pragma unroll
    for (int e = 0; e < 4; ++e) buf[c.t + 16 * e] = v[0][e];
    fft_sync(16);
    const cpx<T>* mir = c.u == 0 ? buf : lds + (c.col ^ 1) * LONG_A;
    cpx<T> X[5];   // this field's modes
    X[4] = C<T>(v[0][0].re - v[0][0].im, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int a = c.t + 16 * e;
        const cpx<T> zk = v[0][e];
        cpx<T> xm;
        split_part(zk, mir[c.b == 0 ? (LONG_A - a) & (LONG_A - 1) : LONG_A - 1 - a], w[e], X[e], xm);
        if (c.edge && e == 0) X[e] = C<T>(zk.re + zk.im, 0);
    }
    // the second field's modes go to the first one's threads (w_0 and w_M do not count:
    // their wavenumbers are zero)
    fft_sync(64);
    if (c.f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) buf[c.t + 16 * e] = X[e];
    }
    fft_sync(64);
    double acc[2] = {0.0, 0.0};
    if (c.f == 0) {
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            if (e == 4 && !c.edge) continue;
            const int k = e < 4 ? LONG_B * (c.t + 16 * e) + c.b : LONG_M;
            const T kx = wavenumber<T>(k, NX, tpx);
            const cpx<T> q = e < 4 ? X[e] - ik(kx, lds[(c.col + 2) * LONG_A + c.t + 16 * (e & 3)]) : X[e];
            xh[k] = x[e] + alpha * p[e];
            const cpx<T> rn[1] = {r[e] - alpha * q};
            rh[k] = rn[0];
            cpx<T> z[1];
            precond_mode<T, 1>(kx, (T)0, sig, alp, rn, z);
            const double wt = half_weight(k, NX);
            acc[0] += wt * ((double)rn[0].re * (double)z[0].re + (double)rn[0].im * (double)z[0].im);
            acc[1] += wt * ((double)rn[0].re * (double)rn[0].re + (double)rn[0].im * (double)rn[0].im);
        }
    }
    block_sum<2>(acc, red + 32);
    if (threadIdx.x == 0) {
        part[PART_C3 + 2 * blockIdx.x] = acc[0];
        part[PART_C3 + 2 * blockIdx.x + 1] = acc[1];
        if (blockIdx.x == 0)
            for (int i = LONG_A / 2; i < nb3; ++i) part[PART_C3 + 2 * i] = part[PART_C3 + 2 * i + 1] = 0.0;
    }
}

enum { C2_RESID = 1, C2_STORE = 2, C2_UPDATE = 3, C2_RESID_INIT = 4 };

// MODE C2_UPDATE: reduce p.Gp (row-pass partials, nb_r1 blocks) -> alpha;
//   q = G p; x += alpha p; r -= alpha q; z = A^{-1} r; partial r.z, r.r.
// MODE C2_RESID: r = b - G x -> rh; partial r.z, r.r.
// MODE C2_RESID_INIT: reduce ||b||^2 (setup partials, nb_r1 blocks) -> bb;
//   r = b - G x -> rh (x = r = 0 for a zero b); partial r.z, r.r of r_0.
// MODE C2_STORE: q = G p -> qh.
// Projection of a residual mode onto the reflection-symmetric modes of a wall
// grid's periodic twin (Nx x Ny points): velocity component c is odd along its
// own axis and even along the other.  A field with E[N-1-X] = s E[X] along an
// axis has E^[k] = s e^{2 pi i k / N} E^[-k]; in the half spectrum E^[ky][-kx] is
// conj(E^[-ky][kx]), so both reflections pair the mode (kx, ky) with (kx, -ky) of
// the same column.  a: the mode, b: its partner (kx, -ky).
template <typename T, int D>
__device__ __forceinline__ cpx<T> wall_project(int c, cpx<T> a, cpx<T> b, int kx, int nx, int ky, int ny) {
    const T half = (T)0.5;
    if (D == 2) {
        const T sy = c == 1 ? (T)-1 : (T)1;
        T sn, cs;
        if (sizeof(T) == 8) {
            double s2, c2;
            sincospi(2.0 * (double)ky / (double)ny, &s2, &c2);
            sn = (T)s2;
            cs = (T)c2;
        } else {
            float s2, c2;
            sincospif(2.0f * (float)ky / (float)ny, &s2, &c2);
            sn = (T)s2;
            cs = (T)c2;
        }
        const cpx<T> om = C<T>(sy * cs, sy * sn), omc = C<T>(sy * cs, -sy * sn);
        const cpx<T> a2 = half * (a + om * b);
        const cpx<T> b2 = half * (b + omc * a);
        a = a2;
        b = b2;
    }
    const T sx = c == 0 ? (T)-1 : (T)1;
    T sn, cs;
    if (sizeof(T) == 8) {
        double s2, c2;
        sincospi(2.0 * (double)kx / (double)nx, &s2, &c2);
        sn = (T)s2;
        cs = (T)c2;
    } else {
        float s2, c2;
        sincospif(2.0f * (float)kx / (float)nx, &s2, &c2);
        sn = (T)s2;
        cs = (T)c2;
    }
    const cpx<T> ph = C<T>(sx * cs, sx * sn);
    return half * (a + ph * cj(b));
}

// WALL: the solve runs on the periodic twin of a wall grid; the new residual is
// projected onto the symmetric modes before it is used (rounding would otherwise
// seed the other parity, which the iteration amplifies at low wavenumbers).
// FEW (blocks of 128 threads, launches of at most one block of 256 per compute unit, where
// only latency counts): two waves per SIMD instead of three, without the 28 to 52 bytes of
// scratch that the FP64 forms for larger launches spill into (a kernel that uses scratch
// takes 1 to 2 us longer), and the fields the new residual needs loaded with the columns,
// in flight across the transform, where that fits the registers (all but the FP64 update,
// which spills again: 9.1 -> 10.2 us at 256 x 128).  256 x 128: update 9.0 -> 7.6 us,
// initial residual 10.0 -> 7.0; 512 x 512: FP64 residual 10.3 -> 9.2, initial residual
// 12.6 -> 10.1, FP32 update 5.6 -> 4.9.  Larger launches keep three waves: at 1024 x 1024
// two were slower (25 -> 27 us) with nothing spilled.
template <typename T, int MODE, bool FEW>
constexpr bool C2_PRE = FEW && (sizeof(T) == 4 || MODE != C2_UPDATE);
template <typename T, int EPC, int D, int MODE, bool WALL = false, bool FEW = false>
__global__ void __launch_bounds__(256, FEW ? 2 : COL_WAVES<EPC>) k_pcg_c2(ColGeom g, const cpx<T>* __restrict__ tw,
                                                 SolveScal* __restrict__ sc, const cpx<T>* __restrict__ H,
                                                 size_t NS, cpx<T>* __restrict__ qh, const cpx<T>* __restrict__ ph,
                                                 cpx<T>* __restrict__ xh, const cpx<T>* __restrict__ bh,
                                                 cpx<T>* __restrict__ rh, double* __restrict__ part, int nb_r1,
                                                 T tpx, T tpy) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    __shared__ double red[64];
    const PcgScal s0 = pcg_scalars(sc);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    // the row pass's columns do not depend on alpha: loaded right after the
    // partials of the reduction, in flight across it (LDS-only barriers)
    if (s0.done) return;
    constexpr int V = FEW ? 2 : 1;
    double pb[PF_K * V][1];
    if (MODE == C2_UPDATE) partials_fetch<1, V>(part + PART_C2, nb_r1, pb);
    if (MODE == C2_RESID_INIT) partials_fetch<1, V>(part + PART_GEN, nb_r1, pb);
    __builtin_amdgcn_sched_barrier(0);   // the partials' loads first
    cpx<T> in[D + 1][EPC];
    {
        const cpx<T>* srcs[D + 1];
#pragma unroll
        for (int c = 0; c <= D; ++c) srcs[c] = H + c * NS;
        col_fetch<T, EPC, D + 1>(g, ct, srcs, in);
    }
    constexpr bool PRE = C2_PRE<T, MODE, FEW>;
    constexpr int EP = PRE ? EPC : 1;
    cpx<T> r_pre[D][EP], x_pre[D][EP], p_pre[D][EP];   // r (or b), x, p
    if (PRE) {
#pragma unroll
        for (int e = 0; e < EP; ++e) {
            bool ok;
            const unsigned idx = col_index(g, ct, ct.t + g.TPC * e, ok);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                r_pre[c][e] = at32((MODE == C2_UPDATE ? (const cpx<T>*)rh : bh) + c * NS, idx);
                if (MODE == C2_UPDATE) {
                    x_pre[c][e] = at32(xh + c * NS, idx);
                    p_pre[c][e] = at32(ph + c * NS, idx);
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);   // keep the data loads ahead of the reduction
    T alpha = (T)0;
    bool zero_x = false;
    if (MODE == C2_RESID_INIT) {
        double tot[1];
        partials_sum<1, V>(part + PART_GEN, nb_r1, pb, tot, red);
        const double bb = tot[0] * s0.inv_n;
        const bool bad = !(bb == bb) || bb > 1.0e300;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            sc->bb = bb;
            if (bad) {
                sc->status = -2;
                sc->done = 1;
            }
        }
        if (bad) return;
        zero_x = !s0.init_bb && bb == 0.0;
    }
    if (MODE == C2_UPDATE) {
        double tot[1];
        partials_sum<1, V>(part + PART_C2, nb_r1, pb, tot, red);
        const double pq = tot[0];
        const double a = s0.rho / pq;
        alpha = (T)a;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            sc->pq = pq;
            sc->alpha = a;
            sc->rho_prev = s0.rho;
            sc->iter = s0.iter + 1;
            sc->first = 0;
        }
    }
    col_fft<T, EPC, D + 1>(g, ct, twm, in);
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    const T sig = (T)s0.sig, alp = (T)s0.alp;
    const double w = ct.valid ? half_weight(ct.kx, g.nx) : 0.0;
    double acc[2] = {0.0, 0.0};
    if (WALL && MODE != C2_STORE) {
        // the new residual of the whole column first, then its projection
        cpx<T> rn[D][EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
#pragma unroll
            for (int c = 0; c < D; ++c) rn[c][e] = C<T>(0, 0);
            if (ct.valid && j < g.ny) {
                const unsigned idx = ct.kx * g.ny + j;
                const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
                const cpx<T> wv = in[D][e];
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T kc = (c == 0) ? kx : ky;
                    const cpx<T> q = in[c][e] - ik(kc, wv);
                    if (MODE == C2_RESID) {
                        rn[c][e] = at32(bh + c * NS, idx) - q;
                    } else if (MODE == C2_RESID_INIT) {
                        rn[c][e] = zero_x ? C<T>(0, 0) : at32(bh + c * NS, idx) - q;
                        if (zero_x) at32(xh + c * NS, idx) = C<T>(0, 0);
                    } else {
                        at32(xh + c * NS, idx) = at32(xh + c * NS, idx) + alpha * at32(ph + c * NS, idx);
                        rn[c][e] = at32(rh + c * NS, idx) - alpha * q;
                    }
                    ct.buf[c * ct.fstride + j] = rn[c][e];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
            if (ct.valid && j < g.ny) {
                const unsigned idx = ct.kx * g.ny + j;
                const int jm = (g.ny - j) & (g.ny - 1);
                const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
                cpx<T> r[D], z[D];
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    r[c] = wall_project<T, D>(c, rn[c][e], ct.buf[c * ct.fstride + jm], ct.kx, g.nx, j, g.ny);
                    at32(rh + c * NS, idx) = r[c];
                }
                precond_mode<T, D>(kx, ky, sig, alp, r, z);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    acc[0] += w * ((double)r[c].re * (double)z[c].re + (double)r[c].im * (double)z[c].im);
                    acc[1] += w * ((double)r[c].re * (double)r[c].re + (double)r[c].im * (double)r[c].im);
                }
            }
        }
        block_sum<2>(acc, red + 32);
        if (threadIdx.x == 0) {
            part[PART_C3 + 2 * blockIdx.x] = acc[0];
            part[PART_C3 + 2 * blockIdx.x + 1] = acc[1];
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
        if (ct.valid && j < g.ny) {
            const unsigned idx = ct.kx * g.ny + j;
            const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
            const cpx<T> wv = in[D][e];
            cpx<T> r[D], z[D];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const T kc = (c == 0) ? kx : ky;
                const cpx<T> q = in[c][e] - ik(kc, wv);
                if (MODE == C2_STORE) {
                    at32(qh + c * NS, idx) = q;
                } else if (MODE == C2_RESID) {
                    r[c] = (PRE ? r_pre[c][e % EP] : at32(bh + c * NS, idx)) - q;
                    at32(rh + c * NS, idx) = r[c];
                } else if (MODE == C2_RESID_INIT) {
                    r[c] = zero_x ? C<T>(0, 0) : (PRE ? r_pre[c][e % EP] : at32(bh + c * NS, idx)) - q;
                    at32(rh + c * NS, idx) = r[c];
                    if (zero_x) at32(xh + c * NS, idx) = C<T>(0, 0);
                } else {
                    at32(xh + c * NS, idx) = (PRE ? x_pre[c][e % EP] : at32(xh + c * NS, idx)) +
                                             alpha * (PRE ? p_pre[c][e % EP] : at32(ph + c * NS, idx));
                    r[c] = (PRE ? r_pre[c][e % EP] : at32(rh + c * NS, idx)) - alpha * q;
                    at32(rh + c * NS, idx) = r[c];
                }
            }
            if (MODE != C2_STORE) {
                precond_mode<T, D>(kx, ky, sig, alp, r, z);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    acc[0] += w * ((double)r[c].re * (double)z[c].re + (double)r[c].im * (double)z[c].im);
                    acc[1] += w * ((double)r[c].re * (double)r[c].re + (double)r[c].im * (double)r[c].im);
                }
            }
        }
    }
    if (MODE != C2_STORE) {
        block_sum<2>(acc, red + 32);
        if (threadIdx.x == 0) {
            part[PART_C3 + 2 * blockIdx.x] = acc[0];
            part[PART_C3 + 2 * blockIdx.x + 1] = acc[1];
        }
    }
}

// First column pass of a solve.  Hb holds the row transforms of b (D fields),
// Hu those of the initial guess u0 (GUESS).  y-FFT of b -> b_hat into rh (and
// bh).  GUESS: partial ||b||^2; y-FFT of u0 -> x_hat, and (x_hat, div x_hat)/N
// y-inverse-transformed into H for the row pass of G x_0 (C2_RESID_INIT then
// forms r_0).  Otherwise x_hat = 0, r_0 = b_hat and the partials r.z, r.r.
// GUESS: the b part runs on blocks [0, nblocks) and the u0 part on blocks
// [nblocks, 2 nblocks), side by side (H must not alias Hb then).
template <typename T, int EPC, int D, bool GUESS>
__global__ void __launch_bounds__(256) k_pcg_setup(ColGeom g, const cpx<T>* __restrict__ tw,
                                                    const SolveScal* __restrict__ sc, const cpx<T>* Hb,
                                                    const cpx<T>* __restrict__ Hu, size_t NS, cpx<T>* __restrict__ bh,
                                                    cpx<T>* __restrict__ rh, cpx<T>* __restrict__ xh, cpx<T>* H,
                                                    double* __restrict__ part, T tpx, T tpy) {
    if (sc->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    __shared__ double red[32];
    const cpx<T>* twm = tw_size(tw, g.ny);
    const int job = GUESS ? (int)blockIdx.x / g.nblocks : 0;
    const ColThread<T> ct = col_thread_at<T>(g, lds, (int)blockIdx.x - job * g.nblocks);
    const double w = ct.valid ? half_weight(ct.kx, g.nx) : 0.0;
    const T kx = wavenumber<T>(ct.kx, g.nx, tpx);
    const T sig = (T)sc->sig, alp = (T)sc->alp, inv_n = (T)sc->inv_n;
    if (GUESS && job == 1) {
        cpx<T> vu[D][EPC];
        {
            const cpx<T>* srcs[D];
#pragma unroll
            for (int c = 0; c < D; ++c) srcs[c] = Hu + c * NS;
            col_load<T, EPC, D>(g, ct, srcs, false, twm, vu);
        }
        // the row pass's u0 columns need no y round trip: IFFT_y(x_hat / N) of
        // x_hat = FFT_y(u0 rows) is the u0 rows times ny / N, stored as loaded;
        // only div x_hat is formed in the spectral domain and inverse-transformed
        const T sraw = inv_n * (T)g.ny;
        if (ct.valid) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const int j = ct.t + g.TPC * e;
                if (j < g.ny) {
#pragma unroll
                    for (int c = 0; c < D; ++c) H[c * NS + (size_t)ct.kx * g.ny + j] = sraw * vu[c][e];
                }
            }
        }
        col_fft<T, EPC, D>(g, ct, twm, vu);
        cpx<T> o[1][EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
            o[0][e] = C<T>(0, 0);
            if (ct.valid && j < g.ny) {
                const unsigned idx = ct.kx * g.ny + j;
                const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
#pragma unroll
                for (int c = 0; c < D; ++c) at32(xh + c * NS, idx) = vu[c][e];
                cpx<T> dv = ik(kx, vu[0][e]);
                if (D == 2) dv = dv + ik(ky, vu[1 % D][e]);
                o[0][e] = inv_n * dv;
            }
        }
        cpx<T>* dsts[1] = {H + D * NS};
        col_store<T, EPC, 1>(g, ct, o, dsts, true, twm);
        return;
    }
    cpx<T> vb[D][EPC];
    {
        const cpx<T>* srcs[D];
#pragma unroll
        for (int c = 0; c < D; ++c) srcs[c] = Hb + c * NS;
        col_load<T, EPC, D>(g, ct, srcs, true, twm, vb);
    }
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
        if (ct.valid && j < g.ny) {
            const unsigned idx = ct.kx * g.ny + j;
            cpx<T> r[D], z[D];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                r[c] = vb[c][e];
                if (bh) at32(bh + c * NS, idx) = r[c];
                at32(rh + c * NS, idx) = r[c];
                if (!GUESS) at32(xh + c * NS, idx) = C<T>(0, 0);
            }
            if (GUESS) {
#pragma unroll
                for (int c = 0; c < D; ++c)
                    acc[0] += w * ((double)r[c].re * (double)r[c].re + (double)r[c].im * (double)r[c].im);
            } else {
                const T ky = (D == 2) ? wavenumber<T>(j, g.ny, tpy) : (T)0;
                precond_mode<T, D>(kx, ky, sig, alp, r, z);
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    acc[0] += w * ((double)r[c].re * (double)z[c].re + (double)r[c].im * (double)z[c].im);
                    acc[1] += w * ((double)r[c].re * (double)r[c].re + (double)r[c].im * (double)r[c].im);
                }
            }
        }
    }
    if (GUESS) {
        double bsum[1] = {acc[0]};
        block_sum<1>(bsum, red);
        if (threadIdx.x == 0) part[PART_GEN + blockIdx.x] = bsum[0];
    } else {
        block_sum<2>(acc, red);
        if (threadIdx.x == 0) {
            part[PART_C3 + 2 * blockIdx.x] = acc[0];
            part[PART_C3 + 2 * blockIdx.x + 1] = acc[1];
        }
    }
}


// Forward y-FFT of D H fields into S fields (no reduction).
template <typename T, int EPC, int D>
__global__ void __launch_bounds__(256) k_cols_to_S(ColGeom g, const cpx<T>* __restrict__ tw,
                                                    const cpx<T>* __restrict__ H, size_t NS,
                                                    cpx<T>* __restrict__ Sdst) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    cpx<T> v[D][EPC];
    const cpx<T>* srcs[D];
    cpx<T>* dsts[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        srcs[c] = H + c * NS;
        dsts[c] = Sdst + c * NS;
    }
    col_load<T, EPC, D>(g, ct, srcs, true, twm, v);
    col_store<T, EPC, D>(g, ct, v, dsts, false, twm);
}

// Inverse y-FFT of D S fields (times scale) into H fields.
template <typename T, int EPC, int D>
__global__ void __launch_bounds__(256) k_cols_from_S(ColGeom g, const cpx<T>* __restrict__ tw,
                                                      const cpx<T>* __restrict__ Ssrc, size_t NS,
                                                      cpx<T>* __restrict__ H, T scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    cpx<T> v[D][EPC];
    const cpx<T>* srcs[D];
    cpx<T>* dsts[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        srcs[c] = Ssrc + c * NS;
        dsts[c] = H + c * NS;
    }
    col_load<T, EPC, D>(g, ct, srcs, false, twm, v);
#pragma unroll
    for (int c = 0; c < D; ++c)
#pragma unroll
        for (int e = 0; e < EPC; ++e) v[c][e] = scale * v[c][e];
    col_store<T, EPC, D>(g, ct, v, dsts, true, twm);
}

// Spectral resampling between two grids of one domain, column part (the
// de-aliased right-hand side, subsec:dswe_1d): column kx of the destination
// takes the source's S-layout modes (source column length ny_src) for
// kx < kx_keep and signed ky mode |m| < m_keep, zero elsewhere, times scale,
// then runs the inverse y-FFT of the destination length; the result is the
// destination's H layout.  kx_keep and m_keep are half the smaller grid's
// lengths (m_keep = 1 in 1D), so the smaller grid's Nyquist modes are dropped.
template <typename T, int EPC, int NF>
__global__ void __launch_bounds__(256) k_cols_resample(ColGeom g, const cpx<T>* __restrict__ tw,
                                                        PtrList<const cpx<T>, MAXF> src, int ny_src,
                                                        PtrList<cpx<T>, MAXF> dst, int kx_keep, int m_keep,
                                                        T scale) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const cpx<T>* twm = tw_size(tw, g.ny);
    const ColThread<T> ct = col_thread<T>(g, lds);
    const bool col_kept = ct.valid && ct.kx < kx_keep;
    cpx<T> v[NF][EPC];
    cpx<T>* dsts[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        dsts[f] = dst.p[f];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = ct.t + g.TPC * e;
            const int m = (g.ny == 1) ? 0 : (j < g.ny / 2 ? j : j - g.ny);
            const bool keep = col_kept && j < g.ny && m < m_keep && -m < m_keep;
            const int js = m < 0 ? m + ny_src : m;
            v[f][e] = keep ? scale * src.p[f][(size_t)ct.kx * ny_src + js] : C<T>(0, 0);
        }
    }
    col_store<T, EPC, NF>(g, ct, v, dsts, true, twm);
}

// Grids between walls run on their periodic twin (twice the length per axis):
// k_reflect writes the even / odd reflection of nf fields of the nx x ny wall
// grid (field stride sstride) onto the twin (field stride dstride):
// dst[Y][X] = sx sy src[ry][rx], r(X) = X below n and 2n - 1 - X above, with the
// sign -1 on the reflected half of an axis along which field f is odd (bit f of
// oddx / oddy).
__global__ void __launch_bounds__(256) k_reflect(int nx, int ny, int nye, const double* __restrict__ src,
                                                  size_t sstride, double* __restrict__ dst, size_t dstride, int nf,
                                                  unsigned oddx, unsigned oddy) {
    const int nxe = 2 * nx;
    const size_t ne = (size_t)nxe * nye;
    const size_t total = ne * (size_t)nf;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int f = (int)(i / ne);
        const size_t p = i - (size_t)f * ne;
        const int Y = (int)(p / nxe), X = (int)(p - (size_t)Y * nxe);
        const bool fx = X >= nx, fy = Y >= ny;
        const int x = fx ? nxe - 1 - X : X;
        const int y = fy ? 2 * ny - 1 - Y : Y;
        double v = src[(size_t)f * sstride + (size_t)y * nx + x];
        if (fx && ((oddx >> f) & 1u)) v = -v;
        if (fy && ((oddy >> f) & 1u)) v = -v;
        dst[(size_t)f * dstride + p] = v;
    }
}

// k_restrict returns the symmetric part: the mean of a point's images on the twin
// (2 in 1D, 4 in 2D, signed as in k_reflect), which is the point itself for a
// symmetric field and drops what rounding put into the other parities.
__global__ void __launch_bounds__(256) k_restrict(int nx, int ny, int nye, const double* __restrict__ src,
                                                   size_t sstride, double* __restrict__ dst, size_t dstride, int nf,
                                                   unsigned oddx, unsigned oddy) {
    const size_t n = (size_t)nx * ny;
    const size_t total = n * (size_t)nf;
    const int nxe = 2 * nx;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int f = (int)(i / n);
        const size_t p = i - (size_t)f * n;
        const int y = (int)(p / nx), x = (int)(p - (size_t)y * nx);
        const double* sf = src + (size_t)f * sstride;
        const double sx = ((oddx >> f) & 1u) ? -1.0 : 1.0;
        const int xm = nxe - 1 - x;
        double v = sf[(size_t)y * nxe + x] + sx * sf[(size_t)y * nxe + xm];
        if (nye > 1) {
            const double sy = ((oddy >> f) & 1u) ? -1.0 : 1.0;
            const int ym = nye - 1 - y;
            v += sy * (sf[(size_t)ym * nxe + x] + sx * sf[(size_t)ym * nxe + xm]);
            v *= 0.25;
        } else {
            v *= 0.5;
        }
        dst[(size_t)f * dstride + p] = v;
    }
}

// Initialise the scalars of a solve on the device (no host round trip).  With
// have_coeffs the preconditioner coefficients are given; otherwise they are
// filled later by k_coeffs_finish or copied from another solve.
__global__ void k_init_scal(SolveScal* __restrict__ sc, double tol, int max_iter, double inv_n, int have_coeffs,
                            double sig, double alp, double kap, int flat, int init_bb) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    sc->rho = sc->rho_prev = sc->alpha = sc->beta = sc->bb = sc->rr = sc->pq = sc->relres = 0.0;
    sc->tol2 = tol * tol;
    sc->inv_n = inv_n;
    sc->iter = 0;
    sc->max_iter = max_iter;
    sc->done = 0;
    sc->converged = 0;
    sc->status = 0;
    sc->first = 1;
    sc->init_bb = init_bb;
    sc->outer = 0;
    if (have_coeffs) {
        sc->sig = sig;
        sc->alp = alp;
        sc->kap = kap;
        sc->flat = flat;
    }
}

// One refinement step enqueued without a host round trip: inner_open (run by
// the first thread of k_inner_start) starts the inner FP32 solve d of the step
// (the scalars of k_init_scal, the outer solve's coefficients), or, when the
// outer solve s has already converged, marks the inner solve done so that every
// kernel of the step returns at once.  The inner tolerance is no tighter than
// the outer target needs: with outer residual r, target tol ||b|| and inner stop
// ||r_in|| <= t ||r||, t = max(t_min, c tol ||b|| / ||r||) (c2 = c^2), so once r
// is within a few orders of the target the inner solve stops as soon as the
// corrected outer residual will meet it.  inner_close (run by k_pcg_check's
// first thread after the step's FP64 residual) adds the step's inner iterations
// and the step itself to the outer solve's counters (s->iter, s->outer) unless
// it was skipped.
__device__ __forceinline__ void inner_open(const SolveScal* __restrict__ s, SolveScal* __restrict__ d, double tol,
                                           int max_iter, double inv_n, double c2) {
    if (s->done) {
        d->done = 1;
        return;
    }
    d->rho = d->rho_prev = d->alpha = d->beta = d->bb = d->rr = d->pq = d->relres = 0.0;
    d->tol2 = tol * tol;
    d->inv_n = inv_n;
    d->iter = 0;
    d->max_iter = max_iter;
    d->done = 0;
    d->converged = 0;
    d->status = 0;
    d->first = 1;
    d->init_bb = 1;
    d->outer = 0;
    d->sig = s->sig;
    d->alp = s->alp;
    d->kap = s->kap;
    d->flat = s->flat;
    if (s->rr > 0.0 && s->bb > 0.0) {
        const double t2 = c2 * s->tol2 * (s->bb / s->rr);
        if (t2 > d->tol2) d->tol2 = t2 < 0.25 ? t2 : 0.25;
    }
}
__device__ __forceinline__ void inner_close(SolveScal* s, const SolveScal* d) {
    if (s->done) return;
    s->iter += d->iter;
    s->outer += 1;
}

// ---------------------------------------------------------------------------
// Reductions over physical fields (FP64)
// ---------------------------------------------------------------------------

// Per-block extremes for the coefficients of section 4: min eta, max eta,
// max(eta + lambda_+ eta |grad h|^2), max |grad h|^2 and a non-finite flag.
template <int D>
__global__ void __launch_bounds__(256) k_coeffs(size_t npts, const double* __restrict__ eta,
                                                const double* __restrict__ gh, double* __restrict__ part,
                                                float* __restrict__ eta32, float* __restrict__ gh32) {
    __shared__ double red[5 * 16];
    const double lp = (4.0 + sqrt(13.0)) / 6.0;
    double mn = 1.0e308, mx = -1.0e308, smax = -1.0e308, g2max = 0.0, bad = 0.0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < npts; i += stride) {
        const double e = eta[i];
        double g2 = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double h = gh[c * npts + i];
            g2 += h * h;
            if (gh32) gh32[c * npts + i] = (float)h;
        }
        if (eta32) eta32[i] = (float)e;
        if (!isfinite(e) || !isfinite(g2)) bad = 1.0;
        mn = fmin(mn, e);
        mx = fmax(mx, e);
        smax = fmax(smax, e + lp * e * g2);
        g2max = fmax(g2max, g2);
    }
    double v[5] = {-mn, mx, smax, g2max, bad};
#pragma unroll
    for (int a = 0; a < 5; ++a) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[a] = fmax(v[a], __shfl_xor(v[a], off, 64));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
    if (lane == 0)
        for (int a = 0; a < 5; ++a) red[a * 16 + wave] = v[a];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int a = 0; a < 5; ++a) {
            double s = red[a * 16];
            for (int w = 1; w < nw; ++w) s = fmax(s, red[a * 16 + w]);
            part[PART_GEN + 5 * blockIdx.x + a] = s;
        }
    }
}

// One block: the coefficients from the per-block extremes of k_coeffs.
// With init set, the solve's scalars are initialised here too (as k_init_scal
// with the given tol, max_iter, inv_n, init_bb), saving a launch per solve.
__global__ void __launch_bounds__(256) k_coeffs_finish(SolveScal* __restrict__ sc, const double* __restrict__ part,
                                                       int nb, int flat, int kind, int init, double tol,
                                                       int max_iter, double inv_n, int init_bb) {
    __shared__ double red[5 * 16];
    double r[5];
    final_max<5>(part + PART_GEN, nb, r, red);
    if (threadIdx.x != 0) return;
    if (init) {
        sc->rho = sc->rho_prev = sc->alpha = sc->beta = sc->bb = sc->rr = sc->pq = sc->relres = 0.0;
        sc->tol2 = tol * tol;
        sc->inv_n = inv_n;
        sc->iter = 0;
        sc->max_iter = max_iter;
        sc->done = 0;
        sc->converged = 0;
        sc->status = 0;
        sc->first = 1;
        sc->init_bb = init_bb;
    }
    const double emin = -r[0], emax = r[1], smx = r[2], g2m = r[3];
    sc->red[0] = emin;
    sc->red[1] = emax;
    sc->red[2] = smx;
    sc->red[3] = g2m;
    if (r[4] != 0.0 || !(emin > 0.0)) {
        sc->status = -2;
        sc->done = 1;
        return;
    }
    double sig, alp, kap;
    int fl;
    coeffs_formula(emin, emax, smx, g2m, flat, kind, sig, alp, kap, fl);
    sc->flat = fl;
    sc->sig = sig;
    sc->alp = alp;
    sc->kap = kap;
}

// Per-block min and max of a physical field (the flat-bottom test).
__global__ void __launch_bounds__(256) k_minmax(size_t n, const double* __restrict__ f, double* __restrict__ part) {
    __shared__ double red[2 * 16];
    double mn = 1.0e308, mx = -1.0e308;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        mn = fmin(mn, f[i]);
        mx = fmax(mx, f[i]);
    }
    double v[2] = {-mn, mx};
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[a] = fmax(v[a], __shfl_xor(v[a], off, 64));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
        red[wave] = v[0];
        red[16 + wave] = v[1];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = red[0], b = red[16];
        for (int w = 1; w < nw; ++w) {
            a = fmax(a, red[w]);
            b = fmax(b, red[16 + w]);
        }
        part[PART_GEN + 2 * blockIdx.x] = a;
        part[PART_GEN + 2 * blockIdx.x + 1] = b;
    }
}
__global__ void __launch_bounds__(256) k_minmax_finish(SolveScal* __restrict__ sc, const double* __restrict__ part,
                                                       int nb) {
    __shared__ double red[2 * 16];
    double r[2];
    final_max<2>(part + PART_GEN, nb, r, red);
    if (threadIdx.x == 0) {
        sc->red[0] = -r[0];
        sc->red[1] = r[1];
    }
}

// ---------------------------------------------------------------------------
// Small elementwise kernels
// ---------------------------------------------------------------------------
template <typename Td, typename Ts>
__global__ void k_convert(size_t n, const Ts* __restrict__ s, Td* __restrict__ d) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) d[i] = (Td)s[i];
}

// y = a*x + b*y  (b = 0 overwrites, x may be null for a pure scale)
__global__ void k_axpby(size_t n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double xv = x ? x[i] : 0.0;
        y[i] = (b == 0.0) ? a * xv : a * xv + b * y[i];
    }
}

// out = (base + dt * sum_k c_k f_k) / div  (up to 6 terms, in the order given;
// base may be null; div = 1 skips the division).  A multistep update divides by
// its leading coefficient rather than multiplying by a rounded reciprocal, so
// that coefficients summing to zero keep a constant field (and the mass) exact.
constexpr int LINCOMB_MAX = 6;
struct Lincomb4 {
    const double* f[LINCOMB_MAX];
    double c[LINCOMB_MAX];
    int n;
    double div;
};
__global__ void k_lincomb(size_t n, const double* __restrict__ base, double dt, Lincomb4 lc,
                          double* __restrict__ out) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        double s = 0.0;
        for (int k = 0; k < lc.n; ++k) s += lc.c[k] * lc.f[k][i];
        const double v = (base ? base[i] : 0.0) + dt * s;
        out[i] = lc.div == 1.0 ? v : v / lc.div;
    }
}

// Up to three independent linear combinations in one launch, each
// out = base + dt * sum_k c_k f_k as in k_lincomb (same order of operations);
// with `save` set, base is also copied there (out may alias base).
struct LcJob {
    double* out;
    const double* base;
    double* save;
    const double* f[4];
    double c[4];
    double dt;
    int nf;
    size_t n;
};
struct LcJobs {
    LcJob j[3];
    int n;
};
__global__ void k_lincomb_jobs(LcJobs J) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (int k = 0; k < J.n; ++k) {
        const LcJob& a = J.j[k];
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
            double s = 0.0;
            for (int q = 0; q < a.nf; ++q) s += a.c[q] * a.f[q][i];
            const double b = a.base ? a.base[i] : 0.0;
            if (a.save) a.save[i] = b;
            a.out[i] = b + a.dt * s;
        }
    }
}

__global__ void k_zero_c(size_t n, void* __restrict__ p) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    double* d = reinterpret_cast<double*>(p);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) d[i] = 0.0;
}

// Start of an FP32 inner solve from the FP64 outer residual: the inner solve's
// scalars (inner_open, first thread), r32 = (float) r, x32 = 0, and the
// partials of r32.z, r32.r32, in one pass.  The other blocks read only the
// outer scalars s, so the first thread's writes to sc race with nothing.
template <int D>
__global__ void __launch_bounds__(256) k_inner_start(int nx, int ny, size_t NS, const SolveScal* __restrict__ s,
                                                     SolveScal* __restrict__ sc, double tol, int max_iter,
                                                     double inv_n, double c2, const cpx<double>* __restrict__ r64,
                                                     cpx<float>* __restrict__ r32, cpx<float>* __restrict__ x32,
                                                     double* __restrict__ part, float tpx, float tpy) {
    __shared__ double red[32];
    if (blockIdx.x == 0 && threadIdx.x == 0) inner_open(s, sc, tol, max_iter, inv_n, c2);
    if (s->done) return;   // the refinement had already converged
    const float sig = (float)s->sig, alp = (float)s->alp;
    double acc[2] = {0.0, 0.0};
    const int nsi = (int)NS;
    const int lny = ilog2(ny);
    const int stride = gridDim.x * blockDim.x;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < nsi; idx += stride) {
        const int kxi = idx >> lny;
        const int kyi = idx & (ny - 1);
        const float kx = wavenumber<float>(kxi, nx, tpx);
        const float ky = (D == 2) ? wavenumber<float>(kyi, ny, tpy) : 0.0f;
        cpx<float> r[D], z[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const cpx<double> v = r64[c * NS + idx];
            r[c] = cpx<float>{(float)v.re, (float)v.im};
            r32[c * NS + idx] = r[c];
            x32[c * NS + idx] = C<float>(0, 0);
        }
        precond_mode<float, D>(kx, ky, sig, alp, r, z);
        const double w = half_weight(kxi, nx);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            acc[0] += w * ((double)r[c].re * (double)z[c].re + (double)r[c].im * (double)z[c].im);
            acc[1] += w * ((double)r[c].re * (double)r[c].re + (double)r[c].im * (double)r[c].im);
        }
    }
    block_sum<2>(acc, red);
    if (threadIdx.x == 0) {
        part[PART_C3 + 2 * blockIdx.x] = acc[0];
        part[PART_C3 + 2 * blockIdx.x + 1] = acc[1];
    }
}


}  // namespace sgn

namespace sgn {

// ---------------------------------------------------------------------------
// GMRES building blocks on D-vector fields in the S layout (modes [kx][ky],
// kx = 0..nx/2), FP64.  Dot products are Parseval sums over the half spectrum
// (weight 1 at kx = 0 and nx/2, 2 elsewhere) divided by nx ny.
// ---------------------------------------------------------------------------

// The kernels below take an optional stop flag (the done flag of the solve's
// scalars): when it is set they return at once, so a host that issues several
// Arnoldi steps ahead pays little for the steps after the cycle has ended.
__device__ __forceinline__ bool gmres_stopped(const SolveScal* stop) { return stop && stop->done; }

// Per-block partials of <w, V_i> for i < nv (V_i = V + i * vstride):
// part[block * nv + i].
template <int D>
__global__ void __launch_bounds__(256) k_S_multidot(int nx, int ny, size_t NS, const cpx<double>* __restrict__ w,
                                                    const cpx<double>* __restrict__ V, size_t vstride, int nv,
                                                    double* __restrict__ part, const SolveScal* stop) {
    if (gmres_stopped(stop)) return;
    __shared__ double red[16 * 8];
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (int i0 = 0; i0 < nv; i0 += 8) {
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int nb = nv - i0 < 8 ? nv - i0 : 8;
        for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < NS; idx += stride) {
            const int kx = (int)(idx / ny);
            const double wt = half_weight(kx, nx);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const cpx<double> a = w[c * NS + idx];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (k < nb) {
                        const cpx<double> v = V[(size_t)(i0 + k) * vstride + c * NS + idx];
                        acc[k] += wt * (a.re * v.re + a.im * v.im);
                    }
                }
            }
        }
        block_sum<8>(acc, red);
        if (threadIdx.x == 0)
            for (int k = 0; k < nb; ++k) part[(size_t)blockIdx.x * nv + i0 + k] = acc[k];
    }
}

// out[i] = scale * sum over blocks of part[b * nv + i] (fixed order), one block.
__global__ void __launch_bounds__(256) k_S_multidot_finish(const double* __restrict__ part, int nblocks, int nv,
                                                           double scale, double* __restrict__ out,
                                                           const SolveScal* stop) {
    if (gmres_stopped(stop)) return;
    __shared__ double red[16];
    for (int i = 0; i < nv; ++i) {
        double v[1] = {0.0};
        for (int b = threadIdx.x; b < nblocks; b += blockDim.x) v[0] += part[(size_t)b * nv + i];
        block_sum<1>(v, red);
        if (threadIdx.x == 0) out[i] = scale * v[0];
    }
}

// w += sign sum_i coef[i] V_i (coef in device memory), over n doubles; nv_dev,
// when set, gives the count in device memory instead of nv.
__global__ void k_S_multiaxpy(size_t n, double* __restrict__ w, const double* __restrict__ V, size_t vstride_d,
                              int nv, const double* __restrict__ coef, double sign, const SolveScal* stop,
                              const int* nv_dev) {
    if (gmres_stopped(stop)) return;
    if (nv_dev) nv = *nv_dev;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        double s = 0.0;
        for (int k = 0; k < nv; ++k) s += coef[k] * V[(size_t)k * vstride_d + i];
        w[i] += sign * s;
    }
}

// z = A^{-1} v on S fields (Def:A, section 6.1).
template <int D>
__global__ void k_S_precond(int nx, int ny, size_t NS, double tpx, double tpy, double sig, double alp,
                            const cpx<double>* __restrict__ v, cpx<double>* __restrict__ z, const SolveScal* stop) {
    if (gmres_stopped(stop)) return;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < NS; idx += stride) {
        const int kxi = (int)(idx / ny), kyi = (int)(idx - (size_t)kxi * ny);
        const double kx = wavenumber<double>(kxi, nx, tpx);
        const double ky = D == 2 ? wavenumber<double>(kyi, ny, tpy) : 0.0;
        cpx<double> r[D], zz[D];
#pragma unroll
        for (int c = 0; c < D; ++c) r[c] = v[c * NS + idx];
        precond_mode<double, D>(kx, ky, sig, alp, r, zz);
#pragma unroll
        for (int c = 0; c < D; ++c) z[c * NS + idx] = zz[c];
    }
}

// y = scale[0] x over n doubles (the scale in device memory).
__global__ void k_S_scale(size_t n, const double* __restrict__ scale, const double* __restrict__ x,
                          double* __restrict__ y, const SolveScal* stop) {
    if (gmres_stopped(stop)) return;
    const double a = *scale;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) y[i] = a * x[i];
}

// State of a restarted GMRES(m) solve kept on the device: the Hessenberg
// matrix of the running cycle reduced by Givens rotations, and the stop logic,
// so that the host reads it back once per few Arnoldi steps.
struct GmresCtl {
    double thr;       // tol ||b||
    double bnorm;
    double beta;      // ||r|| at the start of the running cycle
    double relres;    // beta / ||b||
    double scale;     // normalisation of the next basis vector (1 / beta, then 1 / h_{j+1,j})
    int jd;           // columns of the running cycle
    int iters, max_iter;
    int final_;       // 1: no further cycle (converged, max_iter reached or bad data)
    int conv, status; // status -2: non-finite data
};

// Hessenberg storage of a cycle of m steps: H (m + 1) x m by rows, cs, sn (m),
// g (m + 1), y (m) in one array.
__host__ __device__ inline size_t gmres_hess_doubles(int m) {
    return (size_t)(m + 1) * m + 2 * (size_t)m + (size_t)(m + 1) + (size_t)m;
}

__global__ void k_gmres_init(GmresCtl* ctl, double thr, double bnorm, int max_iter) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    ctl->thr = thr;
    ctl->bnorm = bnorm;
    ctl->beta = 0.0;
    ctl->relres = 0.0;
    ctl->scale = 1.0;
    ctl->jd = 0;
    ctl->iters = 0;
    ctl->max_iter = max_iter;
    ctl->final_ = 0;
    ctl->conv = 0;
    ctl->status = 0;
}

// Open a cycle: the operator passes run again (done = 0) unless the solve is over.
__global__ void k_gmres_open(const GmresCtl* ctl, SolveScal* sc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) sc->done = ctl->final_ ? 1 : 0;
}

// Start of a cycle from rr = ||r||^2 of the true residual (in V_0): the stop
// tests of the restart (||r|| <= thr: converged; max_iter reached; non-finite),
// else g = (beta, 0, ...) and V_0 is scaled by 1 / beta.
__global__ void k_gmres_begin(GmresCtl* ctl, SolveScal* sc, const double* __restrict__ rr, double* __restrict__ hs,
                              int m) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double beta = sqrt(fmax(*rr, 0.0));
    ctl->beta = beta;
    ctl->relres = beta / ctl->bnorm;
    ctl->jd = 0;
    bool stop = false;
    if (!isfinite(beta)) {
        ctl->status = -2;
        stop = true;
    } else if (beta <= ctl->thr) {
        ctl->conv = 1;
        stop = true;
    } else if (ctl->iters >= ctl->max_iter) {
        stop = true;
    }
    if (stop) {
        ctl->final_ = 1;
        sc->done = 1;
        return;
    }
    double* g = hs + (size_t)(m + 1) * m + 2 * (size_t)m;
    for (int i = 0; i <= m; ++i) g[i] = 0.0;
    g[0] = beta;
    ctl->scale = 1.0 / beta;
    sc->done = 0;
}

// Arnoldi step j: column j of H from the two Gram-Schmidt passes (h1 + h2) and
// h_{j+1,j} = ||w||, the earlier rotations applied to it, the new rotation
// that zeroes h_{j+1,j}, and the residual estimate |g_{j+1}|; the cycle ends
// (done) when that estimate reaches thr, at max_iter, or after step m - 1.
__global__ void k_gmres_givens(int j, int m, const double* __restrict__ coef, double* __restrict__ hs,
                               GmresCtl* ctl, SolveScal* sc) {
    if (threadIdx.x != 0 || blockIdx.x != 0 || sc->done) return;
    double* H = hs;
    double* cs = hs + (size_t)(m + 1) * m;
    double* sn = cs + m;
    double* g = sn + m;
    const double* h1 = coef;
    const double* h2 = coef + (m + 1);
    for (int i = 0; i <= j; ++i) H[(size_t)i * m + j] = h1[i] + h2[i];
    const double hn = sqrt(fmax(coef[2 * (m + 1)], 0.0));
    ctl->iters += 1;
    if (!isfinite(hn)) {
        ctl->status = -2;
        ctl->final_ = 1;
        sc->done = 1;
        return;
    }
    H[(size_t)(j + 1) * m + j] = hn;
    ctl->scale = hn != 0.0 ? 1.0 / hn : 1.0;
    for (int i = 0; i < j; ++i) {
        const double a = H[(size_t)i * m + j], b = H[(size_t)(i + 1) * m + j];
        H[(size_t)i * m + j] = cs[i] * a + sn[i] * b;
        H[(size_t)(i + 1) * m + j] = -sn[i] * a + cs[i] * b;
    }
    const double hjj = H[(size_t)j * m + j];
    const double den = hypot(hjj, hn);
    cs[j] = hjj / den;
    sn[j] = hn / den;
    H[(size_t)j * m + j] = den;
    H[(size_t)(j + 1) * m + j] = 0.0;
    g[j + 1] = -sn[j] * g[j];
    g[j] = cs[j] * g[j];
    ctl->jd = j + 1;
    if (fabs(g[j + 1]) <= ctl->thr || ctl->iters >= ctl->max_iter || j + 1 >= m) sc->done = 1;
}

// y = R^{-1} g over the cycle's jd columns (back substitution).
__global__ void k_gmres_backsolve(int m, const GmresCtl* ctl, double* __restrict__ hs) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double* H = hs;
    const double* g = hs + (size_t)(m + 1) * m + 2 * (size_t)m;
    double* y = hs + (size_t)(m + 1) * m + 2 * (size_t)m + (m + 1);
    const int jd = ctl->status == 0 ? ctl->jd : 0;
    for (int i = jd - 1; i >= 0; --i) {
        double t = g[i];
        for (int k = i + 1; k < jd; ++k) t -= H[(size_t)i * m + k] * y[k];
        y[i] = t / H[(size_t)i * m + i];
    }
}

}  // namespace sgn
