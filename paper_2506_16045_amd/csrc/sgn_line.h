// Whole 1D systems in the registers of one workgroup: transforms, constraint
// solves G u = b (Def:G in 1D, section 3.2) and right-hand sides of N = 2M
// points, M a compile-time power of two in [64, 4096].
//
// A solve is a serial chain of transforms of one short line, so what bounds it is
// latency: barriers, LDS round trips and dependent loads, not bytes or flops.
// The layout removes what it can of each:
//   - two fields at a time (p and Dp backwards, a and w forwards), one per half of
//     the workgroup, E = 4 complex entries per thread up to M = 1024, 8 at 2048 and 16
//     at 4096, so a transform is three to five radix-E passes in registers (the last
//     one of what is left) with one LDS exchange between two of them;
//   - the first pass reads and the last pass leaves the natural layout (thread t
//     of G = M / E holds entries t + s G), so the passes around a transform need
//     no LDS trip of their own beyond the real split's;
//   - the Krylov vectors live in the pair layout: a thread holds modes k and
//     M - k together, whose real split (section 6.1's transforms of real data) is
//     one complex product for both; modes 0 and M, both real and of zero
//     wavenumber, share one complex entry;
//   - where a field fits one wave (M <= 256) its exchanges need no barrier, where
//     the whole system does (M <= 128) nothing does; the barriers that remain order
//     LDS only, and the exchanges alternate between two buffers where LDS holds
//     them, so each costs one barrier.
// A system's geometry is a function of its size alone, and the sums run in a fixed
// order, so its result does not depend on what shares its launch.  Workgroups may
// be larger than a system needs: the extra waves only take part in the barriers.
#pragma once

#include "sgn_device.h"

namespace sgn {

constexpr int LINE_MMIN = 64, LINE_MMAX = 4096;   // half lengths this file takes

constexpr int line_log2(int x) { return x <= 1 ? 0 : 1 + line_log2(x / 2); }

template <typename T, int M_>
struct LineGeo {
    static constexpr int M = M_, N = 2 * M_;
    // complex entries per thread of a field: four, which spreads a line over the most
    // waves, while that takes at most 512 threads (FP64 solve per iteration at
    // n = 512: 3.8 us with eight entries in one wave, 3.0 with four in two; n = 1024:
    // 5.5 -> 4.4; n = 2048: 7.6 -> 6.0); then what 512 threads hold (workgroups of
    // 1024 leave 128 registers a thread, and the spills cost more than the waves
    // give: n = 4096 10.5 -> 15.2 us, n = 8192 20 -> 28)
    static constexpr int E = M >= 4096 ? 16 : M >= 2048 ? 8 : 4;
    static constexpr int G = M / E;                  // threads of one field
    static constexpr int TH = 2 * G;                 // threads of a system
    static constexpr bool ONE = TH <= 64;            // one wave holds the system
    static constexpr bool WFLD = G <= 64;            // one wave holds a field
    static constexpr int NP = M / 2 / TH;            // mode pairs per thread
    static constexpr int NW = ONE ? 1 : TH / 64;     // waves of a system
    // LDS bank swizzle: the low bits of an entry's place are XORed with the bits
    // above them, so that the first passes' writes, E entries apart, go to different
    // banks and runs of entries stay permutations of themselves (a padded layout was
    // measured with seven times the conflict cycles: it shifts the runs that one
    // 16-byte access serves across the banks)
    static constexpr int SH = E == 16 ? 4 : 3;
    static constexpr int MK = sizeof(T) == 8 ? 7 : 15;
    static constexpr int FS = M;                     // entries of one field buffer
    static constexpr bool PP = (size_t)4 * FS * sizeof(cpx<T>) <= 128 * 1024;   // two buffers per field
    // FP64 coefficients and x in registers (the longest line reads them from memory)
    static constexpr bool CREG = M < 4096;
    // twiddle bases: in registers where a transform needs few, else staged in LDS
    static constexpr bool TWREG = M <= 512;
};

// The pass of span NS (the product of the radices before it) of an M-point
// Stockham transform: radix E while that fits, then what is left.
template <int M, int NS>
struct LinePass {
    using Geo = LineGeo<double, M>;   // E, G and the plan do not depend on the type
    static constexpr int E = Geo::E, G = Geo::G;
    static constexpr int R = M / NS >= E ? E : M / NS;
    static constexpr int NB = E / R;                   // butterflies per thread
    static constexpr int LB = line_log2(R);            // twiddle bases per index
    static constexpr int KI = NS > G ? NB : 1;         // distinct twiddle indices per thread
    static constexpr int NK = NS < G ? NS : G;         // entries per base of the table
    static constexpr bool LAST = NS * R == M;
    // offsets of this pass's bases: per thread (registers) and in the LDS table
    static constexpr int reg_off() {
        if constexpr (NS == 1) return 0;
        else return LinePass<M, NS / E>::reg_off() + (NS / E > 1 ? LinePass<M, NS / E>::LB : 0);
    }
    static constexpr int tab_off() {
        if constexpr (NS == 1) return 0;
        else return LinePass<M, NS / E>::tab_off() + (NS / E > 1 ? LinePass<M, NS / E>::LB * LinePass<M, NS / E>::NK : 0);
    }
    static constexpr int reg_all() {
        if constexpr (LAST) return NS > 1 ? reg_off() + LB : 0;
        else return LinePass<M, NS * R>::reg_all();
    }
    static constexpr int tab_all() {
        if constexpr (LAST) return NS > 1 ? tab_off() + LB * NK : 0;
        else return LinePass<M, NS * R>::tab_all();
    }
};

// Threads of a workgroup that takes systems of n points (whole waves).
__host__ __device__ constexpr int line_threads_for(int n) {
    const int th[7] = {LineGeo<double, 64>::TH,   LineGeo<double, 128>::TH,  LineGeo<double, 256>::TH,
                       LineGeo<double, 512>::TH,  LineGeo<double, 1024>::TH, LineGeo<double, 2048>::TH,
                       LineGeo<double, 4096>::TH};
    int t = 64;
    for (int i = 0; i < 7; ++i)
        if ((128 << i) <= n && th[i] > t) t = th[i];
    return t;
}
// LDS bytes of the transform buffers of lines of half length M, and with the
// twiddle table behind them (FP64; FP32 transforms round the entries they read).
template <int M>
__host__ __device__ constexpr size_t line_buf_bytes() {
    using D = LineGeo<double, M>;
    using F = LineGeo<float, M>;
    constexpr size_t d = (size_t)(D::PP ? 4 : 2) * D::FS * 16, f = (size_t)(F::PP ? 4 : 2) * F::FS * 8;
    return d > f ? d : f;
}
template <int M>
__host__ __device__ constexpr size_t line_lds_of() {
    return line_buf_bytes<M>() + (LineGeo<double, M>::TWREG ? 0 : (size_t)LinePass<M, 1>::tab_all() * 16);
}
// The largest over the sizes up to n (a batched launch holds any of them).
__host__ __device__ constexpr size_t line_lds_bytes(int n) {
    size_t b = 0;
    const size_t all[7] = {line_lds_of<64>(),   line_lds_of<128>(),  line_lds_of<256>(), line_lds_of<512>(),
                           line_lds_of<1024>(), line_lds_of<2048>(), line_lds_of<4096>()};
    for (int i = 0; i < 7; ++i)
        if ((128 << i) <= n && all[i] > b) b = all[i];
    return b;
}
static_assert(line_lds_bytes(8192) <= 160 * 1024 - 2048, "LDS of a compute unit, less the static arrays");

__device__ __forceinline__ void line_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <typename T>
__device__ __forceinline__ cpx<double> to_f64(cpx<T> v) { return C<double>((double)v.re, (double)v.im); }

// Pair j of a real field (the caller's arrays: aligned to a double, not more).
__device__ __forceinline__ cpx<double> ld2(const double* p, int j) { return C<double>(p[2 * j], p[2 * j + 1]); }
__device__ __forceinline__ void st2(double* p, int j, cpx<double> v) {
    p[2 * j] = v.re;
    p[2 * j + 1] = v.im;
}

// Reduction scratch: doubles [0, 80) for sums and maxima, [96, 112) for p.Gp.

// One system's view of the workgroup: roles of the thread, exchange buffers.
// Where one wave holds the system, lanes beyond its threads repeat the work of the
// others (same values to the same places) and only stay out of the sums; larger
// systems' extra waves skip the work and keep the barriers.
template <typename T, int M>
struct Line {
    using Geo = LineGeo<T, M>;
    cpx<T>* buf;          // [buffer][field][FS], then the twiddle table
    double* red;
    const cpx<T>* tw;     // twiddle tables of every size (global)
    int q;                // thread of the system
    int fld, t;           // field of this thread (0, 1) and its place in it
    bool act;             // this wave works on the system
    bool mine;            // this thread's values count in sums
    int cur;              // buffer of the exchange under way
    static constexpr int NR = Geo::TWREG ? LinePass<M, 1>::reg_all() : 1;
    cpx<T> twr[NR];       // twiddle bases of the passes after the first

    // Stages the twiddle bases; the next block barrier publishes the LDS table (an
    // FP32 line reads the one its FP64 line staged).
    __device__ __forceinline__ Line(void* lds, double* r, const cpx<T>* tables)
        : buf(reinterpret_cast<cpx<T>*>(lds)), red(r), tw(tables) {
        const int tid = threadIdx.x;
        q = tid & (Geo::TH - 1);
        fld = q / Geo::G;
        t = q & (Geo::G - 1);
        mine = tid < Geo::TH;
        act = Geo::ONE || __builtin_amdgcn_readfirstlane(tid) < Geo::TH;
        cur = 0;
        fill<1>();
    }
    __device__ __forceinline__ cpx<double>* table() const {
        return reinterpret_cast<cpx<double>*>(reinterpret_cast<unsigned char*>(buf) + line_buf_bytes<M>());
    }
    template <int NS>
    __device__ __forceinline__ void fill() {
        using P = LinePass<M, NS>;
        if constexpr (NS > 1) {
            const cpx<T>* base = tw_size(tw, P::R * NS);   // W_{R NS}^{k 2^b}
            if constexpr (Geo::TWREG) {
#pragma unroll
                for (int b = 0; b < P::LB; ++b) twr[P::reg_off() + b] = base[(t & (NS - 1)) << b];
            } else if (act && sizeof(T) == 8) {
                for (int i = q; i < P::LB * P::NK; i += Geo::TH)
                    table()[P::tab_off() + i] = to_f64(base[(i & (P::NK - 1)) << (i / P::NK)]);
            }
        }
        if constexpr (!P::LAST) fill<NS * P::R>();
    }
    // This thread's place in its field, opaque to the compiler: tables in global
    // memory indexed by it are read where they are used instead of being hoisted out
    // of the iteration into registers that the data needs.
    __device__ __forceinline__ int place() const {
        int x = t;
        asm volatile("" : "+v"(x));
        return x;
    }
    __device__ __forceinline__ int thread() const {
        int x = q;
        asm volatile("" : "+v"(x));
        return x;
    }
    __device__ __forceinline__ cpx<T>* field(int f) const {
        return buf + (Geo::PP ? cur * 2 * Geo::FS : 0) + f * Geo::FS;
    }
    __device__ __forceinline__ void sync_all() const {
        if (Geo::ONE) line_wave_sync(); else block_lds_barrier();
    }
    __device__ __forceinline__ void sync_fld() const {
        if (Geo::WFLD) line_wave_sync(); else block_lds_barrier();
    }
    // The next exchange's buffer may be written: another one than the last
    // exchange's, or (one buffer) after every reader of it is done.
    __device__ __forceinline__ void turn_fld() {
        if (Geo::PP) cur ^= 1; else sync_fld();
    }
    __device__ __forceinline__ void turn_all() {
        if (Geo::PP) cur ^= 1; else sync_all();
    }
    // After one field's threads have read the other's buffer: where a field's own
    // exchanges are ordered within its wave only, the next one must not overtake.
    __device__ __forceinline__ void crossed() const {
        if (Geo::WFLD && !Geo::ONE) block_lds_barrier();
    }
    // Place of entry i.  The map is linear over XOR, so entry i + d with d's bits
    // outside i's is at el(b, at(i), d): one XOR where d reaches the low bits, and a
    // constant offset.
    static __device__ __forceinline__ constexpr int at(int i) { return i ^ ((i >> Geo::SH) & Geo::MK); }
    static __device__ __forceinline__ cpx<T>& el(cpx<T>* b, int ai, int d) {
        return b[(ai ^ (at(d) & Geo::MK)) + (d & ~Geo::MK)];
    }
    static __device__ __forceinline__ const cpx<T>& el(const cpx<T>* b, int ai, int d) {
        return b[(ai ^ (at(d) & Geo::MK)) + (d & ~Geo::MK)];
    }
};

// ---- transforms -------------------------------------------------------------
template <typename T>
__device__ __forceinline__ cpx<T> line_w16(int m, bool inverse) {   // W_16^m, m = 0..9
    const T c = (T)0.92387953251128675613, s = (T)0.38268343236508977173, r = (T)0.70710678118654752440;
    const T cs[10] = {(T)1, c, r, s, (T)0, -s, -r, -c, (T)-1, -c};
    const T sn[10] = {(T)0, s, r, c, (T)1, c, r, s, (T)0, -s};
    return C<T>(cs[m], inverse ? sn[m] : -sn[m]);
}
template <typename T, int R>
__device__ __forceinline__ void line_dft(cpx<T> (&v)[R], bool inverse) {
    if constexpr (R == 16) {
        cpx<T> a[4][4];
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
            for (int n1 = 0; n1 < 4; ++n1) a[n2][n1] = v[4 * n1 + n2];
            dft_small<T, 4>(a[n2], inverse);
#pragma unroll
            for (int k1 = 1; k1 < 4; ++k1) {
                if (n2 * k1 == 4)
                    a[n2][k1] = inverse ? mul_i(a[n2][k1]) : mul_mi(a[n2][k1]);
                else if (n2)
                    a[n2][k1] = a[n2][k1] * line_w16<T>(n2 * k1, inverse);
            }
        }
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            cpx<T> b[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
            dft_small<T, 4>(b, inverse);
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = b[k2];
        }
    } else {
        dft_small<T, R>(v, inverse);
    }
}

// W_8^i (E = 8) and W_4^i (E = 4), i < 4: the twiddle index of a thread's i-th
// butterfly in a last pass of a smaller radix is its first's plus i G, G / M = 1 / E.
template <typename T, int E>
__device__ __forceinline__ cpx<T> line_wE(int i) {
    const T h = (T)0.70710678118654752440;
    if (E == 4) return i == 0 ? C<T>(1, 0) : C<T>(0, -1);   // i < 2
    return i == 0 ? C<T>(1, 0) : i == 1 ? C<T>(h, -h) : i == 2 ? C<T>(0, -1) : C<T>(-h, -h);
}

// Twiddle bases of the pass: W_{R NS}^{k 2^b}, k the thread's (first) index; the
// other powers by products (no table of all powers; three roundings at most).
template <typename T, int M, int NS>
__device__ __forceinline__ void line_tw(const Line<T, M>& L, cpx<T> (&a)[LinePass<M, NS>::LB]) {
    using P = LinePass<M, NS>;
    if constexpr (LineGeo<T, M>::TWREG) {
#pragma unroll
        for (int b = 0; b < P::LB; ++b) a[b] = L.twr[P::reg_off() + b];
    } else {
        const cpx<double>* tb = L.table() + P::tab_off() + (L.t & (P::NK - 1));
#pragma unroll
        for (int b = 0; b < P::LB; ++b) a[b] = C<T>((T)tb[b * P::NK].re, (T)tb[b * P::NK].im);
    }
}

// Natural-layout entries of a field from and to its buffer.
template <typename T, int M>
__device__ __forceinline__ void line_load(const Line<T, M>& L, const cpx<T>* b, cpx<T> (&v)[LineGeo<T, M>::E]) {
    const int ai = L.at(L.t);
#pragma unroll
    for (int s = 0; s < LineGeo<T, M>::E; ++s) v[s] = L.el(b, ai, s * LineGeo<T, M>::G);
}
template <typename T, int M>
__device__ __forceinline__ void line_store(const Line<T, M>& L, cpx<T>* b, const cpx<T> (&v)[LineGeo<T, M>::E]) {
    const int ai = L.at(L.t);
#pragma unroll
    for (int s = 0; s < LineGeo<T, M>::E; ++s) L.el(b, ai, s * LineGeo<T, M>::G) = v[s];
}

// Field transform, natural layout in and out (unnormalised), from the pass of
// span NS on; `a` holds that pass's twiddle bases.
template <typename T, int M, bool INV, int NS = 1>
__device__ __forceinline__ void line_fft(Line<T, M>& L, cpx<T> (&v)[LineGeo<T, M>::E],
                                         const cpx<T> (&a)[LinePass<M, NS>::LB]) {
    using P = LinePass<M, NS>;
    if (L.act) {
#pragma unroll
        for (int i = 0; i < P::NB; ++i) {
            cpx<T> w[P::R];
            cpx<T> f[P::LB];
            if constexpr (NS > 1) {
#pragma unroll
                for (int b = 0; b < P::LB; ++b) {
                    // the i-th index is the first plus i G: W_{R NS}^{i G 2^b} = W_E^{i 2^b}
                    f[b] = a[b];
                    if (P::KI > 1 && i > 0 && b == 0) f[b] = a[b] * line_wE<T, P::E>(i);
                    if (P::KI > 1 && i > 0 && b == 1) f[b] = a[b] * line_wE<T, P::E>(2 * i);
                    if (INV) f[b] = cj(f[b]);
                }
            }
#pragma unroll
            for (int r = 0; r < P::R; ++r) {
                w[r] = v[i + r * P::NB];
                if constexpr (NS > 1) {
#pragma unroll
                    for (int b = 0; b < P::LB; ++b)
                        if (r & (1 << b)) w[r] = w[r] * f[b];
                }
            }
            line_dft<T, P::R>(w, INV);
#pragma unroll
            for (int r = 0; r < P::R; ++r) v[i + r * P::NB] = w[r];
        }
    }
    if constexpr (!P::LAST) {
        static_assert(P::NB == 1, "passes before the last take radix E");
        constexpr int NS2 = NS * P::R;
        cpx<T> a2[LinePass<M, NS2>::LB];
        L.turn_fld();
        cpx<T>* b = L.field(L.fld);
        if (L.act) {
            const int k = L.t & (NS - 1);
            const int ai = L.at((L.t - k) * P::R + k);
#pragma unroll
            for (int r = 0; r < P::R; ++r) L.el(b, ai, r * NS) = v[r];
        }
        L.sync_fld();
        if (L.act) {
            line_tw<T, M, NS2>(L, a2);
            line_load<T, M>(L, b, v);
        }
        line_fft<T, M, INV, NS2>(L, v, a2);
    }
}
template <typename T, int M, bool INV>
__device__ __forceinline__ void line_transform(Line<T, M>& L, cpx<T> (&v)[LineGeo<T, M>::E]) {
    const cpx<T> none[LinePass<M, 1>::LB] = {};
    line_fft<T, M, INV, 1>(L, v, none);
}

// ---- mode pairs ---------------------------------------------------------------
// Pair e of a thread: tau = tid + e TH in [0, M/2).  Its entries are modes tau and
// M - tau; pair 0 holds (X_0, X_M) as one complex entry, and mode M/2.
template <typename T, int M>
struct LinePairs {
    using Geo = LineGeo<T, M>;
    static constexpr int NP = Geo::NP;
    T tp;                 // 2 pi / L
    static constexpr bool HELD = NP <= 2;   // else read where used
    const cpx<T>* t2;
    cpx<T> wh[HELD ? NP : 1];   // W_N^tau
    __device__ __forceinline__ LinePairs(const Line<T, M>& L, T tp_) : tp(tp_), t2(tw_size(L.tw, 2 * M)) {
        if constexpr (HELD) {
#pragma unroll
            for (int e = 0; e < NP; ++e) wh[e] = t2[tau(L.q, e)];
        }
    }
    __device__ __forceinline__ cpx<T> w(int q, int e) const {
        if constexpr (HELD) return wh[e];
        else return t2[tau(q, e)];
    }
    // pair e of the thread whose index (Line::thread) is q
    static __device__ __forceinline__ int tau(int q, int e) { return q + e * Geo::TH; }
    static __device__ __forceinline__ int other(int q, int e) { return tau(q, e) == 0 ? M / 2 : M - tau(q, e); }
    __device__ __forceinline__ T k0(int q, int e) const { return tp * (T)tau(q, e); }
    __device__ __forceinline__ T k1(int q, int e) const { return tp * (T)other(q, e); }
    // half-spectrum weight of a pair's first entry in the Parseval sums (the second's is 2)
    static __device__ __forceinline__ double w0(int q, int e) { return tau(q, e) == 0 ? 1.0 : 2.0; }
};

// Half-spectrum entries of one pair -> the complex inverse transform's input:
// with S = X_k + X*_m, R = i (X_k - X*_m) W^{-k} (m = M - k): Z_k = S + R, Z_m = (S - R)*.
template <typename T>
__device__ __forceinline__ void pair_c2r(cpx<T> X0, cpx<T> X1, cpx<T> w, bool zero, cpx<T>& Z0, cpx<T>& Z1) {
    const cpx<T> S = X0 + cj(X1), R = mul_i((X0 - cj(X1)) * cj(w));
    Z0 = zero ? C<T>(X0.re + X0.im, X0.re - X0.im) : S + R;
    Z1 = zero ? (T)2 * cj(X1) : cj(S - R);
}
// Forward transform output of one pair -> its half-spectrum entries.
template <typename T>
__device__ __forceinline__ void pair_r2c(cpx<T> Z0, cpx<T> Z1, cpx<T> w, bool zero, cpx<T>& X0, cpx<T>& X1) {
    const T half = (T)0.5;
    const cpx<T> S = half * (Z0 + cj(Z1)), Q = mul_i(w * (half * (Z0 - cj(Z1))));
    X0 = zero ? C<T>(Z0.re + Z0.im, Z0.re - Z0.im) : S - Q;
    X1 = zero ? cj(Z1) : cj(S + Q);
}

// ---- the operator --------------------------------------------------------------
// Pointwise coefficients of G at this thread's points: the outputs are
// a = c0 p + c1 Dp (field 0) and w = c2 Dp + c1 p (field 1) with
// c0 = eta (1 + h_x^2), c1 = eta^2 h_x / 2, c2 = eta^3 / 3, so a thread needs the
// factor of its own field's input (o) and of the other's (x).
template <typename T, int M>
struct LineCoefReg {
    static constexpr int E = LineGeo<T, M>::E;
    static constexpr bool MEM = false;
    cpx<T> o[E], x[E];
    __device__ __forceinline__ LineCoefReg(const Line<T, M>& L, const double* eta, const double* hx) {
        if (!L.act) return;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * LineGeo<T, M>::G;
            const cpx<double> e = ld2(eta, j), h = ld2(hx, j);
            o[s] = C<T>((T)(L.fld ? e.re * e.re * e.re * (1.0 / 3.0) : e.re * (1.0 + h.re * h.re)),
                        (T)(L.fld ? e.im * e.im * e.im * (1.0 / 3.0) : e.im * (1.0 + h.im * h.im)));
            x[s] = C<T>((T)(0.5 * e.re * e.re * h.re), (T)(0.5 * e.im * e.im * h.im));
        }
    }
    // from tables that this thread wrote
    __device__ __forceinline__ LineCoefReg(const Line<T, M>& L, const cpx<T>* own, const cpx<T>* cross) {
        if (!L.act) return;
        const int t = L.place();
#pragma unroll
        for (int s = 0; s < E; ++s) {
            o[s] = own[t + s * LineGeo<T, M>::G];
            x[s] = cross[t + s * LineGeo<T, M>::G];
        }
    }
    __device__ __forceinline__ cpx<T> own(int s, int) const { return o[s]; }
    __device__ __forceinline__ cpx<T> cross(int s, int) const { return x[s]; }
};
// The same from memory (M = 4096 in FP64, whose registers the transform and the
// Krylov vectors fill): tables of N doubles each, read every application.
template <typename T, int M>
struct LineCoefMem {
    static constexpr bool MEM = true;
    const cpx<T>*o, *x;
    __device__ __forceinline__ cpx<T> own(int, int j) const { return o[j]; }
    __device__ __forceinline__ cpx<T> cross(int, int j) const { return x[j]; }
};
// From eta and h_x themselves (the few applications outside the iteration).
template <typename T, int M>
struct LineCoefFly {
    static constexpr bool MEM = true;
    const double *eta, *hx;
    int fld;
    __device__ __forceinline__ cpx<T> own(int, int j) const {
        const cpx<double> e = ld2(eta, j);
        if (fld) return C<T>((T)(e.re * e.re * e.re * (1.0 / 3.0)), (T)(e.im * e.im * e.im * (1.0 / 3.0)));
        const cpx<double> h = ld2(hx, j);
        return C<T>((T)(e.re * (1.0 + h.re * h.re)), (T)(e.im * (1.0 + h.im * h.im)));
    }
    __device__ __forceinline__ cpx<T> cross(int, int j) const {
        const cpx<double> e = ld2(eta, j);
        const cpx<double> h = ld2(hx, j);
        return C<T>((T)(0.5 * e.re * e.re * h.re), (T)(0.5 * e.im * e.im * h.im));
    }
};

// q_hat = G p_hat on the pair layout: a = F a_x, w = F w_x with (a_x, w_x) formed
// pointwise from p and Dp, q = a - D w.  `use(e, q0, q1)` consumes each pair;
// pq receives p.Gp (sum of p a + Dp w over the points).  On entry every reader of
// the buffers is done; on return the last buffer is still being read, so a
// sync_all comes before the next exchange (the callers' reductions hold one).
template <typename T, int M, typename Coef, typename Use>
__device__ __forceinline__ void line_apply(Line<T, M>& L, const LinePairs<T, M>& K,
                                           const cpx<T> (&p)[LineGeo<T, M>::NP][2], const Coef& coef, double& pq,
                                           Use&& use) {
    using Geo = LineGeo<T, M>;
    constexpr int NP = Geo::NP, E = Geo::E, G = Geo::G;
    const T invN = (T)1 / (T)Geo::N;
    cpx<T> v[E];
    // p / N and D p / N as inverse transform inputs
    L.turn_all();
    if (L.act) {
        cpx<T>*fa = L.field(0), *fb = L.field(1);
        const int q = K.HELD ? L.q : L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const bool z = K.tau(q, e) == 0;
            const cpx<T> p0 = invN * p[e][0], p1 = invN * p[e][1];
            cpx<T> z0, z1, y0, y1;
            pair_c2r(p0, p1, K.w(q, e), z, z0, z1);
            pair_c2r(ik(K.k0(q, e), p0), ik(K.k1(q, e), p1), K.w(q, e), z, y0, y1);
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            fa[i0] = z0;
            fa[i1] = z1;
            fb[i0] = y0;
            fb[i1] = y1;
        }
    }
    L.sync_all();
    if (L.act) {
        line_load<T, M>(L, L.field(L.fld), v);
    }
    line_transform<T, M, true>(L, v);
    // the other field's values at the same points, and the products
    L.turn_all();
    if (L.act) {
        line_store<T, M>(L, L.field(L.fld), v);
    }
    L.sync_all();
    double acc = 0.0;
    if (L.act) {
        const cpx<T>* b = L.field(L.fld ^ 1);
        const int ai = L.at(L.t);
        const int t = Coef::MEM ? L.place() : L.t;
        // coefficients from memory: two slots in use, the next two in flight
        constexpr int CH = Coef::MEM ? 2 : 4;
        cpx<T> co[2][CH], cx[2][CH];
        auto fetch = [&](int s0, int k) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                co[k][i] = coef.own(s0 + i, t + (s0 + i) * G);
                cx[k][i] = coef.cross(s0 + i, t + (s0 + i) * G);
            }
        };
        fetch(0, 0);
#pragma unroll
        for (int s0 = 0; s0 < E; s0 += CH) {
            const int k = (s0 / CH) & 1;
            if (Coef::MEM) __builtin_amdgcn_sched_barrier(0);
            if (s0 + CH < E) fetch(s0 + CH, k ^ 1);
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int s = s0 + i;
                const cpx<T> y = L.el(b, ai, s * G);
                const cpx<T> a = C<T>(co[k][i].re * v[s].re + cx[k][i].re * y.re,
                                      co[k][i].im * v[s].im + cx[k][i].im * y.im);
                acc += (double)v[s].re * (double)a.re + (double)v[s].im * (double)a.im;
                v[s] = a;
            }
        }
    }
    L.crossed();
    acc = wave_sum(L.mine ? acc : 0.0);
    if (!Geo::ONE && L.act && (threadIdx.x & 63) == 0) L.red[96 + (threadIdx.x >> 6)] = acc;
    line_transform<T, M, false>(L, v);
    L.turn_all();
    if (L.act) {
        line_store<T, M>(L, L.field(L.fld), v);
    }
    L.sync_all();
    if (Geo::ONE) {
        pq = acc;
    } else {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < Geo::NW; ++w) sum += L.red[96 + w];
        pq = uniform_d(sum);
    }
    if (L.act) {
        const cpx<T>*fa = L.field(0), *fb = L.field(1);
        const int q = K.HELD ? L.q : L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const bool z = K.tau(q, e) == 0;
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            cpx<T> a0, a1, w0, w1;
            pair_r2c(fa[i0], fa[i1], K.w(q, e), z, a0, a1);
            pair_r2c(fb[i0], fb[i1], K.w(q, e), z, w0, w1);
            use(e, a0 - ik(K.k0(q, e), w0), a1 - ik(K.k1(q, e), w1));
        }
    }
}

// Sums of two values over the system, in every thread; orders the buffers too.
template <typename T, int M>
__device__ __forceinline__ void line_sum2(const Line<T, M>& L, double& a, double& b) {
    using Geo = LineGeo<T, M>;
    a = wave_sum(a);
    b = wave_sum(b);
    if (Geo::ONE) {
        L.sync_all();
        return;
    }
    if (L.act && (threadIdx.x & 63) == 0) {
        L.red[2 * (threadIdx.x >> 6)] = a;
        L.red[2 * (threadIdx.x >> 6) + 1] = b;
    }
    L.sync_all();
    double sa = 0.0, sb = 0.0;
#pragma unroll
    for (int w = 0; w < Geo::NW; ++w) {
        sa += L.red[2 * w];
        sb += L.red[2 * w + 1];
    }
    a = uniform_d(sa);
    b = uniform_d(sb);
}
template <typename T, int M, int NV>
__device__ __forceinline__ void line_max(const Line<T, M>& L, double (&v)[NV]) {
    using Geo = LineGeo<T, M>;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = wave_max(v[i]);
    if (Geo::ONE) return;
    if (L.act && (threadIdx.x & 63) == 0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) L.red[i * 16 + (threadIdx.x >> 6)] = v[i];
    }
    L.sync_all();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        double m = L.red[i * 16];
#pragma unroll
        for (int w = 1; w < Geo::NW; ++w) m = fmax(m, L.red[i * 16 + w]);
        v[i] = uniform_d(m);
    }
    L.sync_all();
}

// Natural-layout registers of field 0 and field 1 (real data, transformed) to
// half-spectrum pairs of both: use(e, X0, X1, Y0, Y1).  A sync_all follows before
// the buffers are written again.
template <typename T, int M, typename Use>
__device__ __forceinline__ void line_to_pairs(Line<T, M>& L, const LinePairs<T, M>& K,
                                              cpx<T> (&v)[LineGeo<T, M>::E], Use&& use) {
    using Geo = LineGeo<T, M>;
    line_transform<T, M, false>(L, v);
    L.turn_all();
    if (L.act) {
        line_store<T, M>(L, L.field(L.fld), v);
    }
    L.sync_all();
    if (L.act) {
        const cpx<T>*fa = L.field(0), *fb = L.field(1);
        const int q = K.HELD ? L.q : L.thread();
#pragma unroll
        for (int e = 0; e < Geo::NP; ++e) {
            const bool z = K.tau(q, e) == 0;
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            cpx<T> x0, x1, y0, y1;
            pair_r2c(fa[i0], fa[i1], K.w(q, e), z, x0, x1);
            pair_r2c(fb[i0], fb[i1], K.w(q, e), z, y0, y1);
            use(e, x0, x1, y0, y1);
        }
    }
}

// PCG of section 3.2 on G d = r in precision T from d = 0, preconditioned by the
// diagonal A^{-1} (Def:A in 1D: factors z0, z1 per pair).  r is consumed; x
// accumulates d: add(alpha, p).  Stops when r.r <= tol2 bbref or
// after max_iter iterations; returns the iterations, rr the last r.r.
template <typename T, int M, typename Coef, typename Add>
__device__ __forceinline__ int line_pcg(Line<T, M>& L, const LinePairs<T, M>& K, cpx<T> (&r)[LineGeo<T, M>::NP][2],
                                        const Coef& coef, T sig, T alp, double tol2, double bbref, int max_iter,
                                        double& rr, Add&& add) {
    using Geo = LineGeo<T, M>;
    constexpr int NP = Geo::NP;
    const double dinvN = 1.0 / (double)Geo::N;
    cpx<T> p[NP][2];
    T z0[NP], z1[NP];
    const int q = L.q;
#pragma unroll
    for (int e = 0; e < NP; ++e) {
        const T a = K.k0(q, e), b = K.k1(q, e);
        z0[e] = (T)1 / (sig + alp * a * a);
        z1[e] = (T)1 / (sig + alp * b * b);
        p[e][0] = p[e][1] = C<T>(0, 0);
    }
    auto dots = [&](double& rz, double& r2) {
        double s0 = 0.0, s1 = 0.0;
        if (L.mine) {
#pragma unroll
            for (int e = 0; e < NP; ++e) {
                const double q0 = K.w0(q, e) * ((double)r[e][0].re * (double)r[e][0].re + (double)r[e][0].im * (double)r[e][0].im);
                const double q1 = 2.0 * ((double)r[e][1].re * (double)r[e][1].re + (double)r[e][1].im * (double)r[e][1].im);
                s0 += q0 * (double)z0[e] + q1 * (double)z1[e];
                s1 += q0 + q1;
            }
        }
        s0 *= dinvN;
        s1 *= dinvN;
        line_sum2(L, s0, s1);
        rz = s0;
        r2 = s1;
    };
    double rz, rho_prev = 1.0;
    L.sync_all();   // the reduction scratch may still be read
    dots(rz, rr);
    int it = 0;
    while (!(rr <= tol2 * bbref) && it < max_iter && rr == rr) {
        const T beta = it == 0 ? (T)0 : (T)(rz / rho_prev);
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            p[e][0] = it == 0 ? z0[e] * r[e][0] : z0[e] * r[e][0] + beta * p[e][0];
            p[e][1] = it == 0 ? z1[e] * r[e][1] : z1[e] * r[e][1] + beta * p[e][1];
        }
        double pq;
        T alpha = (T)0;
        line_apply<T, M>(L, K, p, coef, pq, [&](int e, cpx<T> q0, cpx<T> q1) {
            if (e == 0) alpha = (T)(rz / pq);
            r[e][0] = r[e][0] - alpha * q0;
            r[e][1] = r[e][1] - alpha * q1;
        });
        if (L.act) add(alpha, p);
        rho_prev = rz;
        dots(rz, rr);
        ++it;
    }
    return it;
}

// One system's solve G u = b by the workgroup (see blk_solve_system for the
// steps): coefficients of section 4, b_hat, the initial residual (from u when
// `guess`, else from 0), PCG (FP64) or FP32 inner PCG inside FP64 refinement
// (MIXED), and u.  w: workspace of batch_item_doubles(N) doubles.
template <int MODE, int M>
__device__ __forceinline__ BatchResult line_solve(double L_, const double* __restrict__ eta,
                                                  const double* __restrict__ hx, const double* __restrict__ b,
                                                  double* u, bool guess, double* w,
                                                  const cpx<double>* __restrict__ tw64,
                                                  const cpx<float>* __restrict__ tw32, const BatchParams& prm,
                                                  void* lds, double* red) {
    using Geo = LineGeo<double, M>;
    constexpr int N = Geo::N, E = Geo::E, G = Geo::G, NP = Geo::NP;
    Line<double, M> L(lds, red, tw64);
    BatchResult out{};
    // coefficients of section 4 from the extremes of eta and h_x, and b, u into
    // the transform layout (field 0: b, field 1: the guess)
    const double lp = (4.0 + sqrt(13.0)) / 6.0;
    double ex[5] = {-1.0e308, -1.0e308, -1.0e308, 0.0, 0.0};
    cpx<double> v[E];
    if (L.act) {
        const double* src = L.fld ? u : b;
        const bool have = !L.fld || guess;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            const cpx<double> e = ld2(eta, j);
            const cpx<double> h = ld2(hx, j);
            v[s] = have ? ld2(src, j) : C<double>(0, 0);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double ec = c ? e.im : e.re, hc = c ? h.im : h.re, vc = c ? v[s].im : v[s].re;
                const double g2 = hc * hc;
                if (!isfinite(ec) || !isfinite(g2) || !isfinite(vc)) ex[4] = 1.0;
                ex[0] = fmax(ex[0], -ec);
                ex[1] = fmax(ex[1], ec);
                ex[2] = fmax(ex[2], ec + lp * ec * g2);
                ex[3] = fmax(ex[3], g2);
            }
        }
    }
    line_max<double, M, 5>(L, ex);   // (its barriers publish the twiddle table)
    const double emin = -ex[0];
    if (ex[4] != 0.0 || !(emin > 0.0)) {
        out.status = -2;
        out.relres = __builtin_nan("");
        return out;
    }
    double sig, alp, kap;
    int fl;
    if (prm.have_coeffs) {
        sig = prm.sig;
        alp = prm.alp;
        kap = prm.kap;
        fl = prm.flat;
    } else {
        coeffs_formula(emin, ex[1], ex[2], ex[3], prm.flat, prm.coeff_kind, sig, alp, kap, fl);
    }
    out.sig = sig;
    out.alp = alp;
    out.kap = kap;
    out.flat = fl;
    const LinePairs<double, M> K(L, 6.283185307179586476925286766559 / L_);
    // x and (mixed) b in memory, each thread's own entries only
    cpx<double>* bh = reinterpret_cast<cpx<double>*>(w);
    cpx<double>* xh = bh + M;
    constexpr bool XREG = Geo::CREG && MODE == BATCH_FP64;
    cpx<double> r[NP][2], x[XREG ? NP : 1][2];
    double bb = 0.0, dum = 0.0;
#pragma unroll
    for (int e = 0; e < NP; ++e) r[e][0] = r[e][1] = C<double>(0, 0);
    cpx<double> x0[NP][2];
#pragma unroll
    for (int e = 0; e < NP; ++e) x0[e][0] = x0[e][1] = C<double>(0, 0);
    line_to_pairs<double, M>(L, K, v, [&](int e, cpx<double> b0, cpx<double> b1, cpx<double> u0, cpx<double> u1) {
        r[e][0] = b0;
        r[e][1] = b1;
        x0[e][0] = u0;
        x0[e][1] = u1;
        const int q = L.thread();
        bb += K.w0(q, e) * (b0.re * b0.re + b0.im * b0.im) + 2.0 * (b1.re * b1.re + b1.im * b1.im);
        if (MODE == BATCH_MIXED) {
            bh[K.tau(q, e)] = b0;
            bh[K.other(q, e)] = b1;
        }
    });
    bb = L.mine ? bb * (1.0 / (double)N) : 0.0;
    line_sum2(L, bb, dum);
    const double tol2 = prm.tol * prm.tol;
    const bool from_u = guess && bb > 0.0;
    if (!from_u) {
#pragma unroll
        for (int e = 0; e < NP; ++e) x0[e][0] = x0[e][1] = C<double>(0, 0);
    }
    auto keep_x = [&]() {
        if constexpr (!XREG) {
            if (L.act) {
                const int q = L.thread();
#pragma unroll
                for (int e = 0; e < NP; ++e) {
                    xh[K.tau(q, e)] = x0[e][0];
                    xh[K.other(q, e)] = x0[e][1];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < NP; ++e) {
                x[e][0] = x0[e][0];
                x[e][1] = x0[e][1];
            }
        }
    };
    double rr = bb, pq;
    const LineCoefFly<double, M> fly{eta, hx, L.fld};
    if constexpr (MODE == BATCH_FP64) {
        keep_x();
        auto solve = [&](const auto& coef) {
            if (from_u) {
                line_apply<double, M>(L, K, x0, coef, pq, [&](int e, cpx<double> q0, cpx<double> q1) {
                    r[e][0] = r[e][0] - q0;
                    r[e][1] = r[e][1] - q1;
                });
                L.sync_all();
            }
            out.iters = line_pcg<double, M>(L, K, r, coef, sig, alp, tol2, bb, prm.max_iter, rr,
                                            [&](double alpha, const cpx<double> (&p)[NP][2]) {
                if constexpr (XREG) {
#pragma unroll
                    for (int e = 0; e < NP; ++e) {
                        x[e][0] = x[e][0] + alpha * p[e][0];
                        x[e][1] = x[e][1] + alpha * p[e][1];
                    }
                } else {   // every load ahead of the first store
                    const int q = L.thread();
                    cpx<double> y[NP][2];
#pragma unroll
                    for (int e = 0; e < NP; ++e) {
                        y[e][0] = xh[K.tau(q, e)];
                        y[e][1] = xh[K.other(q, e)];
                    }
#pragma unroll
                    for (int e = 0; e < NP; ++e) {
                        xh[K.tau(q, e)] = y[e][0] + alpha * p[e][0];
                        xh[K.other(q, e)] = y[e][1] + alpha * p[e][1];
                    }
                }
            });
        };
        if constexpr (Geo::CREG) {
            const LineCoefReg<double, M> coef(L, eta, hx);
            solve(coef);
        } else {
            // tables c0, c2 (own factors of the two fields) and c1 behind xh
            cpx<double>* c = xh + M;
            cpx<double>* own = c + (L.fld ? M : 0);
            if (L.act) {
#pragma unroll
                for (int s = 0; s < E; ++s) {
                    const int j = L.t + s * G;
                    own[j] = fly.own(s, j);
                    if (!L.fld) c[2 * M + j] = fly.cross(s, j);
                }
            }
            __syncthreads();
            const LineCoefMem<double, M> coef{own, c + 2 * M};
            solve(coef);
        }
    } else {
        auto residual = [&]() {   // r = b - G x and its r.r
            line_apply<double, M>(L, K, x0, fly, pq, [&](int e, cpx<double> q0, cpx<double> q1) {
                const int q = L.thread();
                r[e][0] = bh[K.tau(q, e)] - q0;
                r[e][1] = bh[K.other(q, e)] - q1;
            });
            double s = 0.0, d = 0.0;
            if (L.mine) {
                const int q = L.thread();
#pragma unroll
                for (int e = 0; e < NP; ++e)
                    s += K.w0(q, e) * (r[e][0].re * r[e][0].re + r[e][0].im * r[e][0].im) +
                         2.0 * (r[e][1].re * r[e][1].re + r[e][1].im * r[e][1].im);
            }
            s *= 1.0 / (double)N;
            line_sum2(L, s, d);
            rr = s;
        };
        if (from_u) residual();
        keep_x();
        const double itol2 = prm.inner_tol * prm.inner_tol;
        Line<float, M> F(lds, red, tw32);
        const LinePairs<float, M> KF(F, (float)K.tp);
        // FP32 coefficients, rounded once, in a table behind xh: the registers they
        // take are the refinement's between two inner solves
        cpx<float>* own32 = reinterpret_cast<cpx<float>*>(xh + M) + (L.fld ? 2 * M : 0);
        if (L.act) {
            const int t = L.place();
#pragma unroll
            for (int s = 0; s < E; ++s) {
                if (s % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                const int j = t + s * G;
                const cpx<double> o = fly.own(s, j), c = fly.cross(s, j);
                own32[j] = C<float>((float)o.re, (float)o.im);
                own32[M + j] = C<float>((float)c.re, (float)c.im);
            }
        }
        while (!(rr <= tol2 * bb) && rr == rr && out.outer < prm.max_outer && bb > 0.0) {
            // inner FP32 solve of G d = r to t ||r||, then x += d and the FP64
            // residual r = b - G x; t = max(inner_tol, tol ||b|| / (2 ||r||)),
            // capped at 1/2: no tighter than the outer target needs
            double t2 = 0.25 * tol2 * (bb / rr);
            t2 = t2 < itol2 ? itol2 : (t2 > 0.25 ? 0.25 : t2);
            double irr = 0.0;
            cpx<float> r32[NP][2], d32[NP][2];
#pragma unroll
            for (int e = 0; e < NP; ++e) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    r32[e][c] = C<float>((float)r[e][c].re, (float)r[e][c].im);
                    d32[e][c] = C<float>(0, 0);
                }
            }
            auto inner = [&](const auto& coef32) {
                out.iters += line_pcg<float, M>(F, KF, r32, coef32, (float)sig, (float)alp, t2, rr, prm.max_iter, irr,
                                                [&](float alpha, const cpx<float> (&p)[NP][2]) {
#pragma unroll
                    for (int e = 0; e < NP; ++e) {
                        d32[e][0] = d32[e][0] + alpha * p[e][0];
                        d32[e][1] = d32[e][1] + alpha * p[e][1];
                    }
                });
            };
            if constexpr (Geo::CREG) inner(LineCoefReg<float, M>(F, own32, own32 + M));
            else inner(LineCoefMem<float, M>{own32, own32 + M});
            if (L.act) {
                const int q = L.thread();
#pragma unroll
                for (int e = 0; e < NP; ++e) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        cpx<double>* xp = xh + (c ? K.other(q, e) : K.tau(q, e));
                        x0[e][c] = *xp + C<double>((double)d32[e][c].re, (double)d32[e][c].im);
                        *xp = x0[e][c];
                    }
                }
            }
            residual();
            out.outer += 1;
        }
    }
    out.converged = (bb == 0.0 || rr <= tol2 * bb) ? 1 : 0;
    out.relres = bb > 0.0 ? sqrt(rr / bb) : 0.0;
    if (!(rr == rr)) out.status = -2;
    // u = x (physical), by field 0; the other field carries zeros along
    L.turn_all();
    if (L.act) {
        cpx<double>*fa = L.field(0), *fb = L.field(1);
        const double invN = 1.0 / (double)N;
        const int q = L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            cpx<double> y0, y1;
            if constexpr (XREG) {
                y0 = x[e][0];
                y1 = x[e][1];
            } else {
                y0 = xh[K.tau(q, e)];
                y1 = xh[K.other(q, e)];
            }
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            cpx<double> q0, q1;
            pair_c2r(invN * y0, invN * y1, K.w(q, e), K.tau(q, e) == 0, q0, q1);
            fa[i0] = q0;
            fa[i1] = q1;
            fb[i0] = fb[i1] = C<double>(0, 0);
        }
    }
    L.sync_all();
    if (L.act) {
        line_load<double, M>(L, L.field(L.fld), v);
    }
    line_transform<double, M, true>(L, v);
    if (L.act && L.fld == 0) {
#pragma unroll
        for (int s = 0; s < E; ++s) st2(u, L.t + s * G, v[s]);
    }
    return out;
}

// ---- right-hand side ------------------------------------------------------------
// First (order 1) or second derivative along the line of the real field whose
// points a field's threads hold as pairs (natural layout): forward transform, one
// exchange of mirrored entries, the wavenumber factors applied to the split
// spectrum and joined again for the inverse transform, all inside the field.
template <int M>
__device__ __forceinline__ void line_derivative(Line<double, M>& L, cpx<double> (&v)[LineGeo<double, M>::E],
                                                double tp, bool second) {
    using Geo = LineGeo<double, M>;
    constexpr int E = Geo::E, G = Geo::G;
    line_transform<double, M, false>(L, v);
    L.turn_fld();
    cpx<double>* b = L.field(L.fld);
    if (L.act) line_store<double, M>(L, b, v);
    L.sync_fld();
    if (L.act) {
        const cpx<double>* t2 = tw_size(L.tw, 2 * M);
        const double sc = 0.5 / (double)Geo::N;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int k = L.t + s * G;
            const cpx<double> zm = b[L.at((M - k) & (M - 1))], w = t2[k];
            const cpx<double> S = sc * (v[s] + cj(zm)), Q = mul_i(w * (sc * (v[s] - cj(zm))));
            const cpx<double> xk = S - Q, xm = S + Q;   // X_k and X*_{M-k}, over N
            const double kk = tp * (double)k, km = tp * (double)(M - k);
            // Y_k and Y*_{M-k}: i k X_k and (i k' X_{M-k})* = -i k' X*_{M-k}
            const cpx<double> yk = second ? (-kk * kk) * xk : ik(kk, xk);
            const cpx<double> ym = second ? (-km * km) * xm : ik(-km, xm);
            v[s] = (yk + ym) + mul_i((yk - ym) * cj(w));
            if (k == 0) v[s] = C<double>(0, 0);
        }
    }
    line_transform<double, M, true>(L, v);
}

// f(w, p) of one line (Eq:DSWEcf, Def:bigF): eta_t = -(eta u)_x, U_t = -eta (eta -
// h)_x - T h_x + (S - eta u^2)_x with S, T of Def:bigF.  Three rounds of two
// derivatives, one per field: (u_x, u_xx), ((eta u)_x, (u h_x)_x), then ((S -
// eta u^2)_x, eta_x); the flux enters through S as in 2D, so a right-hand side is
// three forward and three inverse transforms deep (it was seven and six, one
// field at a time).  Ends with a block barrier: eta_t and U_t may be read by any
// thread.
template <int M>
__device__ __forceinline__ void line_rhs(double L_, const double* __restrict__ eta, const double* __restrict__ hx,
                                         const double* __restrict__ u, double* __restrict__ eta_t,
                                         double* __restrict__ U_t, const cpx<double>* __restrict__ tw, void* lds,
                                         double* red) {
    using Geo = LineGeo<double, M>;
    constexpr int E = Geo::E, G = Geo::G;
    Line<double, M> L(lds, red, tw);
    const double tp = 6.283185307179586476925286766559 / L_;
    cpx<double> v[E], d[E];
    if (L.act) {
#pragma unroll
        for (int s = 0; s < E; ++s) d[s] = ld2(u, L.t + s * G);
    }
    line_derivative<M>(L, d, tp, L.fld != 0);   // u_x | u_xx
    if (L.act) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            const cpx<double> f = ld2(L.fld ? hx : eta, j), uu = ld2(u, j);
            v[s] = C<double>(f.re * uu.re, f.im * uu.im);
        }
    }
    line_derivative<M>(L, v, tp, false);        // (eta u)_x | (u h_x)_x
    // each field's share of S and T: field 0 (delta, m) holds
    // -e^3/3 d^2 + e^2 m d + e m b - e u^2 and -e^2/2 d^2 + e m d + m b, field 1
    // (delta_x, beta_x) holds u (e^3/3 d_x + e^2/2 b_x) and u (e^2/2 d_x + e b_x)
    cpx<double> T[E];
    if (L.act) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            const cpx<double> ee = ld2(eta, j), hh = ld2(hx, j), uu = ld2(u, j);
            double S2[2], T2[2], m2[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double e = c ? ee.im : ee.re, h = c ? hh.im : hh.re, w = c ? uu.im : uu.re;
                const double a = c ? d[s].im : d[s].re, m = c ? v[s].im : v[s].re;
                const double q2 = e * e, bt = h * w;
                S2[c] = L.fld ? w * (q2 * e / 3.0 * a + q2 / 2.0 * m)
                              : q2 * e / 3.0 * (-a * a) + q2 * m * a + e * m * bt - e * w * w;
                T2[c] = L.fld ? w * (q2 / 2.0 * a + e * m) : q2 / 2.0 * (-a * a) + e * m * a + m * bt;
                m2[c] = -m;
            }
            if (!L.fld) st2(eta_t, j, C<double>(m2[0], m2[1]));
            d[s] = C<double>(S2[0], S2[1]);
            T[s] = C<double>(T2[0], T2[1]);
        }
    }
    // field 1's share goes to field 0 (its S through buffer 1, its T through buffer 0)
    L.sync_all();
    if (L.act && L.fld) {
        cpx<double>*fa = L.field(0), *fb = L.field(1);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            L.el(fb, L.at(L.t), s * G) = d[s];
            L.el(fa, L.at(L.t), s * G) = T[s];
        }
    }
    L.sync_all();
    if (L.act) {
        const cpx<double>*fa = L.field(0), *fb = L.field(1);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            if (!L.fld) {
                v[s] = d[s] + L.el(fb, L.at(L.t), s * G);
                T[s] = T[s] + L.el(fa, L.at(L.t), s * G);
            } else {
                v[s] = ld2(eta, j);
            }
        }
    }
    L.sync_all();
    line_derivative<M>(L, v, tp, false);        // (S - eta u^2)_x | eta_x
    L.sync_all();
    if (L.act && L.fld) {
        cpx<double>* fb = L.field(1);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            const cpx<double> ee = ld2(eta, j), hh = ld2(hx, j);
            L.el(fb, L.at(L.t), s * G) = C<double>(-ee.re * (v[s].re - hh.re), -ee.im * (v[s].im - hh.im));
        }
    }
    L.sync_all();
    if (L.act && !L.fld) {
        const cpx<double>* fb = L.field(1);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = L.t + s * G;
            const cpx<double> hh = ld2(hx, j), gr = L.el(fb, L.at(L.t), s * G);
            st2(U_t, j, C<double>(v[s].re + (gr.re - hh.re * T[s].re), v[s].im + (gr.im - hh.im * T[s].im)));
        }
    }
    L.sync_all();
}

// h_x = D h and U = G_{eta,h} u of a state given by (eta, h, u); h_x = 0 for a
// constant h (flat).
template <int M>
__device__ __forceinline__ void line_slope(double L_, const double* h, double* hx,
                                           const cpx<double>* __restrict__ tw, void* lds, double* red) {
    using Geo = LineGeo<double, M>;
    Line<double, M> L(lds, red, tw);
    cpx<double> v[Geo::E];
    if (L.act) {
#pragma unroll
        for (int s = 0; s < Geo::E; ++s) v[s] = ld2(h, L.t + s * Geo::G);
    }
    line_derivative<M>(L, v, 6.283185307179586476925286766559 / L_, false);
    if (L.act && L.fld == 0) {
#pragma unroll
        for (int s = 0; s < Geo::E; ++s) st2(hx, L.t + s * Geo::G, v[s]);
    }
    L.sync_all();
}
template <int M>
__device__ __forceinline__ void line_momentum(double L_, const double* eta, const double* hx, const double* u,
                                              double* U, const cpx<double>* __restrict__ tw, void* lds,
                                              double* red) {
    using Geo = LineGeo<double, M>;
    constexpr int E = Geo::E, G = Geo::G, NP = Geo::NP;
    Line<double, M> L(lds, red, tw);
    const LinePairs<double, M> K(L, 6.283185307179586476925286766559 / L_);
    cpx<double> v[E], x[NP][2], g[NP][2];
#pragma unroll
    for (int e = 0; e < NP; ++e) x[e][0] = x[e][1] = g[e][0] = g[e][1] = C<double>(0, 0);
    if (L.act) {
#pragma unroll
        for (int s = 0; s < E; ++s) v[s] = ld2(u, L.t + s * G);
    }
    line_to_pairs<double, M>(L, K, v, [&](int e, cpx<double> a, cpx<double> b, cpx<double>, cpx<double>) {
        x[e][0] = a;
        x[e][1] = b;
    });
    L.sync_all();
    double pq;
    const LineCoefFly<double, M> fly{eta, hx, L.fld};
    line_apply<double, M>(L, K, x, fly, pq, [&](int e, cpx<double> a, cpx<double> b) {
        g[e][0] = a;
        g[e][1] = b;
    });
    L.sync_all();
    L.turn_all();
    if (L.act) {
        cpx<double>*fa = L.field(0), *fb = L.field(1);
        const double invN = 1.0 / (double)Geo::N;
        const int q = L.thread();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            const int i0 = L.at(K.tau(q, e)), i1 = L.at(K.other(q, e));
            cpx<double> q0, q1;
            pair_c2r(invN * g[e][0], invN * g[e][1], K.w(q, e), K.tau(q, e) == 0, q0, q1);
            fa[i0] = fb[i0] = q0;
            fa[i1] = fb[i1] = q1;
        }
    }
    L.sync_all();
    if (L.act) {
        line_load<double, M>(L, L.field(L.fld), v);
    }
    line_transform<double, M, true>(L, v);
    if (L.act && L.fld == 0) {
#pragma unroll
        for (int s = 0; s < E; ++s) st2(U, L.t + s * G, v[s]);
    }
    L.sync_all();
}

// Calls f with the compile-time half length of a line of n points; false when n is
// outside this file's range.
template <typename F>
__device__ __forceinline__ bool line_dispatch(int n, F&& f) {
    switch (n) {
        case 128: f(std::integral_constant<int, 64>{}); return true;
        case 256: f(std::integral_constant<int, 128>{}); return true;
        case 512: f(std::integral_constant<int, 256>{}); return true;
        case 1024: f(std::integral_constant<int, 512>{}); return true;
        case 2048: f(std::integral_constant<int, 1024>{}); return true;
        case 4096: f(std::integral_constant<int, 2048>{}); return true;
        case 8192: f(std::integral_constant<int, 4096>{}); return true;
        default: return false;
    }
}

}  // namespace sgn
