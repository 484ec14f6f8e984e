// Device building blocks of the spectral engine (gfx950, wave64).
//
// Spectral discretisation of section 6.1: every derivative is D = F^{-1}(iK)F
// with the Nyquist wavenumber of each axis set to zero.  A 2D real field
// f[ny][nx] (x fast) goes through two kinds of passes:
//   row pass    : real-to-complex FFT along x of each row, written transposed to
//                 the "H" layout H[kx][y] (kx = 0..nx/2, y contiguous), and the
//                 inverse complex-to-real pass back;
//   column pass : complex FFT along y of each kx column of H (contiguous), giving
//                 the "S" layout S[kx][ky] used for the Krylov state.
// A 1D field is the ny = 1 case: the column pass is then a plain per-mode loop.
// All transforms are unnormalised; callers apply 1/(nx*ny) once per round trip.
//
// FFTs hold their data in registers, four (eight) entries per thread, as radix-4 (8)
// Stockham passes with one LDS exchange between two of them (reg_fft).  A real row of
// length nx is transformed as a complex sequence of length M = nx/2
// (z_j = x_2j + i x_2j+1) followed by the usual even/odd split.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace sgn {

constexpr int TW_LOG = 14;
constexpr int TW_SIZE = 1 << TW_LOG;          // largest transform length
constexpr int TW_ALL = 2 * TW_SIZE - 1;       // entries of the per-size twiddle table

template <typename T>
struct alignas(2 * sizeof(T)) cpx {
    T re, im;
};

template <typename T> __device__ __forceinline__ cpx<T> C(T a, T b) { return cpx<T>{a, b}; }
template <typename T> __device__ __forceinline__ cpx<T> operator+(cpx<T> a, cpx<T> b) { return C(a.re + b.re, a.im + b.im); }
template <typename T> __device__ __forceinline__ cpx<T> operator-(cpx<T> a, cpx<T> b) { return C(a.re - b.re, a.im - b.im); }
template <typename T> __device__ __forceinline__ cpx<T> operator*(cpx<T> a, cpx<T> b) {
    return C(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
template <typename T> __device__ __forceinline__ cpx<T> operator*(T s, cpx<T> a) { return C(s * a.re, s * a.im); }
template <typename T> __device__ __forceinline__ cpx<T> cj(cpx<T> a) { return C(a.re, -a.im); }
template <typename T> __device__ __forceinline__ cpx<T> mul_i(cpx<T> a) { return C(-a.im, a.re); }   // i a
template <typename T> __device__ __forceinline__ cpx<T> mul_mi(cpx<T> a) { return C(a.im, -a.re); }  // -i a
// i k a for a real wavenumber k
template <typename T> __device__ __forceinline__ cpx<T> ik(T k, cpx<T> a) { return C(-k * a.im, k * a.re); }

// Element i of a field at `p`, the same for every lane: a 32-bit byte offset from a
// scalar base (one field of the largest grid is under 2^27 bytes), where a 64-bit
// index would hold two registers and an addition per access.
template <typename V>
__device__ __forceinline__ V& at32(V* p, unsigned i) {
    return *reinterpret_cast<V*>(reinterpret_cast<char*>(const_cast<std::remove_const_t<V>*>(p)) + i * (unsigned)sizeof(V));
}

__device__ __forceinline__ int ilog2(int x) { return 31 - __clz(x); }

// Signed wavenumber of FFT index j on an axis of n points and length L, with
// the Nyquist index n/2 mapped to zero (section 6.1).
template <typename T>
__device__ __forceinline__ T wavenumber(int j, int n, T two_pi_over_L) {
    int m = (j < n / 2) ? j : j - n;
    if (2 * j == n) m = 0;
    return two_pi_over_L * (T)m;
}

// ---------------------------------------------------------------------------
// Twiddles.  The global table holds, for every power of two L <= TW_SIZE, the
// L-th roots of unity W_L^j = exp(-2 pi i j / L) contiguously at offset L - 1
// (2 TW_SIZE - 1 entries).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ const cpx<T>* tw_size(const cpx<T>* __restrict__ tw_all, int L) {
    return tw_all + (L - 1);
}

// ---------------------------------------------------------------------------
// The transform of the short 1D lines (sgn_batch.h): Stockham FFT of length M (a power of
// two, at most 32) on NF fields in LDS at buf + f * fstride, in lockstep, thread t one
// butterfly of each pass: a radix-8 pass where it fits, then one radix-4 or radix-2
// pass for the remaining factor (a pass of radix R over span Ns reads
// x[j + r M/R], twiddles by W_{R Ns}^{k r} with k = j mod Ns, and writes the
// R-point DFT to y[(j - k) R + k + q Ns]).  Every thread of the block must call
// it (it contains block barriers).  twm[m] = W_M^m.
// Forward: exp(-i ...); inverse: exp(+i ...); unnormalised.
// ---------------------------------------------------------------------------

// In-register R-point DFTs (R = 2, 4, 8) of v[0..R).
template <typename T, int R>
__device__ __forceinline__ void dft_small(cpx<T> (&v)[R], bool inverse) {
    if (R == 2) {
        const cpx<T> a = v[0], b = v[1 % R];
        v[0] = a + b;
        v[1 % R] = a - b;
    } else if (R == 4) {
        const cpx<T> a0 = v[0] + v[2 % R], a1 = v[0] - v[2 % R];
        const cpx<T> a2 = v[1 % R] + v[3 % R], d = v[1 % R] - v[3 % R];
        const cpx<T> a3 = inverse ? mul_i(d) : mul_mi(d);
        v[0] = a0 + a2;
        v[1 % R] = a1 + a3;
        v[2 % R] = a0 - a2;
        v[3 % R] = a1 - a3;
    } else {
        // two 4-point DFTs (even and odd inputs), then W_8^q on the odd half
        cpx<T> e[4], o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            e[q] = v[(2 * q) % R];
            o[q] = v[(2 * q + 1) % R];
        }
        dft_small<T, 4>(e, inverse);
        dft_small<T, 4>(o, inverse);
        const T h = (T)0.70710678118654752440;
        const T sg = inverse ? (T)1 : (T)-1;
        const cpx<T> w1 = C<T>(h, sg * h), w3 = C<T>(-h, sg * h);
        const cpx<T> t0 = o[0];
        const cpx<T> t1 = w1 * o[1];
        const cpx<T> t2 = inverse ? mul_i(o[2]) : mul_mi(o[2]);
        const cpx<T> t3 = w3 * o[3];
        v[0] = e[0] + t0;
        v[4 % R] = e[0] - t0;
        v[1 % R] = e[1] + t1;
        v[5 % R] = e[1] - t1;
        v[2 % R] = e[2] + t2;
        v[6 % R] = e[2] - t2;
        v[3 % R] = e[3] + t3;
        v[7 % R] = e[3] - t3;
    }
}

template <typename T, int R, int NF>
__device__ __forceinline__ void fft_pass(cpx<T>* buf, int fstride, int M, int t, const cpx<T>* __restrict__ twm,
                                         bool inverse, int Ns, int sh) {
    const int MR = M / R;
    cpx<T> v[NF][R];
    if (t < MR) {
        const int k = t & (Ns - 1);
        cpx<T> w[R];
#pragma unroll
        for (int r = 1; r < R; ++r) {
            w[r] = twm[(k * r) << sh];   // W_{R Ns}^{k r} = W_M^{k r M / (R Ns)}
            if (inverse) w[r].im = -w[r].im;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const cpx<T>* bf = buf + f * fstride;
            v[f][0] = bf[t];
#pragma unroll
            for (int r = 1; r < R; ++r) v[f][r] = bf[t + r * MR] * w[r];
        }
    }
    __syncthreads();
    if (t < MR) {
        const int k = t & (Ns - 1), o = (t - k) * R + k;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            dft_small<T, R>(v[f], inverse);
            cpx<T>* bf = buf + f * fstride;
#pragma unroll
            for (int q = 0; q < R; ++q) bf[o + q * Ns] = v[f][q];
        }
    }
    __syncthreads();
}

template <typename T, int NF>
__device__ __forceinline__ void lds_fft(cpx<T>* buf, int fstride, int M, int t, const cpx<T>* __restrict__ twm,
                                        bool inverse) {
    const int logM = ilog2(M);
    int Ns = 1, logNs = 0;
    if (M >= 8) {
        fft_pass<T, 8, NF>(buf, fstride, M, t, twm, inverse, 1, logM - 3);
        Ns = 8;
        logNs = 3;
    }
    if (Ns * 4 <= M) {
        fft_pass<T, 4, NF>(buf, fstride, M, t, twm, inverse, Ns, logM - (logNs + 2));
        Ns <<= 2;
        logNs += 2;
    }
    if (Ns * 2 <= M) fft_pass<T, 2, NF>(buf, fstride, M, t, twm, inverse, Ns, logM - (logNs + 1));
}

// Block barrier that orders LDS only.  __syncthreads() fences all memory, which
// makes every wave wait for its global loads in flight (vmcnt(0)) at the
// barrier; kernels that issue their data loads before a reduction or an LDS
// exchange keep them in flight across such barriers.
__device__ __forceinline__ void block_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders LDS accesses of the G threads of one transform (thread indices t in
// [0, G), G a power of two): within a wave LDS runs in issue order and only the
// compiler needs fencing; wider transforms take the block barrier (every thread of
// the block must call it).
__device__ __forceinline__ void fft_sync(int G) {
    if (G <= 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    } else {
        block_lds_barrier();
    }
}

// Place of entry i in an exchange: the low bits XORed with the bits above, so that
// the strided writes of the first passes and the contiguous reads both spread over
// the banks (16-byte entries are served eight lanes at a time, 8-byte ones
// sixteen).  Linear over XOR.
template <typename T>
__device__ __forceinline__ int fft_at(int i) { return i ^ ((i >> 3) & (sizeof(T) == 8 ? 7 : 15)); }

// FFT of M points (a power of two) of NF fields held in the registers of G =
// max(M / E, 1) threads, natural layout in and out: v[f][e] is entry t + G e.
// Radix-E Stockham passes in registers and one LDS exchange between two of them
// (field f at buf + f fstride); the remaining factor is the last pass.  Against
// the same transform with its data in LDS (lds_fft) it saves the way in and out and
// half the barriers, and its barriers leave global accesses in flight: columns of 1024
// (three fields, FP64) 51 -> 40 us for 513 x 3, columns of 2048 262 -> 157 us for
// 1025 x 3; 256 x 128, the right-hand side's inverse row pass 56 -> 27 us.  twm[m] =
// W_M^m inside the table of all sizes.  Loading the twiddles a further pass ahead cost
// more in occupancy than it saved (513 x 3 columns of 1024: 40 -> 49 us).  Starts with a sync (buf may still be read by
// the same threads), ends without one.
template <typename T, int E, int NF>
__device__ __forceinline__ void reg_fft(cpx<T> (*v)[E], cpx<T>* buf, int fstride, int M, int t, int G,
                                        const cpx<T>* __restrict__ twm, bool inverse) {
    constexpr int LE = E == 8 ? 3 : 2;
    static_assert(E == 4 || E == 8, "radix of the passes");
    if (M < E) {   // one thread holds all of it
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (M == 2) {
                const cpx<T> a = v[f][0], b = v[f][1];
                v[f][0] = a + b;
                v[f][1] = a - b;
            } else if (M == 4) {
                cpx<T> w[4] = {v[f][0], v[f][1], v[f][2], v[f][3]};
                dft_small<T, 4>(w, inverse);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[f][e] = w[e];
            }
        }
        return;
    }
    const cpx<T>* all = twm - (M - 1);
#pragma unroll
    for (int f = 0; f < NF; ++f) dft_small<T, E>(v[f], inverse);
    const int at_t = fft_at<T>(t);
    int Np = 1;   // span of the pass just done
    while (Np * E < M) {
        const int Ns = Np * E, rem = M / Ns;   // this pass: span Ns, radix min(E, rem)
        // twiddle bases W_{R Ns}^{k 2^b} (the other powers by products), in flight
        // across the exchange; in a last pass of a smaller radix each of the thread's
        // butterflies has its own index t + i G
        cpx<T> a[4];
        if (rem >= E) {
            const cpx<T>* base = all + (E * Ns - 1);
            const int k = t & (Ns - 1);
#pragma unroll
            for (int b = 0; b < LE; ++b) a[b] = base[k << b];
        } else if (E == 8 && rem == 4) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[2 * i] = twm[t + i * G];
                a[2 * i + 1] = twm[2 * (t + i * G)];
            }
        } else {
#pragma unroll
            for (int i = 0; i < E / 2; ++i) a[i] = twm[t + i * G];
        }
        if (inverse) {
#pragma unroll
            for (int b = 0; b < 4; ++b) a[b].im = -a[b].im;
        }
        fft_sync(G);
        {
            const int k = t & (Np - 1);
            const int at_o = fft_at<T>((t - k) * E + k);
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int q = 0; q < E; ++q) buf[f * fstride + (at_o ^ fft_at<T>(q * Np))] = v[f][q];
        }
        fft_sync(G);
        int at_r = at_t;
        asm volatile("" : "+v"(at_r));   // addresses formed here, not held across the passes
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int e = 0; e < E; ++e) v[f][e] = buf[f * fstride + (at_r ^ fft_at<T>(e * G))];
        if (rem >= E) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
#pragma unroll
                for (int r = 1; r < E; ++r)
#pragma unroll
                    for (int b = 0; b < LE; ++b)
                        if (r & (1 << b)) v[f][r] = v[f][r] * a[b];
                dft_small<T, E>(v[f], inverse);
            }
        } else if (E == 8 && rem == 4) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const cpx<T> a1 = a[2 * i], a2 = a[2 * i + 1];
                    cpx<T> w[4] = {v[f][i], v[f][(i + 2) % E] * a1, v[f][(i + 4) % E] * a2,
                                   (v[f][(i + 6) % E] * a1) * a2};
                    dft_small<T, 4>(w, inverse);
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[f][(i + 2 * r) % E] = w[r];
                }
        } else {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < E / 2; ++i) {
                    const cpx<T> x = v[f][i], y = v[f][i + E / 2] * a[i];
                    v[f][i] = x + y;
                    v[f][i + E / 2] = x - y;
                }
        }
        Np = Ns;
    }
}

// ---------------------------------------------------------------------------
// Row geometry: a block holds R rows of TPR threads each; row r of the block is
// grid row row0 + r.  Thread t of a row owns complex positions j = t + TPR*e
// (e < EPC), i.e. real positions 2j and 2j+1.  LDS: NF fields x R rows of M+1
// complex entries (field stride R (M+1)).
// ---------------------------------------------------------------------------
struct RowGeom {
    int nx, ny, M, TPR, R, nblocks;
    int lgR, lgT;   // log2 of R and TPR
};

template <typename T>
struct RowThread {
    int r, t, y, row0;
    int tid;      // thread within the R TPR threads of the rows
    bool valid;
    cpx<T>* lds;  // LDS base of field 0
    int fstride;  // R (M+1)
};

// Map a launch block index to a row group so that consecutive row groups land on
// the same XCD (blocks are dealt round-robin over 8 XCDs, each with its own L2):
// neighbouring row groups share the cache lines of the transposed H layout.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    if ((nb & 7) != 0) return b;
    return (b & 7) * (nb >> 3) + (b >> 3);
}

// Row thread `tid` (of R TPR) of row block `blk` (blockIdx.x, or the block within one
// part of a launch that runs several independent row jobs side by side).
template <typename T>
__device__ __forceinline__ RowThread<T> row_thread_at(const RowGeom& g, cpx<T>* lds, int blk, int tid) {
    RowThread<T> rt;
    rt.tid = tid;
    rt.r = tid >> g.lgT;
    rt.t = tid & (g.TPR - 1);
    rt.row0 = xcd_remap(blk, g.nblocks) * g.R;
    rt.y = rt.row0 + rt.r;
    rt.valid = rt.y < g.ny;
    rt.lds = lds;
    rt.fstride = g.R * (g.M + 1);
    return rt;
}
template <typename T>
__device__ __forceinline__ RowThread<T> row_thread(const RowGeom& g, cpx<T>* lds) {
    return row_thread_at<T>(g, lds, blockIdx.x, threadIdx.x);
}

// LDS entries a row kernel with NF fields needs.
__host__ __device__ inline int row_lds_data(const RowGeom& g, int NF) { return NF * g.R * (g.M + 1); }

// row_inverse in pieces, for passes that overlap a field's transposed loads with
// other work: row_fetch issues the loads of this thread's mirrored pairs (k, M - k)
// (R (M/2 + 1) pairs over R M / EPC threads: EPC/2 each, R more for the first
// threads), row_join forms the inverse transform's input from them in the field's
// LDS region; row_inverse_lds transforms what a barrier has made visible there.
template <typename T, int EPC>
struct RowPairs {
    static constexpr int Q = EPC / 2 + 1;
    cpx<T> Xk[Q], Xm[Q];
};
// The thread index, opaque to the compiler: what is formed from it (pair indices,
// offsets, split twiddles) is formed again for each field instead of being held in
// registers across the fields' transforms.
__device__ __forceinline__ int row_tid(int tid) {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
}
template <typename T, int EPC>
__device__ __forceinline__ void row_fetch(const RowGeom& g, const RowThread<T>& rt, const cpx<T>* __restrict__ H,
                                          RowPairs<T, EPC>& X) {
    const int tid = row_tid(rt.tid), nt = g.R << g.lgT;
    const int M = g.M, ny = g.ny, totalp = (M / 2 + 1) << g.lgR;
    const int y = rt.row0 + (tid & (g.R - 1));   // nt is a multiple of R
#pragma unroll
    for (int q = 0; q < RowPairs<T, EPC>::Q; ++q) {
        const int i = tid + q * nt, p = i >> g.lgR;
        const bool ok = i < totalp && y < ny;
        X.Xk[q] = ok ? at32(H, p * ny + y) : C<T>(0, 0);
        X.Xm[q] = ok ? at32(H, (M - p) * ny + y) : C<T>(0, 0);
    }
}
// One pair of the real split each way.  With S = X_k + X*_m, D = i (X_k - X*_m)
// W^{-k} (m = M - k): Z_k = S + D, Z_m = (S - D)*; and back with S = (Z_k + Z*_m) / 2,
// D = i W^k (Z_k - Z*_m) / 2: X_k = S - D, X_m = (S + D)*.  One product serves both.
template <typename T>
__device__ __forceinline__ void split_join(cpx<T> Xk, cpx<T> Xm, cpx<T> w, cpx<T>& Zk, cpx<T>& Zm) {
    const cpx<T> S = Xk + cj(Xm), Dd = mul_i((Xk - cj(Xm)) * cj(w));
    Zk = S + Dd;
    Zm = cj(S - Dd);
}
template <typename T>
__device__ __forceinline__ void split_part(cpx<T> Zk, cpx<T> Zm, cpx<T> w, cpx<T>& Xk, cpx<T>& Xm) {
    const T half = (T)0.5;
    const cpx<T> S = half * (Zk + cj(Zm)), Dd = mul_i(w * (half * (Zk - cj(Zm))));
    Xk = S - Dd;
    Xm = cj(S + Dd);
}
// dx != 0: the entries are first multiplied by i k_x dx (tpx = 2 pi / Lx; the
// Nyquist entry has no wavenumber).
template <typename T, int EPC>
__device__ __forceinline__ void row_join(const RowGeom& g, const RowThread<T>& rt, const RowPairs<T, EPC>& X,
                                         cpx<T>* field, const cpx<T>* __restrict__ tw_all, T dx = (T)0,
                                         T tpx = (T)0) {
    const int tid = row_tid(rt.tid), nt = g.R << g.lgT;
    const int M = g.M, totalp = (M / 2 + 1) << g.lgR;
    const cpx<T>* tw2 = tw_size(tw_all, 2 * M);
    cpx<T>* b = field + (tid & (g.R - 1)) * (M + 1);
    cpx<T> w[RowPairs<T, EPC>::Q];
#pragma unroll
    for (int q = 0; q < RowPairs<T, EPC>::Q; ++q) {
        const int k = (tid + q * nt) >> g.lgR;
        w[q] = tw2[k < M ? k : 0];
    }
#pragma unroll
    for (int q = 0; q < RowPairs<T, EPC>::Q; ++q) {
        const int i = tid + q * nt;
        if (i >= totalp) continue;
        const int k = i >> g.lgR, m = M - k;
        cpx<T> xk = X.Xk[q], xm = X.Xm[q];
        if (dx != (T)0) {
            xk = ik(dx * (tpx * (T)k), xk);
            xm = ik(k == 0 ? (T)0 : dx * (tpx * (T)m), xm);
        }
        if (k == 0) {
            b[0] = C<T>(xk.re + xm.re, xk.re - xm.re);
        } else {
            cpx<T> zk, zm;
            split_join(xk, xm, w[q], zk, zm);
            b[m] = zm;
            b[k] = zk;
        }
    }
}
template <typename T, int EPC, int NF>
__device__ __forceinline__ void row_inverse_lds(const RowGeom& g, const RowThread<T>& rt, const cpx<T>* twm,
                                                cpx<T> (*z)[EPC]) {
    const int M = g.M;
    cpx<T>* rowb = rt.lds + rt.r * (M + 1);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = rt.t + g.TPR * e;
            if (j < M) z[f][e] = rowb[f * rt.fstride + j];
        }
    }
    reg_fft<T, EPC, NF>(z, rowb, rt.fstride, M, rt.t, g.TPR, twm, true);
}

// Inverse row transforms of NF fields: H_f[kx][y] (kx = 0..M) -> real pairs
// z[f][e] = (x_2j, x_2j+1), unnormalised (nx times the inverse DFT).  The
// imaginary parts of the kx = 0 and kx = nx/2 entries are ignored (real signal).
// The even/odd recombination Z_k = (X_k + X*_{M-k}) + i (X_k - X*_{M-k}) W_nx^{-k}
// is formed from each mirrored pair (k, M - k) as it goes to LDS, so it costs no
// LDS pass of its own; the transposed loads of all fields are in flight together.
template <typename T, int EPC, int NF>
__device__ __forceinline__ void row_inverse(const RowGeom& g, const RowThread<T>& rt,
                                            const cpx<T>* const (&H)[NF],
                                            const cpx<T>* __restrict__ tw_all, const cpx<T>* twm,
                                            cpx<T> (&z)[NF][EPC]) {
    RowPairs<T, EPC> X[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) row_fetch<T, EPC>(g, rt, H[f], X[f]);
#pragma unroll
    for (int f = 0; f < NF; ++f) row_join<T, EPC>(g, rt, X[f], rt.lds + f * rt.fstride, tw_all);
    fft_sync(g.R << g.lgT);
    row_inverse_lds<T, EPC, NF>(g, rt, twm, z);
    fft_sync(g.R << g.lgT);
}

// Forward row transforms of NF fields: real pairs z[f][e] -> H_f[kx][y] for
// kx = 0..M, each value multiplied by `scale` (z is used up).  The recombination
// X_k = (Z_k + Z*_{M-k})/2 - i W_nx^k (Z_k - Z*_{M-k})/2 is formed as each entry
// is stored (no LDS pass of its own).
template <typename T, int EPC, int NF>
__device__ __forceinline__ void row_forward(const RowGeom& g, const RowThread<T>& rt, cpx<T> (&z)[NF][EPC],
                                            cpx<T>* const (&H)[NF], const cpx<T>* __restrict__ tw_all,
                                            const cpx<T>* twm, T scale) {
    const int M = g.M, R = g.R, ny = g.ny, nt = g.R << g.lgT;
    const cpx<T>* tw2 = tw_size(tw_all, 2 * M);
    cpx<T>* rowb = rt.lds + rt.r * (M + 1);
    reg_fft<T, EPC, NF>(z, rowb, rt.fstride, M, rt.t, g.TPR, twm, false);
    fft_sync(g.TPR);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int j = rt.t + g.TPR * e;
            if (j < M) rowb[f * rt.fstride + j] = z[f][e];
        }
    }
    fft_sync(nt);
    constexpr int Q = EPC / 2 + 1;
    const int tid = row_tid(rt.tid);
    const int totalp = (M / 2 + 1) << g.lgR;
    const int ry = tid & (R - 1), y = rt.row0 + ry;
    cpx<T> w[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int k = (tid + q * nt) >> g.lgR;
        w[q] = tw2[k < M ? k : 0];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const cpx<T>* b = rt.lds + f * rt.fstride + ry * (M + 1);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = tid + q * nt;
            if (i >= totalp || y >= ny) continue;
            const int k = i >> g.lgR, m = M - k;
            const cpx<T> zk = b[k];
            cpx<T> xk, xm;
            if (k == 0) {
                xk = C<T>(zk.re + zk.im, 0);
                xm = C<T>(zk.re - zk.im, 0);
            } else {
                split_part(zk, b[m], w[q], xk, xm);
            }
            at32(H[f], k * ny + y) = scale * xk;
            if (m != k) at32(H[f], m * ny + y) = scale * xm;
        }
    }
    fft_sync(nt);
}

// The block barriers of row_forward, for threads of the block that have no row to
// transform meanwhile.
template <int EPC>
__device__ __forceinline__ void row_forward_idle(const RowGeom& g) {
    if (g.TPR > 64) {
        for (int Np = 1; Np * EPC < g.M; Np *= EPC) {
            block_lds_barrier();
            block_lds_barrier();
        }
        block_lds_barrier();
    }
    if ((g.R << g.lgT) > 64) {
        block_lds_barrier();
        block_lds_barrier();
    }
}

// ---------------------------------------------------------------------------
// Column geometry: a block holds Cb columns (kx) of TPC threads each; column c
// is kx = blockIdx.x * Cb + c.  Thread t owns modes j = t + TPC*e (e < EPC,
// j < ny).  LDS: NF fields x Cb columns of ny entries (field stride Cb ny).
// ---------------------------------------------------------------------------
struct ColGeom {
    int nx, ny, nxh, TPC, Cb, nblocks;
    int lgT;   // log2 of TPC
};

template <typename T>
struct ColThread {
    int c, t, kx;
    bool valid;
    cpx<T>* buf;  // field 0 of this column
    int fstride;  // Cb ny
};

__host__ __device__ inline int col_lds_data(const ColGeom& g, int NF) { return NF * g.Cb * g.ny; }

// Column thread of column block `blk` (blockIdx.x, or the block within one part
// of a launch that runs several column jobs side by side).
template <typename T>
__device__ __forceinline__ ColThread<T> col_thread_at(const ColGeom& g, cpx<T>* lds, int blk) {
    ColThread<T> ct;
    ct.c = threadIdx.x >> g.lgT;
    ct.t = threadIdx.x & (g.TPC - 1);
    ct.kx = blk * g.Cb + ct.c;
    ct.valid = ct.kx < g.nxh;
    ct.buf = lds + ct.c * g.ny;
    ct.fstride = g.Cb * g.ny;
    return ct;
}
template <typename T>
__device__ __forceinline__ ColThread<T> col_thread(const ColGeom& g, cpx<T>* lds) {
    return col_thread_at<T>(g, lds, blockIdx.x);
}

// Load NF columns of H (or S) into registers (col_fetch), then optionally
// transform them along y (col_fft); col_load does both.
// Entry (column kx, row j) of a column-layout field, clamped in range (entry 0
// of the field where the lane has no entry), and whether it is a real entry.
// The loads through it are unconditional: predicated loads make the compiler
// wait for every load in flight (see partials_fetch).
template <typename T>
__device__ __forceinline__ unsigned col_index(const ColGeom& g, const ColThread<T>& ct, int j, bool& ok) {
    ok = ct.valid && j < g.ny;
    return ok ? (unsigned)(ct.kx * g.ny + j) : 0u;
}
// A lane without an entry (a column past nx/2 in the last block) holds a copy
// of entry 0: finite, transformed with its column and never stored or summed
// (the callers guard outputs and weights by ct.valid).
template <typename T, int EPC, int NF>
__device__ __forceinline__ void col_fetch(const ColGeom& g, const ColThread<T>& ct, const cpx<T>* const (&H)[NF],
                                          cpx<T> (&v)[NF][EPC]) {
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        bool ok;
        const unsigned idx = col_index(g, ct, ct.t + g.TPC * e, ok);
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f][e] = at32(H[f], idx);
    }
}
template <typename T, int EPC, int NF>
__device__ __forceinline__ void col_fft(const ColGeom& g, const ColThread<T>& ct, const cpx<T>* twm,
                                        cpx<T> (&v)[NF][EPC]) {
    if (g.ny > 1) {
        reg_fft<T, EPC, NF>(v, ct.buf, ct.fstride, g.ny, ct.t, g.TPC, twm, false);
        fft_sync(g.TPC);
    }
}
// col_load: lanes without an entry hold zeros.
template <typename T, int EPC, int NF>
__device__ __forceinline__ void col_load(const ColGeom& g, const ColThread<T>& ct, const cpx<T>* const (&H)[NF],
                                         bool fft, const cpx<T>* twm, cpx<T> (&v)[NF][EPC]) {
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int j = ct.t + g.TPC * e;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (j < g.ny) v[f][e] = ct.valid ? at32(H[f], ct.kx * g.ny + j) : C<T>(0, 0);
    }
    if (fft) col_fft<T, EPC, NF>(g, ct, twm, v);
}

// Optionally inverse-transform NF columns along y, then store them to H (or S).
template <typename T, int EPC, int NF>
__device__ __forceinline__ void col_store(const ColGeom& g, const ColThread<T>& ct, cpx<T> (&v)[NF][EPC],
                                          cpx<T>* const (&H)[NF], bool ifft, const cpx<T>* twm) {
    const int ny = g.ny;
    if (ifft && ny > 1) {
        reg_fft<T, EPC, NF>(v, ct.buf, ct.fstride, ny, ct.t, g.TPC, twm, true);
        fft_sync(g.TPC);
    }
    if (ct.valid) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const int j = ct.t + g.TPC * e;
                if (j < ny) at32(H[f], ct.kx * ny + j) = v[f][e];
            }
        }
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double lane_d(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// Sum over the 64 lanes (all active), the same in every lane: a tree inside each
// row of 16 by data-parallel moves, then the four rows through scalar registers
// (six shuffles of a double through LDS cost about five times as long).
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_d<0xB1>(v);     // lanes ^ 1
    v += dpp_d<0x4E>(v);     // lanes ^ 2
    v += dpp_d<0x141>(v);    // the other four of eight
    v += dpp_d<0x140>(v);    // the other eight of sixteen
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_d<0xB1>(v));
    v = fmax(v, dpp_d<0x4E>(v));
    v = fmax(v, dpp_d<0x141>(v));
    v = fmax(v, dpp_d<0x140>(v));
    return fmax(fmax(lane_d(v, 0), lane_d(v, 16)), fmax(lane_d(v, 32), lane_d(v, 48)));
}

// ---------------------------------------------------------------------------
// Deterministic reductions.  Each block reduces NACC doubles in a fixed tree
// (wave sums, then waves in order) and writes them to partials[block]; every block
// of the next kernel sums the partials in the one order of partials_sum, so the
// result does not depend on scheduling and is the same in all of them.
// ---------------------------------------------------------------------------
template <int NACC>
__device__ __forceinline__ void block_wave_sums(double (&v)[NACC]) {
    if ((blockDim.x & 63) == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) v[a] = wave_sum(v[a]);
        return;
    }
#pragma unroll
    for (int a = 0; a < NACC; ++a) {   // blocks with lanes missing (the smallest grids)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[a] += __shfl_xor(v[a], off, 64);
    }
}
template <int NACC>
__device__ __forceinline__ void block_sum(double (&v)[NACC], double* red /*LDS, NACC*16*/) {
    block_wave_sums<NACC>(v);
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) red[a * 16 + wave] = v[a];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) {
            double s = 0.0;
            for (int w = 0; w < nw; ++w) s += red[a * 16 + w];
            v[a] = s;
        }
    }
    __syncthreads();
}

// block_sum with the same result in every thread, behind one LDS-only barrier: red
// must not be written again before another barrier of the block.
template <int NACC>
__device__ __forceinline__ void block_sum_all(double (&v)[NACC], double* red /*LDS, NACC*16*/) {
    block_wave_sums<NACC>(v);
    const int nw = (blockDim.x + 63) >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) red[a * 16 + (threadIdx.x >> 6)] = v[a];
    }
    block_lds_barrier();
#pragma unroll
    for (int a = 0; a < NACC; ++a) {
        double s = 0.0;
        for (int w = 0; w < nw; ++w) s += red[a * 16 + w];
        v[a] = s;
    }
}

// Sum of the per-block partials (layout partials[NACC*b + a]): place t of 256 adds blocks
// t, t+256, ... in order, then the fixed block tree.  The order, and so the value, is
// the same in every kernel that reduces the same partials, whatever its block size (128,
// or at least 256 threads; on 64 threads for up to 64 blocks).  Every thread of the
// block must call both steps.
// Two steps, so that a kernel can issue the partials' loads ahead
// of its data loads (a wait for a load also waits for every load issued before
// it): partials_fetch loads the partials of up to 256 PF_K blocks into registers,
// partials_sum adds them and those of any further blocks; the result is in every thread
// (see block_sum_all for red).
// No loop over the first ones: a load inside a loop makes the compiler wait for every
// load in flight at the loop entry.
constexpr int PF_K = 3;   // the column launches of 1024-point rows: 513 blocks
// V = 2: a block of 128 threads, each standing for two of the 256 (the same order).
template <int NACC, int V = 1>
__device__ __forceinline__ void partials_fetch(const double* __restrict__ partials, unsigned nblocks,
                                               double (&pb)[PF_K * V][NACC]) {
    // branch-free: every lane loads an in-range entry (predicated loads would
    // make the compiler wait for all loads); partials_sum drops the extra ones
#pragma unroll
    for (int k = 0; k < PF_K * V; ++k) {
        const unsigned b = threadIdx.x + (256u / V) * k;
        const unsigned bc = (threadIdx.x < 256 && b < nblocks) ? b : 0u;
#pragma unroll
        for (int a = 0; a < NACC; ++a) pb[k][a] = partials[(size_t)NACC * bc + a];
    }
}
template <int NACC, int V = 1>
__device__ __forceinline__ void partials_sum(const double* __restrict__ partials, unsigned nblocks,
                                             const double (&pb)[PF_K * V][NACC], double (&v)[NACC], double* red) {
    double acc[V][NACC];
#pragma unroll
    for (int i = 0; i < V; ++i)
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[i][a] = 0.0;
#pragma unroll
    for (int k = 0; k < PF_K * V; ++k) {
        const bool ok = threadIdx.x < 256 && threadIdx.x + (256u / V) * k < nblocks;
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[k % V][a] += ok ? pb[k][a] : 0.0;
    }
    if (nblocks > 256u * PF_K) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            for (unsigned b = threadIdx.x + (256u / V) * i + 256u * PF_K; threadIdx.x < 256 && b < nblocks; b += 256) {
#pragma unroll
                for (int a = 0; a < NACC; ++a) acc[i][a] += partials[(size_t)NACC * b + a];
            }
        }
    }
    if (V == 1) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) v[a] = acc[0][a];
        block_sum_all<NACC>(v, red);
        return;
    }
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        block_wave_sums<NACC>(acc[i]);
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int a = 0; a < NACC; ++a) red[a * 16 + i * (4 / V) + wave] = acc[i][a];
        }
    }
    block_lds_barrier();
#pragma unroll
    for (int a = 0; a < NACC; ++a) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) s += red[a * 16 + w];
        v[a] = s;
    }
}

// Maximum of the per-block partials by one block (order independent);
// the result is in thread 0.
template <int NACC>
__device__ __forceinline__ void final_max(const double* __restrict__ partials, unsigned nblocks,
                                          double (&v)[NACC], double* red) {
#pragma unroll
    for (int a = 0; a < NACC; ++a) v[a] = -1.0e308;
    for (unsigned b = threadIdx.x; b < nblocks; b += blockDim.x) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) v[a] = fmax(v[a], partials[(size_t)NACC * b + a]);
    }
#pragma unroll
    for (int a = 0; a < NACC; ++a) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[a] = fmax(v[a], __shfl_xor(v[a], off, 64));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) red[a * 16 + wave] = v[a];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) {
            double m = red[a * 16];
            for (int w = 1; w < nw; ++w) m = fmax(m, red[a * 16 + w]);
            v[a] = m;
        }
    }
    __syncthreads();
}

// Mode weight of the half spectrum for Parseval sums: kx = 0 and kx = nx/2 appear
// once in the full spectrum, every other kx twice (with its conjugate).
__device__ __forceinline__ double half_weight(int kx, int nx) {
    return (kx == 0 || 2 * kx == nx) ? 1.0 : 2.0;
}

// (sigma*, alpha*, kappa_ub) of Eq:FlatbathCoeff (flat), Eq:Optcoeff and
// Eq:Optcoeffb (kind 0) or Remark 4.2 (kind 1) from min eta, max eta,
// max(eta + lambda_+ eta |grad h|^2) and max |grad h|^2.  flat < 0 selects the
// flat formulas iff |grad h|_max = 0; the choice is returned in fl.
__host__ __device__ inline void coeffs_formula(double emin, double emax, double smx, double g2m, int flat, int kind,
                                               double& sig, double& alp, double& kap, int& fl) {
    const double lp = (4.0 + sqrt(13.0)) / 6.0;
    const double lm = (4.0 - sqrt(13.0)) / 6.0;
    const double ratio3 = (emax / emin) * (emax / emin) * (emax / emin);
    fl = flat < 0 ? (g2m == 0.0 ? 1 : 0) : (flat != 0 ? 1 : 0);
    if (fl) {
        sig = emax;
        alp = emax * emax * emax / 3.0;
        kap = ratio3;
    } else if (kind == 0) {
        sig = smx;
        alp = lp * emax * emax * emax;
        kap = fmax(smx / emin, (lp / lm) * ratio3);
    } else {
        sig = emax * (1.0 + lp * g2m);
        alp = lp * emax * emax * emax;
        kap = fmax((emax / emin) * (1.0 + lp * g2m), (lp / lm) * ratio3);
    }
}

}  // namespace sgn
