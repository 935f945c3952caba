// LDS-resident tile FFT engine for gfx950 (wave64).
//
// A tile holds W real pencils ("columns") of one transform axis.  Columns
// 2s and 2s+1 form complex sequence s (real part / imaginary part), so one
// complex FFT of length N = 2M transforms two real pencils at once.  The tile
// lives in LDS as a real array buf[row * rs + col] (rows 0..N-1, rs = W + 1:
// the odd padding keeps row-wise and column-wise accesses nearly free of
// bank conflicts); complex element (n, s) is (buf[n*rs + 2s], buf[n*rs + 2s+1]).
//
// Transform kinds built on the length-N complex FFT (M = N/2):
//   forward, zero padded : f_1..f_{M-1} at positions 1..M-1, zeros elsewhere;
//                          C[k] = sum_j f_j cos(pi k j/M), k = 0..M
//                          S[k] = sum_j f_j sin(pi k j/M), k = 1..M-1
//                          "slot" layout: row k = C[k], row M+k = S[k]
//                          (S alone is the raw DST-I)
//   forward, even        : f_0..f_M mirrored to length N; the spectrum is real,
//                          F[k] = f_0 + (-1)^k f_M + 2 sum_{j=1}^{M-1} f_j cos(pi k j/M)
//   inverse, hermitian   : from slots C, S: y_j = sum_{k=0}^{N-1} F_k e^{+i pi k j/M}
//                          with F_k = C_k - i S_k and F_{N-k} = conj(F_k), i.e.
//                          y_j = C_0 + (-1)^j C_M + 2 sum_{k=1}^{M-1}(C_k cos + S_k sin)
//
// The FFT itself is a Stockham autosort transform with radix-2/3/4/5/8
// butterflies held in registers (FP64 also 7, 11 and 13); larger prime factors
// take a dense product on the matrix cores (FP64) or direct sums (FP32).  Twiddles
// come from a table w[t] = exp(-2 pi i t/N) computed on the host in extended precision.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ips {

template <typename T>
struct alignas(2 * sizeof(T)) cx {
    T x, y;
};

template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

template <typename T>
__device__ __forceinline__ cx<T> cadd(cx<T> a, cx<T> b) { return {a.x + b.x, a.y + b.y}; }

template <typename T>
__device__ __forceinline__ cx<T> csub(cx<T> a, cx<T> b) { return {a.x - b.x, a.y - b.y}; }

// multiply by -i (forward) or +i (inverse); the direction is a template
// argument throughout the engine, so no per-element selects are emitted
template <typename T, bool INV>
__device__ __forceinline__ cx<T> rot90(cx<T> a)
{
    if constexpr (INV)
        return cx<T>{-a.y, a.x};
    else
        return cx<T>{a.y, -a.x};
}

constexpr int kMaxStages = 16;

// Transform lengths by the radices they need: any, powers of two (2, 4, 8), or
// no prime factor above 5.
enum LenKind { kAnyLen = 0, kPow2 = 1, kSmooth = 2 };

struct FftDesc {
    int N;   // transform length (even)
    int M;   // N / 2
    int nst; // number of Stockham stages
    int direct; // large prime radices as direct sums in every precision (mixed plans)
    int rad[kMaxStages];
    int ns[kMaxStages];          // product of the radices before the stage
    unsigned nsmag[kMaxStages];  // ceil(2^32 / ns) for ns not a power of two, else 0
    int nslg[kMaxStages];        // log2(ns) when ns is a power of two
};

// j mod ns for j < 2^16 (exact with the precomputed reciprocal)
__device__ __forceinline__ int fmod_ns(int j, int ns, unsigned mag, int lg)
{
    if (mag == 0) return j & (ns - 1);
    const int q = (int)__umulhi((unsigned)j, mag);
    return j - q * ns;
}

template <typename T>
__device__ __forceinline__ cx<T> lds_c(const T *buf, int rs, int n, int s)
{
    const T *p = buf + n * rs + 2 * s;
    return {p[0], p[1]};
}

template <typename T>
__device__ __forceinline__ void lds_cs(T *buf, int rs, int n, int s, cx<T> v)
{
    T *p = buf + n * rs + 2 * s;
    p[0] = v.x;
    p[1] = v.y;
}

template <typename T, bool INV>
__device__ __forceinline__ cx<T> twid(const cx<T> *tw, int t)
{
    cx<T> w = tw[t];
    if constexpr (INV) w.y = -w.y;
    return w;
}

// Last step of a length-8 DFT from the length-4 DFTs e of the even and o of
// the odd inputs: a[k] = e[k] + w8^k o[k], a[k+4] = e[k] - w8^k o[k].
template <typename T, bool INV>
__device__ __forceinline__ void dft8_combine(cx<T> *a, const cx<T> *e, const cx<T> *o)
{
    const T r = (T)0.70710678118654752440084436210484903928;
    cx<T> o1, o3;
    if constexpr (INV) {
        o1 = cx<T>{r * (o[1].x - o[1].y), r * (o[1].x + o[1].y)};
        o3 = cx<T>{-r * (o[3].x + o[3].y), r * (o[3].x - o[3].y)};
    } else {
        o1 = cx<T>{r * (o[1].x + o[1].y), r * (o[1].y - o[1].x)};
        o3 = cx<T>{r * (o[3].y - o[3].x), -r * (o[3].x + o[3].y)};
    }
    const cx<T> o2 = rot90<T, INV>(o[2]);
    a[0] = cadd(e[0], o[0]);
    a[4] = csub(e[0], o[0]);
    a[1] = cadd(e[1], o1);
    a[5] = csub(e[1], o1);
    a[2] = cadd(e[2], o2);
    a[6] = csub(e[2], o2);
    a[3] = cadd(e[3], o3);
    a[7] = csub(e[3], o3);
}

// Length-8 DFT of a[0..3] followed by four zeros: the first stage of a
// transform whose upper half of inputs is zero (zero-padded sequences).
template <typename T, bool INV>
__device__ __forceinline__ void dft8_lower(cx<T> *a)
{
    const cx<T> r2 = rot90<T, INV>(a[2]), r3 = rot90<T, INV>(a[3]);
    const cx<T> e[4] = {cadd(a[0], a[2]), cadd(a[0], r2), csub(a[0], a[2]), csub(a[0], r2)};
    const cx<T> o[4] = {cadd(a[1], a[3]), cadd(a[1], r3), csub(a[1], a[3]), csub(a[1], r3)};
    dft8_combine<T, INV>(a, e, o);
}

// In-register DFT of odd prime length R from the sums a_r + a_{R-r} and the
// differences a_r - a_{R-r}: with A_q the cosine sum of the first and B_q the
// sine sum of the second, X_q and X_{R-q} are A_q + and - rot90(B_q), a quarter
// of the multiplications of the direct sums. The roots are read from the table
// (literals would be hoisted out of the loop over the stages and held in
// registers throughout: 224 instead of 140 VGPRs per thread).
template <int R, bool INV>
__device__ __forceinline__ void dft_odd(cx<double> *a, const cx<double> *tw, int N)
{
    constexpr int H = (R - 1) / 2;
    cx<double> w[H];
#pragma unroll
    for (int m = 1; m <= H; ++m) w[m - 1] = tw[m * (N / R)]; // (cos, -sin) 2 pi m / R
    cx<double> x0 = a[0];
#pragma unroll
    for (int r = 1; r <= H; ++r) {
        const cx<double> t = a[r];
        a[r] = cadd(t, a[R - r]);
        a[R - r] = csub(t, a[R - r]);
        x0 = cadd(x0, a[r]);
    }
    cx<double> p[H], q[H];
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        cx<double> A = a[0], B = {0.0, 0.0};
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            const int m = (r * k) % R;
            const double c = w[(m <= H ? m : R - m) - 1].x;
            const double sn = m <= H ? -w[m - 1].y : w[R - m - 1].y;
            A.x = fma(c, a[r].x, A.x);
            A.y = fma(c, a[r].y, A.y);
            B.x = fma(sn, a[R - r].x, B.x);
            B.y = fma(sn, a[R - r].y, B.y);
        }
        const cx<double> t = rot90<double, INV>(B);
        p[k - 1] = cadd(A, t);
        q[k - 1] = csub(A, t);
    }
    a[0] = x0;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        a[k] = p[k - 1];
        a[R - k] = q[k - 1];
    }
}

// In-register DFT of length R (forward: exp(-2 pi i/R); inverse: conjugate).
template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_small(cx<T> *a, const cx<T> *tw, int N)
{
    if constexpr (R == 2) {
        cx<T> t = a[1];
        a[1] = csub(a[0], t);
        a[0] = cadd(a[0], t);
    } else if constexpr (R == 4) {
        cx<T> s02 = cadd(a[0], a[2]), d02 = csub(a[0], a[2]);
        cx<T> s13 = cadd(a[1], a[3]), d13 = rot90<T, INV>(csub(a[1], a[3]));
        a[0] = cadd(s02, s13);
        a[2] = csub(s02, s13);
        a[1] = cadd(d02, d13);
        a[3] = csub(d02, d13);
    } else if constexpr (R == 8) {
        cx<T> e[4] = {a[0], a[2], a[4], a[6]};
        cx<T> o[4] = {a[1], a[3], a[5], a[7]};
        dft_small<T, 4, INV>(e, tw, N);
        dft_small<T, 4, INV>(o, tw, N);
        dft8_combine<T, INV>(a, e, o);
    } else if constexpr (R == 3) {
        // w3 = -1/2 -/+ i sqrt(3)/2:  X1,2 = a0 - (a1 + a2)/2 +/- rot90((sqrt(3)/2)(a1 - a2))
        const T h = (T)0.86602540378443864676372317075293618347;
        const cx<T> t1 = cadd(a[1], a[2]);
        const cx<T> t2 = {a[0].x - (T)0.5 * t1.x, a[0].y - (T)0.5 * t1.y};
        const cx<T> t3 = rot90<T, INV>(cx<T>{h * (a[1].x - a[2].x), h * (a[1].y - a[2].y)});
        a[0] = cadd(a[0], t1);
        a[1] = cadd(t2, t3);
        a[2] = csub(t2, t3);
    } else if constexpr (R == 5) {
        // with b1 = a1 + a4, b2 = a2 + a3, d1 = a1 - a4, d2 = a2 - a3 and
        // c_m = cos(2 pi m/5), s_m = sin(2 pi m/5):
        //   X1,4 = a0 + c1 b1 + c2 b2 +/- rot90(s1 d1 + s2 d2)
        //   X2,3 = a0 + c2 b1 + c1 b2 +/- rot90(s2 d1 - s1 d2)
        const T c1 = (T)0.30901699437494742410229341718281905886, c2 = (T)-0.80901699437494742410229341718281905886;
        const T s1 = (T)0.95105651629515357211643933337938214340, s2 = (T)0.58778525229247312916870595463907276860;
        const cx<T> b1 = cadd(a[1], a[4]), b2 = cadd(a[2], a[3]), d1 = csub(a[1], a[4]), d2 = csub(a[2], a[3]);
        const cx<T> t1 = {a[0].x + c1 * b1.x + c2 * b2.x, a[0].y + c1 * b1.y + c2 * b2.y};
        const cx<T> t2 = {a[0].x + c2 * b1.x + c1 * b2.x, a[0].y + c2 * b1.y + c1 * b2.y};
        const cx<T> u1 = rot90<T, INV>(cx<T>{s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y});
        const cx<T> u2 = rot90<T, INV>(cx<T>{s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y});
        a[0] = cadd(a[0], cadd(b1, b2));
        a[1] = cadd(t1, u1);
        a[4] = csub(t1, u1);
        a[2] = cadd(t2, u2);
        a[3] = csub(t2, u2);
    } else {
        static_assert(sizeof(T) == 8, "FP32 tiles take direct sums for these radices");
        dft_odd<R, INV>(a, tw, N);
    }
}

// One Stockham stage of radix R (R <= 13) over nseq = 2^lgs sequences of
// length N.  MAXE bounds the complex elements a thread holds
// (nseq * N <= MAXE * NT).
template <typename T, int R, int MAXE, int NT, bool INV>
__device__ __forceinline__ void stage_bfly(T *buf, int rs, int lgs, const FftDesc &fd, int st,
                                           const cx<T> *tw, int tid)
{
    constexpr int BPT = (MAXE + R - 1) / R;
    const int N = fd.N, Ns = fd.ns[st];
    const int NR = N / R;
    const int nbf = (NR << lgs);
    const int tstep = N / (Ns * R);
    const int smask = (1 << lgs) - 1;
    cx<T> v[BPT][R];
    int base[BPT];
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const int b = tid + i * NT;
        if (b < nbf) {
            const int s = b & smask, j = b >> lgs;
            const int jm = fmod_ns(j, Ns, fd.nsmag[st], fd.nslg[st]);
            base[i] = (j - jm) * R + jm;
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = lds_c(buf, rs, j + r * NR, s);
            if (jm != 0) {
                const int e = jm * tstep;
#pragma unroll
                for (int r = 1; r < R; ++r) v[i][r] = cmul(v[i][r], twid<T, INV>(tw, e * r));
            }
            dft_small<T, R, INV>(v[i], tw, N);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const int b = tid + i * NT;
        if (b < nbf) {
            const int s = b & smask;
#pragma unroll
            for (int r = 0; r < R; ++r) lds_cs(buf, rs, base[i] + r * Ns, s, v[i][r]);
        }
    }
    __syncthreads();
}

// floor(x / d) = __umulhi(x, recip_u(d)) for 0 <= x < 2^16, 2 <= d < 2^16.
__device__ __forceinline__ unsigned recip_u(int d) { return 0xffffffffu / (unsigned)d + 1u; }

// Most items of a direct stage per thread: at most MAXE NT / (R ST) groups times
// ceil(R / QT), most groups per frequency at R = 7 (4 of 2, 2 of 4), 13 (4 of 4) and
// 11 (2 of 8).
template <int MAXE, int ST, int QT>
constexpr int direct_items()
{
    constexpr int R = QT == 1 ? 1 : QT == 2 ? 7 : QT == 4 ? 13 : 11, G = QT == 1 ? 1 : QT == 8 ? 2 : 4;
    return (MAXE * G + ST * R - 1) / (ST * R);
}

// Stockham stage of any radix as direct sums. A thread forms ST * QT outputs,
// QT neighbouring frequencies of ST sequences, so that an input read from LDS
// serves QT outputs and a twiddle ST (one output at a time was bound by its two
// LDS reads per input, 16 bytes for four FP32 operations).
template <typename T, int MAXE, int NT, bool INV, int ST, int QT>
__device__ __forceinline__ void stage_direct(T *buf, int rs, int lgs, const FftDesc &fd, int st,
                                                    const cx<T> *tw, int tid)
{
    constexpr int IPT = direct_items<MAXE, ST, QT>();
    const int N = fd.N, Ns = fd.ns[st], R = fd.rad[st];
    const int NR = N / R, tstep = N / (Ns * R);
    const int ncg = (NR << lgs) / ST;  // (position, group of ST sequences)
    const int nqg = (R + QT - 1) / QT;
    const int items = ncg * nqg, lgsg = lgs - (ST == 2 ? 1 : 0);
    const unsigned mag = recip_u(ncg);
    cx<T> acc[IPT][QT][ST];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int e = tid + i * NT;
        if (e >= items) continue;
        const int qg = (int)__umulhi((unsigned)e, mag), cg = e - qg * ncg;
        const int s0 = (cg & ((1 << lgsg) - 1)) * ST, j = cg >> lgsg;
        const int jm = fmod_ns(j, Ns, fd.nsmag[st], fd.nslg[st]);
        int E[QT], ex[QT];
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            const int q = min(qg * QT + u, R - 1);
            E[u] = jm * tstep + q * NR; // exponent per input index r, in units of w_N
            ex[u] = 0;
        }
#pragma unroll
        for (int v = 0; v < ST; ++v) {
            const cx<T> x = lds_c(buf, rs, j, s0 + v);
#pragma unroll
            for (int u = 0; u < QT; ++u) acc[i][u][v] = x;
        }
        for (int r = 1; r < R; ++r) {
            cx<T> x[ST];
#pragma unroll
            for (int v = 0; v < ST; ++v) x[v] = lds_c(buf, rs, j + r * NR, s0 + v);
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                ex[u] += E[u];
                if (ex[u] >= N) ex[u] -= N;
                const cx<T> w = twid<T, INV>(tw, ex[u]);
#pragma unroll
                for (int v = 0; v < ST; ++v) acc[i][u][v] = cadd(acc[i][u][v], cmul(x[v], w));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int e = tid + i * NT;
        if (e >= items) continue;
        const int qg = (int)__umulhi((unsigned)e, mag), cg = e - qg * ncg;
        const int s0 = (cg & ((1 << lgsg) - 1)) * ST, j = cg >> lgsg;
        const int jm = fmod_ns(j, Ns, fd.nsmag[st], fd.nslg[st]);
        const int base = (j - jm) * R + jm;
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            const int q = qg * QT + u;
            if (q < R) {
#pragma unroll
                for (int v = 0; v < ST; ++v) lds_cs(buf, rs, base + q * Ns, s0 + v, acc[i][u][v]);
            }
        }
    }
    __syncthreads();
}

typedef double v4d __attribute__((ext_vector_type(4)));

// The value of the neighbouring lane (lane ^ 1).
__device__ __forceinline__ double swap_pair(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xF, 0xF, true); // quad_perm [1,0,3,2]
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Most 16 x 16 output blocks of stage_prime per wave.
constexpr int kPrimeBlocks = 4;

// Blocks of stage_prime: 16 frequencies (of 0..(R-1)/2) by 16 real columns.
__device__ __forceinline__ int prime_blocks(const FftDesc &fd, int st, int lgs)
{
    const int R = fd.rad[st], ncol = (fd.N / R) << (lgs + 1);
    return ((R + 1) / 2 + 15) / 16 * ((ncol + 15) >> 4);
}

// FP64 Stockham stage of an odd prime radix R on the matrix cores. The inputs
// are replaced in LDS by the (twiddled) sums a_r = x_r + x_{R-r} and differences
// b_r = x_r - x_{R-r}, r = 1..h, h = (R-1)/2; then with the real columns of the
// tile at all N/R positions as columns,
//   A_q = x_0 + sum_r cos(2 pi q r/R) a_r,   B_q = sum_r sin(2 pi q r/R) b_r
// are two (h+1) x h by h x columns products, and X_q, X_{R-q} = A_q -/+ i B_q:
// half of the multiplications of the direct sums, in 16 x 16 x 4 MFMAs whose
// operands cost 32 bytes of LDS reads per 32 multiply-adds of a lane (direct sums
// one output at a time: 32 bytes per 4, which bound them). With the shared direct
// sums and the register radices: 64 boxes of 33..193 nodes 22.1 -> 12.4 ms,
// 182x174x167 6.40 -> 1.91 ms, 97x90x113 0.69 -> 0.35 ms. One wave owns a block's cosine and
// sine sums. A lane's four results are rows 4 v + lane/16, column lane & 15; the
// real and imaginary parts of a sequence are neighbouring columns, so B_q's other
// part comes from the neighbouring lane.
template <int NT, bool INV>
__device__ __forceinline__ void stage_prime(double *buf, int rs, int lgs, const FftDesc &fd, int st,
                                            const cx<double> *tw, int tid)
{
    const int N = fd.N, Ns = fd.ns[st], R = fd.rad[st];
    const int NR = N / R, h = (R - 1) / 2, tstep = N / (Ns * R);
    const int lgW = lgs + 1, smask = (1 << lgs) - 1;
    {
        const int ncx = NR << lgs; // (position, sequence) pairs
        const unsigned mag = recip_u(ncx);
        for (int e = tid; e < h * ncx; e += NT) {
            const int r1 = (int)__umulhi((unsigned)e, mag), cj = e - r1 * ncx, r = r1 + 1;
            const int s = cj & smask, j = cj >> lgs;
            const int jm = fmod_ns(j, Ns, fd.nsmag[st], fd.nslg[st]);
            cx<double> u = lds_c(buf, rs, j + r * NR, s), v = lds_c(buf, rs, j + (R - r) * NR, s);
            if (jm != 0) {
                u = cmul(u, twid<double, INV>(tw, jm * tstep * r));
                v = cmul(v, twid<double, INV>(tw, jm * tstep * (R - r)));
            }
            lds_cs(buf, rs, j + r * NR, s, cadd(u, v));
            lds_cs(buf, rs, j + (R - r) * NR, s, csub(u, v));
        }
    }
    __syncthreads();
    const int lane = tid & 63, lm = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncol = NR << lgW, ncb = (ncol + 15) >> 4, nblk = ncb * ((h + 16) >> 4);
    v4d A[kPrimeBlocks], B[kPrimeBlocks];
#pragma unroll
    for (int i = 0; i < kPrimeBlocks; ++i) {
        const int b = wave + i * (NT / 64);
        if (b >= nblk) continue;
        const int qb = b / ncb, col = min((b - qb * ncb) * 16 + lm, ncol - 1);
        const int j = col >> lgW, c = col & ((1 << lgW) - 1);
        const double *p = buf + j * rs + c;
        const int pitch = NR * rs;
        const double x0 = p[0];
        A[i] = v4d{x0, x0, x0, x0};
        B[i] = v4d{0.0, 0.0, 0.0, 0.0};
        // row q of the cosines and sines, r = 1 + lk + 4 step; q r mod R by steps
        // (rows beyond h are computed and not used)
        const int q = min(qb * 16 + lm, h);
        const unsigned magR = recip_u(R);
        auto modR = [&](int x) { return x - (int)__umulhi((unsigned)x, magR) * R; };
        int m = modR(q * (1 + lk));
        const int dm = modR(4 * q);
        for (int r0 = 1; r0 <= h; r0 += 4) {
            const int r = min(r0 + lk, h);
            const bool in = r0 + lk <= h;
            const cx<double> w = tw[m * NR];
            const double a = p[r * pitch], d = p[(R - r) * pitch];
            m += dm;
            if (m >= R) m -= R;
            A[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? w.x : 0.0, a, A[i], 0, 0, 0);
            B[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? -w.y : 0.0, d, B[i], 0, 0, 0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPrimeBlocks; ++i) {
        const int b = wave + i * (NT / 64);
        if (b >= nblk) continue;
        const int qb = b / ncb, col = (b - qb * ncb) * 16 + lm;
        const int j = min(col, ncol - 1) >> lgW, c = col & ((1 << lgW) - 1);
        const int jm = fmod_ns(j, Ns, fd.nsmag[st], fd.nslg[st]);
        double *p = buf + ((j - jm) * R + jm) * rs + c;
        const int pitch = Ns * rs;
        // X_q = A_q - i B_q (forward): real part A.x + B.y, imaginary A.y - B.x
        const bool plus = ((lm & 1) == 0) != INV;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double o = swap_pair(B[i][v]);
            const int q = qb * 16 + 4 * v + lk;
            if (q <= h && col < ncol) {
                p[q * pitch] = plus ? A[i][v] + o : A[i][v] - o;
                if (q > 0) p[(R - q) * pitch] = plus ? A[i][v] - o : A[i][v] + o;
            }
        }
    }
    __syncthreads();
}

// Whether the direct sums of a stage of radix R at NR positions share their reads
// (see stage_direct): not where that leaves threads idle, i.e. where the rounds of items
// that a thread goes through, times the LDS reads of an input, are fewer one output at a
// time. Mixed plans, one output at a time -> shared: 98^3 solve (R = 97, full tiles) 1001
// -> 572 us, adjoint of 603^2 (43) 446 -> 412; adjoint of 1000^2 (37) 617 -> 712, of 212^2
// (211, narrow tiles) 424 -> 718, solve of 14^3 (13) 139 -> 170.
template <bool F64, int NT>
__host__ __device__ __forceinline__ bool direct_shared(int R, int NR, int lgs)
{
    const int S = lgs > 0 ? 2 : 1, Q = (F64 ? 4 : 8) / S, np = NR << lgs;
    const int si = np / S * ((R + Q - 1) / Q); // items, shared
    return (si + NT - 1) / NT * (S + Q) <= (np * R + NT - 1) / NT * 2;
}

// Stockham stage of any other radix. FP64 plans: 7, 11 and 13 in registers, larger
// primes on the matrix cores while a wave holds the blocks (all lengths up to
// 1024). Otherwise direct sums. In the mixed modes (fd.direct) every transform
// takes those: the sixth-order symbol multiplies the rounding of the FP64 face
// spectra by up to (M pi)^4, so that another order of their sums would move the
// FP32 results by up to their own rounding (182x174x167: 6e-9, and 2e-8).
template <typename T, int MAXE, int NT, bool INV>
__device__ __forceinline__ void stage_other(T *buf, int rs, int lgs, const FftDesc &fd, int st, const cx<T> *tw,
                                            int tid)
{
    if constexpr (sizeof(T) == 8) {
        if (!fd.direct) {
            const int R = fd.rad[st];
            if (R == 7) return stage_bfly<T, 7, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, tid);
            if (R == 11) return stage_bfly<T, 11, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, tid);
            if (R == 13) return stage_bfly<T, 13, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, tid);
            if (prime_blocks(fd, st, lgs) <= kPrimeBlocks * (NT / 64))
                return stage_prime<NT, INV>(buf, rs, lgs, fd, st, tw, tid);
        }
    }
    // outputs per item: half as many held registers in FP64
    constexpr int Q2 = sizeof(T) == 8 ? 2 : 4;
    if (direct_shared<sizeof(T) == 8, NT>(fd.rad[st], fd.N / fd.rad[st], lgs)) {
        if (lgs > 0)
            stage_direct<T, MAXE, NT, INV, 2, Q2>(buf, rs, lgs, fd, st, tw, tid);
        else
            stage_direct<T, MAXE, NT, INV, 1, 2 * Q2>(buf, rs, lgs, fd, st, tw, tid);
    } else {
        stage_direct<T, MAXE, NT, INV, 1, 1>(buf, rs, lgs, fd, st, tw, tid);
    }
}

// Stockham stage with every size known at compile time: transform length
// N, radix R, product of the earlier radices NS (a power of two), row pitch
// RS and 2^LGS sequences.  Same data movement as stage_bfly; the index and
// twiddle arithmetic folds to shifts and constants.
template <typename T, int R, int NT, int N, int NS, int RS, int LGS, bool INV>
__device__ __forceinline__ void stage_ct(T *buf, const cx<T> *tw, int tid)
{
    constexpr int NR = N / R, NBF = NR << LGS, TSTEP = N / (NS * R), SMASK = (1 << LGS) - 1;
    constexpr int BPT = (NBF + NT - 1) / NT;
    cx<T> v[BPT][R];
    int base[BPT];
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const int b = tid + i * NT;
        if (NBF % NT == 0 || b < NBF) {
            const int sq = b & SMASK, j = b >> LGS;
            const int jm = j & (NS - 1);
            base[i] = (j - jm) * R + jm;
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = lds_c(buf, RS, j + r * NR, sq);
            if (NS > 1 && jm != 0) {
                const int e = jm * TSTEP;
#pragma unroll
                for (int r = 1; r < R; ++r) v[i][r] = cmul(v[i][r], twid<T, INV>(tw, e * r));
            }
            dft_small<T, R, INV>(v[i], tw, N);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const int b = tid + i * NT;
        if (NBF % NT == 0 || b < NBF) {
            const int sq = b & SMASK;
#pragma unroll
            for (int r = 0; r < R; ++r) lds_cs(buf, RS, base[i] + r * NS, sq, v[i][r]);
        }
    }
    __syncthreads();
}

// Compile-time transforms for the common power-of-two lengths at the
// default tile widths (radix-8 stages first, as factor_fft orders them).
// tid: the thread index (a caller that runs several transforms in a loop
// may pass one the compiler cannot see through, so that the per-thread index
// and twiddle values are recomputed for each transform instead of being held
// in registers across the loop).
template <typename T, int NT, int N, int RS, int LGS, bool INV>
__device__ __forceinline__ void fft_ct(T *buf, const cx<T> *tw, int tid)
{
    if constexpr (N == 256) {
        stage_ct<T, 8, NT, N, 1, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 8, NT, N, 8, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 4, NT, N, 64, RS, LGS, INV>(buf, tw, tid);
    } else if constexpr (N == 512) {
        stage_ct<T, 8, NT, N, 1, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 8, NT, N, 8, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 8, NT, N, 64, RS, LGS, INV>(buf, tw, tid);
    } else if constexpr (N == 1024) {
        stage_ct<T, 8, NT, N, 1, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 8, NT, N, 8, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 8, NT, N, 64, RS, LGS, INV>(buf, tw, tid);
        stage_ct<T, 2, NT, N, 512, RS, LGS, INV>(buf, tw, tid);
    }
}

// Element offset r * rsd + c * csd of a tile in 32-bit arithmetic with
// 24-bit multiplies: the launchers check that strides stay below 2^23 and a
// tile spans less than 2^31 elements (true for every supported grid).
__device__ __forceinline__ int toff(int r, int64_t rsd, int c, int64_t csd)
{
    return __mul24(r, (int)rsd) + __mul24(c, (int)csd);
}

// Radix of the last stage of the compile-time transforms.
template <int N>
struct CtLast {
    static constexpr int R = N == 256 || N == 2048 ? 4 : N == 512 || N == 4096 ? 8 : 2;
};

// ---------------------------------------------------------------------------
// Register tiles: N = 256 .. 8192 (a power of two), 2048 / N sequences (one from
// N = 2048 on), one radix-8 butterfly per thread in every stage.
//
// The tile is an array of complex elements, row-major, with one row of padding
// after every eight: elements are aligned, so each is one 8- or 16-byte LDS
// access, and the stride-8 row writes of the first stage, the block writes of the
// later ones and the consecutive rows that every stage reads each fall on all banks
// evenly (row pitch W + 1 took two accesses per element, with conflicts).
//
// The last stage of a transform leaves thread (j, s) with rows j + r N/8, r < 8,
// of sequence s in registers, and the first stage of the next one starts from
// the same rows. With j assigned to the threads in pairs (j, N/8 - j) of lanes that
// mirror each other, row N - k of a row k lies in the mirror lane, so whatever
// combines rows k and N - k (cosine and sine parts, the spectral combination)
// works on registers with one cross-lane move per value instead of two or four
// passes over the tile in LDS.
// ---------------------------------------------------------------------------
template <int LEN, int SEQS = (LEN >= 2048 ? 1 : 2048 / LEN)>
struct RegTile {
    static constexpr int N = LEN, NSEQ = SEQS, W = 2 * NSEQ;
    static constexpr int LGS = NSEQ == 8 ? 3 : NSEQ == 4 ? 2 : NSEQ == 2 ? 1 : 0;
    static constexpr int P = N / 8;          // rows between the elements of a thread
    static constexpr int NTH = P * NSEQ;     // threads of the block
    static constexpr int ELEMS = (N + N / 8) * NSEQ; // LDS elements
    static constexpr bool LTW = N <= 2048;   // twiddles in LDS (else the global table)
    // lane ^ (2 NSEQ - 1): row_mirror, row_half_mirror, quad_perm [3,2,1,0], [1,0,3,2]
    static constexpr int MIRROR = NSEQ == 8 ? 0x140 : NSEQ == 4 ? 0x141 : NSEQ == 2 ? 0x1B : 0xB1;
    // a column's rows one after the other (sequence s at s * SP): 16 dwords off a
    // multiple of the 64 banks per sequence in FP32
    static constexpr int SP = N + 8;
};

// LDS bytes of a register tile and its twiddles.
template <typename T, typename R>
constexpr size_t rt_lds()
{
    return ((R::LTW ? R::N : 0) + R::ELEMS) * sizeof(cx<T>);
}

template <typename R>
__device__ __forceinline__ constexpr int rt_row(int row)
{
    return (row + (row >> 3)) * R::NSEQ;
}

template <typename T>
__device__ __forceinline__ cx<T> rt_get(const cx<T> *p)
{
    typedef T V __attribute__((ext_vector_type(2)));
    const V v = *reinterpret_cast<const V *>(p);
    return {v.x, v.y};
}

template <typename T>
__device__ __forceinline__ void rt_put(cx<T> *p, cx<T> v)
{
    typedef T V __attribute__((ext_vector_type(2)));
    *reinterpret_cast<V *>(p) = V{v.x, v.y};
}

// Thread -> (j, s), and the paired form.
template <typename R>
__device__ __forceinline__ void rt_plain(int tid, int &j, int &s)
{
    j = tid >> R::LGS;
    s = tid & (R::NSEQ - 1);
}

template <typename R>
__device__ __forceinline__ void rt_paired(int tid, int &j, int &s)
{
    const int u = tid >> R::LGS, m = u >> 1, odd = u & 1, l = tid & (R::NSEQ - 1);
    j = odd ? (m ? R::P - m : R::P / 2) : m;
    s = odd ? R::NSEQ - 1 - l : l;
}

template <typename R>
__device__ __forceinline__ float rt_mirror(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), R::MIRROR, 0xF, 0xF, true));
}

template <typename R>
__device__ __forceinline__ double rt_mirror(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), R::MIRROR, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), R::MIRROR, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Rows N - k of the rows k = j + r N/8, r < 4, of a paired thread, from the rows
// a[0..7] of its own and its mirror thread (k = 0: itself).
template <typename T, typename R>
__device__ __forceinline__ void rt_reflect(const cx<T> (&a)[8], int j, cx<T> (&b)[4])
{
    // (selects on values: a branch would make the compiler address the arrays)
    const bool z = j == 0, h = j == R::P / 2;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cx<T> t0 = a[(8 - r) & 7], t1 = a[7 - r];
        const cx<T> m = {rt_mirror<R>(t1.x), rt_mirror<R>(t1.y)};
        b[r].x = z ? t0.x : h ? t1.x : m.x;
        b[r].y = z ? t0.y : h ? t1.y : m.y;
    }
}

// The inverse: rows j + r N/8, r = 4..7, of an odd sequence (row N - k the negative
// of row k, rows 0 and N/2 zero) from its rows k = j + r N/8, r < 4, in a[0..3] of
// the thread and its mirror.
template <typename T, typename R>
__device__ __forceinline__ void rt_unfold_odd(cx<T> (&a)[8], int j)
{
    const bool z = j == 0, h = j == R::P / 2;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cx<T> t1 = a[r];
        const cx<T> m = {rt_mirror<R>(t1.x), rt_mirror<R>(t1.y)};
        // row j + (7 - r) N/8; of j = 0: row (4 + (3 - r)) N/8, the mirror of row (r + 1) N/8
        const cx<T> t8 = r < 3 ? a[r + 1] : cx<T>{(T)0, (T)0};
        a[7 - r].x = -(z ? t8.x : h ? t1.x : m.x);
        a[7 - r].y = -(z ? t8.y : h ? t1.y : m.y);
    }
}

// Inputs of the hermitian synthesis from the cosine rows C and sine rows S of k = j +
// r N/8, r < 4 (of k = 0: S holds row N/2): z(k) = C + i-swapped S, the upper rows
// N - k from the mirror lane (of j = 0 the thread's own).
template <typename T, typename R>
__device__ __forceinline__ void rt_unfold_herm(const cx<T> (&C)[4], const cx<T> (&S)[4], int j, cx<T> (&v)[8])
{
    const bool z0 = j == 0, h = j == R::P / 2;
    cx<T> up[4];
    const cx<T> cm = S[0];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const T sa = r == 0 && z0 ? (T)0 : S[r].x, sb = r == 0 && z0 ? (T)0 : S[r].y;
        v[r] = cx<T>{C[r].x + sb, C[r].y - sa};
        up[r] = cx<T>{C[r].x - sb, C[r].y + sa}; // row N - k
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cx<T> own = r < 3 ? up[r + 1] : cm;
        const cx<T> m = {rt_mirror<R>(up[r].x), rt_mirror<R>(up[r].y)};
        v[7 - r].x = z0 ? own.x : h ? up[r].x : m.x;
        v[7 - r].y = z0 ? own.y : h ? up[r].y : m.y;
    }
}

// First stage (radix 8): rows j + r N/8 in a, written to the tile.
template <typename T, typename R, bool INV>
__device__ __forceinline__ void rt_first(cx<T> *buf, cx<T> (&a)[8], int j, int s)
{
    rt_pin(a);
    dft_small<T, 8, INV>(a, nullptr, R::N);
    cx<T> *p = buf + 9 * j * R::NSEQ + s;
#pragma unroll
    for (int r = 0; r < 8; ++r) rt_put(p + r * R::NSEQ, a[r]);
    __syncthreads();
}

// As rt_first for rows N/2.. that are zero (a[0..3] given).
template <typename T, typename R>
__device__ __forceinline__ void rt_first_zpad(cx<T> *buf, cx<T> (&a)[8], int j, int s)
{
    dft8_lower<T, false>(a);
    cx<T> *p = buf + 9 * j * R::NSEQ + s;
#pragma unroll
    for (int r = 0; r < 8; ++r) rt_put(p + r * R::NSEQ, a[r]);
    __syncthreads();
}

template <typename T, typename R>
__device__ __forceinline__ void rt_rows(const cx<T> *buf, cx<T> (&a)[8], int j, int s)
{
    const cx<T> *p = buf + rt_row<R>(j) + s;
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = rt_get(p + r * rt_row<R>(R::P));
}

// One radix-8 stage in LDS after product NS of earlier radices.
template <typename T, typename R, int NS, bool INV>
__device__ __forceinline__ void rt_stage(cx<T> *buf, const cx<T> *tw, int tid)
{
    int j, s;
    rt_plain<R>(tid, j, s);
    cx<T> a[8];
    rt_rows<T, R>(buf, a, j, s);
    const int jm = j & (NS - 1);
    if (jm != 0) {
        const int e = jm * (R::N / (NS * 8));
#pragma unroll
        for (int r = 1; r < 8; ++r) a[r] = cmul(a[r], twid<T, INV>(tw, e * r));
    }
    dft_small<T, 8, INV>(a, tw, R::N);
    __syncthreads();
    cx<T> *p = buf + rt_row<R>((j - jm) * 8 + jm) + s;
#pragma unroll
    for (int r = 0; r < 8; ++r) rt_put(p + r * rt_row<R>(NS), a[r]);
    __syncthreads();
}

// The stages between the first and the last.
template <typename T, typename R, bool INV>
__device__ __forceinline__ void rt_middle(cx<T> *buf, const cx<T> *tw, int tid)
{
    rt_stage<T, R, 8, INV>(buf, tw, tid);
    if constexpr (R::N >= 1024) rt_stage<T, R, 64, INV>(buf, tw, tid);
    if constexpr (R::N >= 8192) rt_stage<T, R, 512, INV>(buf, tw, tid);
}

// Values as they come back from memory: keeps the compiler from contracting an
// operation on them with the one that made them (so that results do not depend
// on where a value is kept).
template <typename T, int K>
__device__ __forceinline__ void rt_pin(cx<T> (&a)[K])
{
#pragma unroll
    for (int r = 0; r < K; ++r) asm volatile("" : "+v"(a[r].x), "+v"(a[r].y));
}

// The last stage (radix 4, 8 or 2 for N = 256, 512, 1024, and so on): rows j + r N/8 of the
// result in a. No barrier.
template <typename T, typename R, bool INV>
__device__ __forceinline__ void rt_last(const cx<T> *buf, const cx<T> *tw, cx<T> (&a)[8], int j, int s)
{
    constexpr int RX = CtLast<R::N>::R, NB = 8 / RX; // NB butterflies of radix RX
    rt_rows<T, R>(buf, a, j, s);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int e = j + i * R::P;
        cx<T> v[RX];
#pragma unroll
        for (int r = 0; r < RX; ++r) v[r] = a[i + NB * r];
        if (e != 0) {
#pragma unroll
            for (int r = 1; r < RX; ++r) v[r] = cmul(v[r], twid<T, INV>(tw, e * r));
        }
        dft_small<T, RX, INV>(v, tw, R::N);
#pragma unroll
        for (int r = 0; r < RX; ++r) a[i + NB * r] = v[r];
    }
    rt_pin(a);
}

// Cosine and sine parts of a zero-padded forward transform (rows a of a paired
// thread): C and S of rows k = j + r N/8, r < 4, of both columns; S of k = 0 is
// C_{N/2}, as in the slot layout.
template <typename T, typename R>
__device__ __forceinline__ void rt_slots(const cx<T> (&a)[8], int j, cx<T> (&C)[4], cx<T> (&S)[4])
{
    cx<T> b[4];
    rt_reflect<T, R>(a, j, b);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        C[r] = cx<T>{(T)0.5 * (a[r].x + b[r].x), (T)0.5 * (a[r].y + b[r].y)};
        S[r] = cx<T>{(T)0.5 * (b[r].y - a[r].y), (T)0.5 * (a[r].x - b[r].x)};
    }
    S[0].x = j == 0 ? a[4].x : S[0].x;
    S[0].y = j == 0 ? a[4].y : S[0].y;
}

// Two neighbouring elements as one access (element-aligned only, which global
// memory instructions take).
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) pair_t {
    T a, b;
};

// Rows t = j + r N/8, r < 4, of columns 2s and 2s + 1 from global memory: source
// row t - row0 (row0 = 1: row t = 0 is zero). Element (row, column) is
// src[row*rsd + col], with col0, col1 the offsets of the two columns (negative:
// zero). dir = 1 or -1: col1 = col0 + dir for every thread of the block, read
// together (two single loads cost two passes over the same cache lines).
template <typename TI, typename R>
__device__ __forceinline__ void rt_fetch(TI (&x)[8], const TI *src, int64_t rsd, int col0, int col1, int dir, int j,
                                         int row0)
{
    const int step = __mul24(R::P, (int)rsd);
    int o = __mul24(j - row0, (int)rsd);
    const bool first = j >= row0;
    if (dir != 0) {
        const int c = min(col0, col1);
        const bool rev = dir < 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = r > 0 || first;
            const pair_t<TI> v = *reinterpret_cast<const pair_t<TI> *>(src + (ok ? o : 0) + c);
            x[2 * r] = ok ? (rev ? v.b : v.a) : (TI)0;
            x[2 * r + 1] = ok ? (rev ? v.a : v.b) : (TI)0;
            o += step;
        }
        return;
    }
    const int c0 = max(col0, 0), c1 = max(col1, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool ok = r > 0 || first;
        const int q = ok ? o : 0;
        const TI v0 = src[q + c0], v1 = src[q + c1];
        x[2 * r] = ok && col0 >= 0 ? v0 : (TI)0;
        x[2 * r + 1] = ok && col1 >= 0 ? v1 : (TI)0;
        o += step;
    }
}

// The thread index in a loop over stages, opaque to the compiler: per-thread index
// values of every stage would otherwise be held in registers across the loop (FP64,
// all radices: 248 instead of 144 VGPRs).
template <int NT>
__device__ __forceinline__ int stage_tid(int tid)
{
    asm volatile("" : "+v"(tid));
    return tid & (NT - 1);
}

// Full length-N complex FFT of 2^lgs sequences held in LDS (in place), in the
// direction INV (false: exp(-2 pi i t/N), true: the conjugate).
// KD: the radices that are compiled in (LenKind; a kernel for fewer of them holds
// fewer registers).
// CT = false keeps the generic stages only (kernels whose full tiles of the powers of
// two are register tiles).  tid: see fft_ct.
template <typename T, int MAXE, int NT, int KD, bool CT, bool INV>
__device__ __forceinline__ void fft_tile_dir(T *buf, int rs, int lgs, const FftDesc &fd, const cx<T> *tw, int tid)
{
    if constexpr (KD == kPow2 && CT && NT == 256) {
        // (N, tile width) pairs of the default tile budget: N * W / 2 = MAXE * NT
        if constexpr (MAXE == 8) {
            if (fd.N == 512 && rs == 9) return fft_ct<T, NT, 512, 9, 2, INV>(buf, tw, tid);
            if (fd.N == 256 && rs == 17) return fft_ct<T, NT, 256, 17, 3, INV>(buf, tw, tid);
            if (fd.N == 1024 && rs == 5) return fft_ct<T, NT, 1024, 5, 1, INV>(buf, tw, tid);
        }
    }
    if constexpr (KD == kPow2) {
        for (int st = 0; st < fd.nst; ++st) {
            const int R = fd.rad[st];
            const int t = MAXE > 8 ? stage_tid<NT>(tid) : tid; // (FP32 contractions of 16 elements a thread: 134 -> 91 VGPRs)
            if (R == 8)
                stage_bfly<T, 8, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t);
            else if (R == 4)
                stage_bfly<T, 4, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t);
            else
                stage_bfly<T, 2, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t);
        }
        return;
    }
    for (int st = 0; st < fd.nst; ++st) {
        const int t = stage_tid<NT>(tid);
        switch (fd.rad[st]) {
        case 2: stage_bfly<T, 2, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t); break;
        case 3: stage_bfly<T, 3, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t); break;
        case 4: stage_bfly<T, 4, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t); break;
        case 5: stage_bfly<T, 5, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t); break;
        case 8: stage_bfly<T, 8, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t); break;
        default:
            if constexpr (KD == kAnyLen) stage_other<T, MAXE, NT, INV>(buf, rs, lgs, fd, st, tw, t);
            break;
        }
    }
}

// fft_tile_dir with the direction as an argument (a constant argument folds
// to one instantiation).  tid: see fft_ct (-1: threadIdx.x).
template <typename T, int MAXE, int NT, int KD = kAnyLen, bool CT = true>
__device__ __forceinline__ void fft_tile(T *buf, int rs, int lgs, const FftDesc &fd, const cx<T> *tw, bool inv,
                                         int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    if (inv)
        fft_tile_dir<T, MAXE, NT, KD, CT, true>(buf, rs, lgs, fd, tw, tid);
    else
        fft_tile_dir<T, MAXE, NT, KD, CT, false>(buf, rs, lgs, fd, tw, tid);
}

// After a forward zero-padded FFT: write C and S in slot layout (in place).
template <typename T, int MAXE, int NT>
__device__ __forceinline__ void post_cs(T *buf, int rs, int lgs, int M, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    constexpr int PPT = MAXE / 2 + 1;
    const int N = 2 * M;
    const int tot = (M + 1) << lgs;
    const int smask = (1 << lgs) - 1;
    T ca[PPT], cb[PPT], sa[PPT], sb[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int e = tid + i * NT;
        if (e < tot) {
            const int s = e & smask, k = e >> lgs;
            const cx<T> z1 = lds_c(buf, rs, k, s);
            const cx<T> z2 = lds_c(buf, rs, k == 0 ? 0 : N - k, s);
            ca[i] = (T)0.5 * (z1.x + z2.x);
            cb[i] = (T)0.5 * (z1.y + z2.y);
            sa[i] = (T)0.5 * (z2.y - z1.y);
            sb[i] = (T)0.5 * (z1.x - z2.x);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int e = tid + i * NT;
        if (e < tot) {
            const int s = e & smask, k = e >> lgs;
            buf[k * rs + 2 * s] = ca[i];
            buf[k * rs + 2 * s + 1] = cb[i];
            if (k >= 1 && k < M) {
                buf[(M + k) * rs + 2 * s] = sa[i];
                buf[(M + k) * rs + 2 * s + 1] = sb[i];
            }
        }
    }
    __syncthreads();
}

// Before an inverse FFT: slots (C, S) -> hermitian-packed complex sequences.
template <typename T, int MAXE, int NT>
__device__ __forceinline__ void pre_herm(T *buf, int rs, int lgs, int M, bool c_zero, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    constexpr int PPT = MAXE / 2 + 1;
    const int N = 2 * M;
    const int tot = (M + 1) << lgs;
    const int smask = (1 << lgs) - 1;
    cx<T> z1[PPT], z2[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int e = tid + i * NT;
        if (e < tot) {
            const int s = e & smask, k = e >> lgs;
            T ca = 0, cb = 0, sa = 0, sb = 0;
            if (!c_zero) {
                ca = buf[k * rs + 2 * s];
                cb = buf[k * rs + 2 * s + 1];
            }
            if (k >= 1 && k < M) {
                sa = buf[(M + k) * rs + 2 * s];
                sb = buf[(M + k) * rs + 2 * s + 1];
            }
            z1[i] = {ca + sb, cb - sa};
            z2[i] = {ca - sb, cb + sa};
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int e = tid + i * NT;
        if (e < tot) {
            const int s = e & smask, k = e >> lgs;
            lds_cs(buf, rs, k, s, z1[i]);
            if (k >= 1 && k < M) lds_cs(buf, rs, N - k, s, z2[i]);
        }
    }
    __syncthreads();
}

// Even extension: rows 1..M-1 copied to rows N-1..M+1.
template <typename T, int NT>
__device__ __forceinline__ void pre_even(T *buf, int rs, int lgW, int M, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    const int N = 2 * M;
    const int tot = (M - 1) << lgW;
    for (int e = tid; e < tot; e += NT) {
        const int c = e & ((1 << lgW) - 1), j = 1 + (e >> lgW);
        buf[(N - j) * rs + c] = buf[j * rs + c];
    }
    __syncthreads();
}

template <typename T, int NT>
__device__ __forceinline__ void zero_rows(T *buf, int rs, int lgW, int r0, int r1, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    const int tot = (r1 - r0) << lgW;
    const int cm = (1 << lgW) - 1;
    for (int e = tid; e < tot; e += NT) buf[(r0 + (e >> lgW)) * rs + (e & cm)] = (T)0;
}

template <typename T, int NT>
__device__ __forceinline__ void load_twiddles(cx<T> *dst, const cx<double> *src, int N)
{
    for (int t = threadIdx.x; t < N; t += NT) {
        cx<double> w = src[t];
        dst[t] = {(T)w.x, (T)w.y};
    }
}

// f(c, r) over the columns c < ncols and rows r < nrows of rows-contiguous data in a tile
// of 2^lgW columns: a wave takes 64 consecutive rows of a column, several waves the same
// column where the tile has fewer columns than the block waves (one wave per column
// left 14 of 16 idle: 3001x65 solve 479 -> 422 us, 3001^2 1291 -> 1163,
// 513x513x65 mixed 1381 -> 1296).
template <int NT, typename F>
__host__ __device__ __forceinline__ void by_columns(int lgW, int ncols, int nrows, int tid, F f)
{
    constexpr int lgNW = NT == 1024 ? 4 : 2;
    static_assert(NT == 64 << lgNW, "blocks of 4 or 16 waves");
    const int lane = tid & 63, wave = tid >> 6, lgc = lgW < lgNW ? lgW : lgNW;
    for (int c = wave & ((1 << lgc) - 1); c < ncols; c += 1 << lgc)
        for (int r = (wave >> lgc) * 64 + lane; r < nrows; r += 64 << (lgNW - lgc)) f(c, r);
}

// Global -> LDS: rows [0, nrows) x cols [0, W = 2^lgW) of the tile land at
// LDS rows row0.. ; columns >= ncols are zero.  Element (r, c) is
// src[r*rsd + c*csd].  Rows-contiguous sources are read one column per wave.
template <typename T, typename TI, int NT>
__device__ __forceinline__ void tile_load(T *buf, int rs, int row0, const TI *src, int nrows, int ncols,
                                          int64_t rsd, int64_t csd, int lgW, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    const int W = 1 << lgW;
    if (rsd == 1 && csd != 1) {
        by_columns<NT>(lgW, W, nrows, tid,
                       [&](int c, int r) { buf[(row0 + r) * rs + c] = c < ncols ? (T)src[c * csd + r] : (T)0; });
    } else {
        const int cm = W - 1;
        const int tot = nrows << lgW;
        for (int e = tid; e < tot; e += NT) {
            const int c = e & cm, r = e >> lgW;
            T v = (T)0;
            if (c < ncols) v = (T)src[toff(r, rsd, c, csd)];
            buf[(row0 + r) * rs + c] = v;
        }
    }
}

// Global -> LDS for a tile of two column sets: tile column j < W/2 holds
// source column cA + j (if j < nA), tile column W/2 + j holds source column
// cB - j (if j < nB); every other column is zero.  Element (r, col) is
// src[r*rsd + col*csd].  Rows-contiguous sources are read by whole waves per
// column (several waves per column when the tile has fewer columns than the
// block has waves).
template <typename T, typename TI, int NT>
__device__ void tile_load_pair(T *buf, int rs, int row0, const TI *src, int nrows, int64_t rsd, int64_t csd,
                               int lgW, int cA, int nA, int cB, int nB, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    const int W = 1 << lgW, Wh = W >> 1;
    auto src_col = [&](int c) -> int {
        const int j = c < Wh ? c : c - Wh;
        return c < Wh ? (j < nA ? cA + j : -1) : (j < nB ? cB - j : -1);
    };
    if (rsd == 1 && csd != 1) {
        constexpr int NW = NT / 64;
        const int lane = tid & 63, wave = tid >> 6;
        const int cstep = NW < W ? NW : W;
        const int rstep = (NW / cstep) * 64;
        const int rbeg = (wave / cstep) * 64 + lane;
        for (int c = wave % cstep; c < W; c += cstep) {
            const int sc = src_col(c);
            T *dst = buf + row0 * rs + c;
            if (sc >= 0) {
                const TI *col = src + sc * csd;
                for (int r = rbeg; r < nrows; r += rstep) dst[r * rs] = (T)col[r];
            } else {
                for (int r = rbeg; r < nrows; r += rstep) dst[r * rs] = (T)0;
            }
        }
        return;
    }
    const int cm = W - 1;
    const int tot = nrows << lgW;
    for (int e = tid; e < tot; e += NT) {
        const int c = e & cm, r = e >> lgW;
        const int sc = src_col(c);
        T v = (T)0;
        if (sc >= 0) v = (T)src[toff(r, rsd, sc, csd)];
        buf[(row0 + r) * rs + c] = v;
    }
}

// The element mapping of tile_load_pair for a compile-time width WC, split
// in two halves so that a loop over tiles can fetch the next tile into
// registers (fetch_pair) while it transforms the current one, and write them
// to LDS afterwards (put_pair).  Each thread holds EPT elements; covers()
// tells whether that is enough for nrows rows.
template <int NT, int WC, int EPT>
struct PairMap {
    static constexpr int NW = NT / 64;
    static constexpr int CSTEP = NW < WC ? NW : WC;  // rows-contiguous: columns per sweep of the waves
    static constexpr int CPT = WC / CSTEP;           // columns per thread
    static constexpr int RB = EPT / CPT;             // rows per column per thread
    static constexpr int RSTEP = (NW / CSTEP) * 64;
    __host__ __device__ static bool covers(int nrows, bool rows_contiguous)
    {
        return rows_contiguous ? RB * RSTEP >= nrows : EPT * NT >= nrows * WC;
    }
};

template <int WC>
__device__ __forceinline__ int pair_src_col(int c, int cA, int nA, int cB, int nB)
{
    constexpr int Wh = WC / 2;
    const int j = c < Wh ? c : c - Wh;
    return c < Wh ? (j < nA ? cA + j : -1) : (j < nB ? cB - j : -1);
}

// MIR = false: plain tile, tile column c holds source column cA + c (c < nA).
template <typename TI, int NT, int WC, int EPT, bool MIR = true>
__device__ __forceinline__ void fetch_pair(TI (&v)[EPT], const TI *src, int nrows, int64_t rsd, int64_t csd,
                                           int cA, int nA, int cB, int nB, int tid)
{
    auto src_col = [&](int c) {
        if constexpr (MIR)
            return pair_src_col<WC>(c, cA, nA, cB, nB);
        else
            return c < nA ? cA + c : -1;
    };
    using PM = PairMap<NT, WC, EPT>;
    if (rsd == 1 && csd != 1) {
        const int lane = tid & 63, wave = tid >> 6;
        const int rbeg = (wave / PM::CSTEP) * 64 + lane;
#pragma unroll
        for (int kc = 0; kc < PM::CPT; ++kc) {
            const int sc = src_col(wave % PM::CSTEP + kc * PM::CSTEP);
            const TI *col = src + (int64_t)(sc < 0 ? 0 : sc) * csd;
#pragma unroll
            for (int kr = 0; kr < PM::RB; ++kr) {
                const int r = rbeg + kr * PM::RSTEP;
                v[kc * PM::RB + kr] = (sc >= 0 && r < nrows) ? col[r] : (TI)0;
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int e = tid + k * NT;
        const int c = e & (WC - 1), r = e / WC;
        const int sc = src_col(c);
        v[k] = (sc >= 0 && r < nrows) ? src[toff(r, rsd, sc, csd)] : (TI)0;
    }
}

template <typename T, typename TI, int NT, int WC, int EPT>
__device__ __forceinline__ void put_pair(T *buf, int rs, int row0, const TI (&v)[EPT], int nrows, bool rows_contiguous,
                                         int tid)
{
    using PM = PairMap<NT, WC, EPT>;
    if (rows_contiguous) {
        const int lane = tid & 63, wave = tid >> 6;
        const int rbeg = (wave / PM::CSTEP) * 64 + lane;
#pragma unroll
        for (int kc = 0; kc < PM::CPT; ++kc) {
            const int c = wave % PM::CSTEP + kc * PM::CSTEP;
#pragma unroll
            for (int kr = 0; kr < PM::RB; ++kr) {
                const int r = rbeg + kr * PM::RSTEP;
                if (r < nrows) buf[(row0 + r) * rs + c] = (T)v[kc * PM::RB + kr];
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int e = tid + k * NT;
        const int c = e & (WC - 1), r = e / WC;
        if (r < nrows) buf[(row0 + r) * rs + c] = (T)v[k];
    }
}

// q[0] + q[s] + ... + q[(n-1) s] with four independent partial sums, so that
// four loads are in flight at a time: ((a0 + a1) + (a2 + a3)).
template <typename T, typename TI>
__device__ __forceinline__ T sum_strided(const TI *q, int n, int64_t s)
{
    T a0 = (T)0, a1 = (T)0, a2 = (T)0, a3 = (T)0;
    int k = 0;
    for (; k + 4 <= n; k += 4) {
        a0 += (T)q[k * s];
        a1 += (T)q[(k + 1) * s];
        a2 += (T)q[(k + 2) * s];
        a3 += (T)q[(k + 3) * s];
    }
    for (; k < n; ++k) a0 += (T)q[k * s];
    return (a0 + a1) + (a2 + a3);
}

// As tile_load (columns contiguous or generic), but every element is the sum
// of nsum copies spaced sstride apart (summing partial results on the fly).
template <typename T, typename TI, int NT>
__device__ __forceinline__ void tile_load_sum(T *buf, int rs, int row0, const TI *src, int nrows, int ncols,
                                              int64_t rsd, int64_t csd, int lgW, int nsum, int64_t sstride,
                                              int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    const int W = 1 << lgW;
    if (rsd == 1 && csd != 1) {
        by_columns<NT>(lgW, W, nrows, tid, [&](int c, int r) {
            T v = (T)0;
            if (c < ncols) v = sum_strided<T>(src + c * csd + r, nsum, sstride);
            buf[(row0 + r) * rs + c] = v;
        });
        return;
    }
    const int cm = W - 1;
    const int tot = nrows << lgW;
    for (int e = tid; e < tot; e += NT) {
        const int c = e & cm, r = e >> lgW;
        T v = (T)0;
        if (c < ncols) v = sum_strided<T>(src + toff(r, rsd, c, csd), nsum, sstride);
        buf[(row0 + r) * rs + c] = v;
    }
}

// LDS -> global: LDS rows row0..row0+nrows-1, cols [0, ncols) go to
// dst[r*rsd + c*csd] scaled by `scale`.
template <typename T, typename TO, int NT>
__device__ __forceinline__ void tile_store(const T *buf, int rs, int row0, TO *dst, int nrows, int ncols,
                                           int64_t rsd, int64_t csd, T scale, int lgW, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    if (rsd == 1 && csd != 1) {
        by_columns<NT>(lgW, ncols, nrows, tid,
                       [&](int c, int r) { dst[c * csd + r] = (TO)(scale * buf[(row0 + r) * rs + c]); });
    } else {
        const int cm = (1 << lgW) - 1;
        const int tot = nrows << lgW;
        for (int e = tid; e < tot; e += NT) {
            const int c = e & cm, r = e >> lgW;
            if (c < ncols) dst[toff(r, rsd, c, csd)] = (TO)(scale * buf[(row0 + r) * rs + c]);
        }
    }
}

// As tile_store, but the scaled values are added to the destination.
template <typename T, typename TO, int NT>
__device__ __forceinline__ void tile_store_acc(const T *buf, int rs, int row0, TO *dst, int nrows, int ncols,
                                               int64_t rsd, int64_t csd, T scale, int lgW, int tid = -1)
{
    if (tid < 0) tid = threadIdx.x;
    if (rsd == 1 && csd != 1) {
        by_columns<NT>(lgW, ncols, nrows, tid,
                       [&](int c, int r) { dst[c * csd + r] += (TO)(scale * buf[(row0 + r) * rs + c]); });
    } else {
        const int cm = (1 << lgW) - 1;
        const int tot = nrows << lgW;
        for (int e = tid; e < tot; e += NT) {
            const int c = e & cm, r = e >> lgW;
            if (c < ncols) dst[toff(r, rsd, c, csd)] += (TO)(scale * buf[(row0 + r) * rs + c]);
        }
    }
}

// Blocks are dealt to the 8 XCDs round-robin; remap so that each XCD works on
// one contiguous range of logical tiles (neighbouring tiles share its L2).
__device__ __forceinline__ int xcd_remap(int bid, int nblocks)
{
    constexpr int kXcd = 8;
    if (nblocks < kXcd || nblocks % kXcd != 0) return bid;
    return (bid % kXcd) * (nblocks / kXcd) + bid / kXcd;
}

} // namespace ips
