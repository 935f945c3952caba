// Boundary convolution kernel of the infinite-domain Poisson solver (gfx950):
// boundary values as sums over slices of 2D (3D problems) or 1D (2D problems)
// discrete convolutions, accumulated in Fourier space with the kernel spectra
// (Section 4, eqs. Trap2D, Trap2Dconvolution, convolution).
// Instantiated per transform and input type: conv.hip (FP64), conv_f32.hip and
// conv_mixed.hip (FP32 transforms).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ips {

// Batch entry of the logical block group q: for each wavenumber k_b of the other
// axis its cosine slot and its sine slot are neighbours (q = 0 -> slot 0;
// q = 2kb-1 -> slot kb; q = 2kb -> slot Mo+kb, kb < Mo; q = 2Mo-1 -> slot Mo).
__device__ __forceinline__ int cc_batch(int q, int Mo)
{
    if (Mo == 0) return q;
    if (q == 0) return 0;
    if (q == 2 * Mo - 1) return Mo;
    return (q & 1) ? (q + 1) / 2 : Mo + q / 2;
}

// ---------------------------------------------------------------------------
// Boundary convolution, contraction over the tile columns (3D and 2D)
// ---------------------------------------------------------------------------
// Columns c and ncols-1-c lie at mirrored distances from the two faces: the
// kernel spectrum that weights column c for face 0 weights column ncols-1-c
// for face M, and the other way round.  A tile therefore holds W/2 columns
// c0.. of the first half and their mirrors ncols-1-c0.. (the middle column of
// an odd count only once), so each kernel-spectrum value loaded serves two
// columns, and with the C and S rows of the pencil transform four products
// per face.
template <typename T, typename TI, int MAXE, bool WB, int KD, int RPT, int NTT, int WHC>
__global__ __launch_bounds__(NTT) void k_cc(CcArgs a, int nchunk)
{
    constexpr bool BIG = NTT != NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const FftDesc &fd = a.fd;
    // the prefetching variants run one tile width only (their launcher checks it)
    const int N = fd.N, M = fd.M, W = WHC > 0 ? 2 * WHC : a.W, rs = BIG ? W : W + 1;
    const int lgW = 31 - __clz(W), lgs = lgW - 1, Wh = W >> 1;
    const cx<T> *tw = tw_table<T, BIG>(smem, a.tw, a.twf);
    T *buf = reinterpret_cast<T *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<T>)));
    // Logical order: for each wavenumber k_b of the other axis, its cos slot
    // and its sin slot are neighbours, so the blocks reading the same kernel
    // spectra K[.][k_b][.] run together on one XCD (shared L2).
    const int lb = xcd_remap(blockIdx.x, nchunk * a.nbatch);
    const int ch = lb % nchunk, bt = cc_batch(lb / nchunk, a.Mo);
    const int kb = a.Mo > 0 ? (bt <= a.Mo ? bt : bt - a.Mo) : 0;
    const TI *in = static_cast<const TI *>(a.in) + bt * a.ibs;
    T *Bout = static_cast<T *>(a.Bout);
    // Slot rows per thread: t = threadIdx.x + i NTT < M, i < TPT, owns rows t
    // and M + t, i.e. C_t and S_t (which share the kernel spectrum value) for
    // t >= 1, and C_0 and C_M for t = 0.
    constexpr int TPT = RPT / 2;
    double a10[TPT], a11[TPT], a20[TPT], a21[TPT]; // [row 1|2][face 0|M]
#pragma unroll
    for (int i = 0; i < TPT; ++i) a10[i] = a11[i] = a20[i] = a21[i] = 0.0;
    if (!BIG) load_twiddles<T, NTT>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    const int hc = (a.ncols + 1) >> 1; // first-half columns (the chunked range)
    // tiles of this chunk: a contiguous run of columns, or (interleaved) every
    // nchunk-th tile, so that the blocks of one batch entry, which run side by
    // side, read neighbouring columns at the same time (strided pencils share
    // their cache lines across those blocks instead of re-fetching them)
    const int cbeg = a.interleave ? ch * Wh : ch * a.cols_per_chunk;
    const int cend = a.interleave ? hc : min(hc, cbeg + a.cols_per_chunk);
    const int cstep = a.interleave ? nchunk * Wh : Wh;
    // PF (compile-time width): the next tile is fetched into registers while
    // the current one is transformed and contracted
    constexpr bool PF = WHC > 0;
    constexpr int WCF = PF ? 2 * WHC : 2;
    const bool rcont = a.irs == 1 && a.ics != 1;
    auto n_a = [&](int c) { return min(Wh, cend - c); };
    auto n_b = [&](int c) { return min(n_a(c), max(0, (a.ncols - 2 * c) >> 1)); };
    TI pf[MAXE];
    if constexpr (PF)
        if (cbeg < cend)
            fetch_pair<TI, NTT, WCF, MAXE>(pf, in, a.nrows_in, a.irs, a.ics, cbeg, n_a(cbeg), a.ncols - 1 - cbeg,
                                          n_b(cbeg), threadIdx.x);
    for (int c0 = cbeg; c0 < cend; c0 += cstep) {
        const int nA = n_a(c0);
        const int m0 = a.ncols - 1 - c0; // mirror of c0
        const int nB = n_b(c0);          // mirrors distinct from their column
        // the thread index, opaque to the compiler: per-thread index and
        // twiddle values are recomputed for each tile rather than held in
        // registers across the loop
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        tid &= NTT - 1; // the range (known bits) of the thread index
        zero_rows<T, NTT>(buf, rs, lgW, 0, 1, tid);
        zero_rows<T, NTT>(buf, rs, lgW, 1 + a.nrows_in, N, tid);
        if constexpr (PF) {
            put_pair<T, TI, NTT, WCF, MAXE>(buf, rs, 1, pf, a.nrows_in, rcont, tid);
            const int c1 = c0 + cstep;
            if (c1 < cend)
                fetch_pair<TI, NTT, WCF, MAXE>(pf, in, a.nrows_in, a.irs, a.ics, c1, n_a(c1), a.ncols - 1 - c1,
                                              n_b(c1), tid);
        } else {
            tile_load_pair<T, TI, NTT>(buf, rs, 1, in, a.nrows_in, a.irs, a.ics, lgW, c0, nA, m0, nB, tid);
        }
        __syncthreads();
        fft_tile<T, MAXE, NTT, KD, false>(buf, rs, lgs, fd, tw, false, tid);
        post_cs<T, MAXE, NTT>(buf, rs, lgs, M, tid);
        if (WB && (a.Mo == 0 || bt > a.Mo)) {
            const int64_t bb = a.Mo == 0 ? 0 : (int64_t)(bt - a.Mo - 1) * a.Bbs;
            const int lane = tid & 63, wave = tid >> 6;
            for (int c = wave; c < W; c += NTT / 64) {
                const int j = c < Wh ? c : c - Wh;
                const int col = c < Wh ? (j < nA ? c0 + j : -1) : (j < nB ? m0 - j : -1);
                if (col < 0) continue;
                const int64_t cb = (int64_t)col * a.Bcs + bb;
                for (int r = lane; r < M - 1; r += 64) {
                    const T v = buf[(M + 1 + r) * rs + c];
                    if (a.Bf32)
                        static_cast<float *>(a.Bout)[cb + (int64_t)r * a.Brs] = (float)v;
                    else
                        Bout[cb + (int64_t)r * a.Brs] = v;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            const int t = tid + i * NTT;
            if (t < M) {
                const bool two = t > 0; // row M + t is S_t (else C_M, see below)
                const T *r1 = buf + t * rs, *r2 = buf + (M + t) * rs;
                // FP64 kernel spectra and FP64 sums in every mode: an FP32 slot
                // value is widened exactly, so the boundary sums accumulate in FP64
                const double *Kr = static_cast<const double *>(a.K) + (int64_t)kb * a.Ko;
                const double *KA = Kr + t + (int64_t)c0 * a.Kd; // K at column c0 + j
                const double *KB = Kr + t + (int64_t)m0 * a.Kd; // K at column m0 - j
                using TA = double;
                TA s10 = a10[i], s11 = a11[i], s20 = a20[i], s21 = a21[i];
                auto col_pair = [&](int j) {
                    const TA kA = KA[(int64_t)j * a.Kd], kB = KB[-(int64_t)j * a.Kd];
                    const TA ud = (TA)r1[j], um = (TA)r1[Wh + j];
                    const TA vd = two ? (TA)r2[j] : (TA)0, vm = two ? (TA)r2[Wh + j] : (TA)0;
                    s10 = fma(kA, ud, s10);
                    s10 = fma(kB, um, s10);
                    s11 = fma(kB, ud, s11);
                    s11 = fma(kA, um, s11);
                    s20 = fma(kA, vd, s20);
                    s20 = fma(kB, vm, s20);
                    s21 = fma(kB, vd, s21);
                    s21 = fma(kA, vm, s21);
                };
                if (WHC > 0 && nA == WHC) {
#pragma unroll
                    for (int j = 0; j < WHC; ++j) col_pair(j);
                } else {
                    for (int j = 0; j < nA; ++j) col_pair(j);
                }
                if (!two) {
                    // C_M (no sine partner) with its own kernel spectrum
                    const double *MA = Kr + M + (int64_t)c0 * a.Kd, *MB = Kr + M + (int64_t)m0 * a.Kd;
                    for (int j = 0; j < nA; ++j) {
                        const TA kA = MA[(int64_t)j * a.Kd], kB = MB[-(int64_t)j * a.Kd];
                        const TA vd = (TA)r2[j], vm = (TA)r2[Wh + j];
                        s20 = fma(kA, vd, s20);
                        s20 = fma(kB, vm, s20);
                        s21 = fma(kB, vd, s21);
                        s21 = fma(kA, vm, s21);
                    }
                }
                a10[i] = s10;
                a11[i] = s11;
                a20[i] = s20;
                a21[i] = s21;
            }
        }
        __syncthreads();
    }
    // FP64 partials [face][chunk][batch][slot]: slot rows t and M + t
    const int64_t o0 = ((int64_t)ch * a.nbatch + bt) * N, o1 = o0 + (int64_t)nchunk * a.nbatch * N;
    double *pp = static_cast<double *>(a.part);
#pragma unroll
    for (int i = 0; i < TPT; ++i) {
        const int t = threadIdx.x + i * NTT;
        if (t < M) {
            pp[o0 + t] = a10[i];
            pp[o1 + t] = a11[i];
            pp[o0 + M + t] = a20[i];
            pp[o1 + M + t] = a21[i];
        }
    }
}

// The contraction in register tiles (see RegTile): inputs straight from global
// memory (the next tile's during the transform) into the first stage; the cosine
// and sine parts are formed in registers after the last stage and written to the
// LDS once, sequence by sequence, for the sums over the columns (same thread per
// slot row and same order of the sums as k_cc; PAIRS: tiles of twice the width whose
// halves belong to neighbouring chunks, each with its own sums). Bound by LDS (45% of
// its cycles, half of it conflicts) and the latency of B and K. 257^3: FP64 219/209/214
// -> 200/180/183 us, FP32 112/124/115 -> 112/115/111 us; 513^3 FP32 1010/1288/1251 ->
// 726/968/950 (single chunks 709/1237/1258).
template <typename T, typename TI, typename R, bool WB, bool PAIRS>
__global__ __launch_bounds__(R::NTH) void k_cc_rt(CcArgs a, int nchunk)
{
    constexpr int N = R::N, M = N / 2, W = R::W, Wh = W / 2, P = R::P, NTH = R::NTH;
    extern __shared__ __align__(16) unsigned char smem[];
    const cx<T> *tw = tw_table<T, !R::LTW>(smem, a.tw, a.twf);
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem) + (R::LTW ? N : 0);
    // PAIRS: chunks NG ch .. of Wg first-half columns each per tile
    constexpr int NG = PAIRS ? 2 : 1, Wg = Wh / NG;
    const int nblk = (nchunk + NG - 1) / NG;
    const int lb = xcd_remap(blockIdx.x, nblk * a.nbatch);
    const int ch = lb % nblk * NG, bt = cc_batch(lb / nblk, a.Mo);
    const int kb = a.Mo > 0 ? (bt <= a.Mo ? bt : bt - a.Mo) : 0;
    const TI *in = static_cast<const TI *>(a.in) + bt * a.ibs;
    constexpr int TPT = M / NTH > 0 ? M / NTH : 1;
    double a10[TPT][NG], a11[TPT][NG], a20[TPT][NG], a21[TPT][NG]; // [row 1|2][face 0|M]
#pragma unroll
    for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g) a10[i][g] = a11[i][g] = a20[i][g] = a21[i][g] = 0.0;
    if constexpr (R::LTW) load_twiddles<T, NTH>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    const int hc = (a.ncols + 1) >> 1; // first-half columns (the chunked range)
    const int cbeg = a.interleave ? ch * Wg : ch * a.cols_per_chunk;
    const int cend = a.interleave ? hc : min(hc, cbeg + a.cols_per_chunk);
    const int cstep = a.interleave ? nchunk * Wg : Wh;
    const int wmax = PAIRS && ch + NG > nchunk ? Wg : Wh; // the last of an odd number of chunks
    auto n_a = [&](int c) { return min(wmax, cend - c); };
    auto n_b = [&](int c) { return min(n_a(c), max(0, (a.ncols - 2 * c) >> 1)); };
    // source column of tile column c of the tile at c0 (-1: none)
    auto src_col = [&](int c, int c0, int nA, int nB) {
        const int jj = c < Wh ? c : c - Wh;
        return c < Wh ? (jj < nA ? c0 + jj : -1) : (jj < nB ? a.ncols - 1 - c0 - jj : -1);
    };
    auto fetch = [&](TI(&x)[8], int c0, int tid) {
        int j, s;
        rt_plain<R>(tid, j, s);
        const int nA = n_a(c0), nB = n_b(c0);
        const int q0 = src_col(2 * s, c0, nA, nB), q1 = src_col(2 * s + 1, c0, nA, nB), ics = (int)a.ics;
        // (full tiles of contiguous columns: ascending, or descending among the mirrors)
        const int dir = nA == Wh && nB == Wh && ics == 1 && Wh > 1 ? (2 * s < Wh ? 1 : -1) : 0;
        rt_fetch<TI, R>(x, in, a.irs, q0 < 0 ? -1 : __mul24(q0, ics), q1 < 0 ? -1 : __mul24(q1, ics), dir, j, 1);
    };
    TI x[8];
    if (cbeg < cend) fetch(x, cbeg, threadIdx.x);
    __syncthreads(); // the twiddles
    for (int c0 = cbeg; c0 < cend; c0 += cstep) {
        const int nA = n_a(c0), nB = n_b(c0);
        const int m0 = a.ncols - 1 - c0; // mirror of c0
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid)); // (as in k_cc)
        tid &= NTH - 1;
        int j, s;
        rt_plain<R>(tid, j, s);
        cx<T> v[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = cx<T>{(T)x[2 * r], (T)x[2 * r + 1]};
        if (c0 + cstep < cend) fetch(x, c0 + cstep, tid);
        rt_first_zpad<T, R>(buf, v, j, s);
        rt_middle<T, R, false>(buf, tw, tid);
        rt_paired<R>(tid, j, s);
        rt_last<T, R, false>(buf, tw, v, j, s);
        cx<T> C[4], S[4];
        rt_slots<T, R>(v, j, C, S);
        __syncthreads();
        // slot rows k and M + k of sequence s (row M of k = 0: the last cosine row)
        {
            cx<T> *p = buf + s * R::SP + j;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rt_put(p + r * P, C[r]);
                rt_put(p + M + r * P, S[r]);
            }
        }
        __syncthreads();
        if (WB && (a.Mo == 0 || bt > a.Mo)) {
            const int64_t bb = a.Mo == 0 ? 0 : (int64_t)(bt - a.Mo - 1) * a.Bbs;
            const int lane = tid & 63, wave = tid >> 6;
            for (int c = wave; c < W; c += NTH / 64) {
                const int col = src_col(c, c0, nA, nB);
                if (col < 0) continue;
                const int64_t cb = (int64_t)col * a.Bcs + bb;
                const T *q = reinterpret_cast<const T *>(buf + (c >> 1) * R::SP + M + 1) + (c & 1);
                for (int r = lane; r < M - 1; r += 64) {
                    if (a.Bf32)
                        static_cast<float *>(a.Bout)[cb + (int64_t)r * a.Brs] = (float)q[2 * r];
                    else
                        static_cast<T *>(a.Bout)[cb + (int64_t)r * a.Brs] = q[2 * r];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < TPT; ++i)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int t = tid + i * NTH;
                if (NTH > M && t >= M) continue;
                const bool two = t > 0; // row M + t is S_t (else C_M, see below)
                const T *r1 = reinterpret_cast<const T *>(buf + t), *r2 = r1 + 2 * M;
                auto at = [&](const T *r, int c) { return (double)r[(c >> 1) * 2 * R::SP + (c & 1)]; };
                const double *Kr = a.K + (int64_t)kb * a.Ko;
                const double *KA = Kr + t + (int64_t)c0 * a.Kd; // K at column c0 + jj
                const double *KB = Kr + t + (int64_t)m0 * a.Kd; // K at column m0 - jj
                double s10 = a10[i][g], s11 = a11[i][g], s20 = a20[i][g], s21 = a21[i][g];
                auto col_pair = [&](int jj) {
                    const double kA = KA[(int64_t)jj * a.Kd], kB = KB[-(int64_t)jj * a.Kd];
                    const double ud = at(r1, jj), um = at(r1, Wh + jj);
                    const double vd = two ? at(r2, jj) : 0.0, vm = two ? at(r2, Wh + jj) : 0.0;
                    s10 = fma(kA, ud, s10);
                    s10 = fma(kB, um, s10);
                    s11 = fma(kB, ud, s11);
                    s11 = fma(kA, um, s11);
                    s20 = fma(kA, vd, s20);
                    s20 = fma(kB, vm, s20);
                    s21 = fma(kB, vd, s21);
                    s21 = fma(kA, vm, s21);
                };
                const int j0 = g * Wg, j1 = min(j0 + Wg, nA);
                if (j1 == j0 + Wg) {
#pragma unroll
                    for (int jj = 0; jj < Wg; ++jj) col_pair(j0 + jj);
                } else {
                    for (int jj = j0; jj < j1; ++jj) col_pair(jj);
                }
                if (!two) {
                    // C_M (no sine partner) with its own kernel spectrum
                    const double *MA = Kr + M + (int64_t)c0 * a.Kd, *MB = Kr + M + (int64_t)m0 * a.Kd;
                    for (int jj = j0; jj < j1; ++jj) {
                        const double kA = MA[(int64_t)jj * a.Kd], kB = MB[-(int64_t)jj * a.Kd];
                        const double vd = at(r2, jj), vm = at(r2, Wh + jj);
                        s20 = fma(kA, vd, s20);
                        s20 = fma(kB, vm, s20);
                        s21 = fma(kB, vd, s21);
                        s21 = fma(kA, vm, s21);
                    }
                }
                a10[i][g] = s10;
                a11[i][g] = s11;
                a20[i][g] = s20;
                a21[i][g] = s21;
            }
        __syncthreads();
    }
    // FP64 partials [face][chunk][batch][slot]: slot rows t and M + t
#pragma unroll
    for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int t = threadIdx.x + i * NTH;
            if ((NTH > M && t >= M) || ch + g >= nchunk) continue;
            const int64_t o0 = ((int64_t)(ch + g) * a.nbatch + bt) * N, o1 = o0 + (int64_t)nchunk * a.nbatch * N;
            a.part[o0 + t] = a10[i][g];
            a.part[o1 + t] = a11[i][g];
            a.part[o0 + M + t] = a20[i][g];
            a.part[o1 + M + t] = a21[i][g];
        }
}

template <typename T, typename TI, bool WB, typename R, bool PAIRS>
static void launch_cc_rt(const CcArgs &a, int nchunk, hipStream_t st)
{
    const size_t lds = rt_lds<T, R>();
    const int nblk = PAIRS ? (nchunk + 1) / 2 : nchunk;
    set_lds((const void *)&k_cc_rt<T, TI, R, WB, PAIRS>, lds);
    hipLaunchKernelGGL((k_cc_rt<T, TI, R, WB, PAIRS>), dim3(nblk * a.nbatch), dim3(R::NTH), lds, st, a, nchunk);
}

template <typename T, typename TI, int MAXE, bool WB, int KD, int RPT, int NTT = NT, int WHC = 0>
static void launch_cc_k(const CcArgs &a, int nchunk, hipStream_t st)
{
    const size_t lds = tile_lds<T>(a.fd.N, a.W);
    set_lds((const void *)&k_cc<T, TI, MAXE, WB, KD, RPT, NTT, WHC>, lds);
    hipLaunchKernelGGL((k_cc<T, TI, MAXE, WB, KD, RPT, NTT, WHC>), dim3(nchunk * a.nbatch), dim3(NTT), lds,
                       st, a, nchunk);
}

// Compile-time widths (W = 16, 8 for 2M = 256, 512; W = 4 for lengths in
// (512, 1024]) get a fully unrolled contraction and the register prefetch of
// the next tile (shorter lengths other than powers of two measured faster
// without, in batches of small uneven boxes).
template <int WHC, int MAXE, int NTT = NT>
static bool prefetch_fits(const CcArgs &a)
{
    return a.W == 2 * WHC && PairMap<NTT, 2 * WHC, MAXE>::covers(a.nrows_in, a.irs == 1 && a.ics != 1);
}

template <typename T, typename TI, int MAXE, bool WB>
static void launch_cc_m(const CcArgs &a, int nchunk, hipStream_t st)
{
    auto go = [&](auto kd) {
        constexpr int KD = decltype(kd)::value;
        constexpr bool P2 = KD == kPow2;
        if (a.fd.N <= 2 * NT) {
            if constexpr (P2) {
                if (prefetch_fits<8, MAXE>(a)) return launch_cc_k<T, TI, MAXE, WB, KD, 2, NT, 8>(a, nchunk, st);
                if (prefetch_fits<4, MAXE>(a)) return launch_cc_k<T, TI, MAXE, WB, KD, 2, NT, 4>(a, nchunk, st);
            }
            launch_cc_k<T, TI, MAXE, WB, KD, 2>(a, nchunk, st);
            return;
        }
        // (W = 4 at 2M = 1024 and every tile at 2048 are register tiles up to 8 NT elements)
        constexpr bool RT = P2 && MAXE == 8;
        if (a.fd.N <= 4 * NT) {
            if constexpr (!RT)
                if (prefetch_fits<2, MAXE>(a)) return launch_cc_k<T, TI, MAXE, WB, KD, 4, NT, 2>(a, nchunk, st);
            launch_cc_k<T, TI, MAXE, WB, KD, 4>(a, nchunk, st);
        } else if constexpr (!RT) {
            launch_cc_k<T, TI, MAXE, WB, KD, 8>(a, nchunk, st);
        }
    };
    if constexpr (MAXE == 8)
        by_kind(a.fd.N, go);
    else
        by_pow2(a.fd.N, go);
}

template <typename T, typename TI, bool WB>
hipError_t launch_cc_t(const CcArgs &a, int nchunk, hipStream_t st)
{
    const int work = (a.W / 2) * a.fd.N;
    const bool rt = a.nrows_in == a.fd.M - 1;
    if (a.pairs) {
        if (!rt || a.fd.N != 1024 || a.W != RegTile<1024, 4>::W || !a.interleave) return hipErrorInvalidValue;
        launch_cc_rt<T, TI, WB, RegTile<1024, 4>, true>(a, nchunk, st);
        return hipGetLastError();
    }
    if (rt && rt_tile<0>(a.fd.N, a.W, [&](auto tile) { launch_cc_rt<T, TI, WB, decltype(tile), false>(a, nchunk, st); }))
        return hipGetLastError();
    if (big_fft(a.fd.N)) {
        // one complex sequence (a column and its mirror) per tile; rows per thread = N / NTB <= 8
        if (a.W != 2 || a.fd.N > 8 * NTB) return hipErrorInvalidValue;
        if (a.fd.N <= 4 * NTB)
            launch_cc_k<T, TI, 4, WB, kAnyLen, 4, NTB>(a, nchunk, st);
        else
            launch_cc_k<T, TI, 8, WB, kAnyLen, 8, NTB>(a, nchunk, st);
        return hipGetLastError();
    }
    // (no other kernel holds these rows of a power of two)
    if (is_pow2(a.fd.N) && a.fd.N > 4 * NT && work <= 8 * NT) return hipErrorInvalidValue;
    if (work <= 8 * NT)
        launch_cc_m<T, TI, 8, WB>(a, nchunk, st);
    else
        launch_cc_m<T, TI, 16, WB>(a, nchunk, st);
    return hipGetLastError();
}

} // namespace ips
