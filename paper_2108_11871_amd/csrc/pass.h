// Pencil transforms of the infinite-domain Poisson solver (gfx950): DST-I,
// zero-padded cosine/sine, even (DCT-I) and hermitian-synthesis transforms
// along one axis of a strided 2D/3D array (Sections 3, 4, 5).
// Instantiated per type: pass.hip (FP64), pass_f32.hip (FP32 input) and
// pass_mixed.hip (FP64 input, FP32 transforms).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ips {

// Tile lb -> (column block cb, batch entry bt).  Column blocks vary fastest,
// except where the output's batch stride is 1: there neighbouring batch
// entries come first, so that the blocks that run side by side (on one XCD)
// write neighbouring words of the same cache lines (a tile row writes its W
// values at the output's column stride).
__device__ __forceinline__ void tile_of(const PassArgs &a, int ncb, int lb, int &cb, int &bt)
{
    if (a.obs == 1 && a.nbatch > 1) {
        bt = lb % a.nbatch;
        cb = lb / a.nbatch;
    } else {
        cb = lb % ncb;
        bt = lb / ncb;
    }
}

// One tile of a pass: tile lb (column block lb % ncb of batch entry lb / ncb),
// loaded into LDS (rows placed as the input mode needs), transformed along its
// rows and stored.
template <typename T, typename TI, typename TO, int MAXE, int KD, int NTT>
__device__ __forceinline__ void pass_tile(const PassArgs &a, int lb)
{
    constexpr bool BIG = NTT != NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const FftDesc &fd = a.fd;
    const int N = fd.N, M = fd.M, W = a.W, rs = BIG ? W : W + 1;
    const int lgW = 31 - __clz(W), lgs = lgW - 1;
    const cx<T> *tw = tw_table<T, BIG>(smem, a.tw, a.twf);
    T *buf = reinterpret_cast<T *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<T>)));
    const int ncb = (a.ncols + W - 1) / W;
    int cb, bt;
    tile_of(a, ncb, lb, cb, bt);
    const int c0 = cb * W;
    const int nc = min(W, a.ncols - c0);
    const TI *in = static_cast<const TI *>(a.in) + bt * a.ibs + c0 * a.ics;
    TO *out = static_cast<TO *>(a.out) + bt * a.obs + c0 * a.ocs;
    if (!BIG) load_twiddles<T, NTT>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    bool inv = false;
    if (a.in_mode == IN_ZPAD) {
        zero_rows<T, NTT>(buf, rs, lgW, 0, 1);
        zero_rows<T, NTT>(buf, rs, lgW, 1 + a.nrows_in, N);
        tile_load<T, TI, NTT>(buf, rs, 1, in, a.nrows_in, nc, a.irs, a.ics, lgW);
        __syncthreads();
    } else if (a.in_mode == IN_ZPAD0) {
        zero_rows<T, NTT>(buf, rs, lgW, a.nrows_in, N);
        tile_load<T, TI, NTT>(buf, rs, 0, in, a.nrows_in, nc, a.irs, a.ics, lgW);
        __syncthreads();
    } else if (a.in_mode == IN_EVEN) {
        tile_load<T, TI, NTT>(buf, rs, 0, in, a.nrows_in, nc, a.irs, a.ics, lgW);
        __syncthreads();
        pre_even<T, NTT>(buf, rs, lgW, M);
    } else if (a.in_mode == IN_HERM) {
        if (a.nsum > 1)
            tile_load_sum<T, TI, NTT>(buf, rs, 0, in, a.nrows_in, nc, a.irs, a.ics, lgW, a.nsum,
                                      a.sstride);
        else
            tile_load<T, TI, NTT>(buf, rs, 0, in, a.nrows_in, nc, a.irs, a.ics, lgW);
        __syncthreads();
        pre_herm<T, MAXE, NTT>(buf, rs, lgs, M, false);
        inv = true;
    } else {
        tile_load<T, TI, NTT>(buf, rs, M + 1, in, a.nrows_in, nc, a.irs, a.ics, lgW);
        __syncthreads();
        pre_herm<T, MAXE, NTT>(buf, rs, lgs, M, true);
        inv = true;
    }
    fft_tile<T, MAXE, NTT, KD>(buf, rs, lgs, fd, tw, inv);
    if (a.in_mode == IN_ZPAD || a.in_mode == IN_ZPAD0) post_cs<T, MAXE, NTT>(buf, rs, lgs, M);
    if (a.accum)
        tile_store_acc<T, TO, NTT>(buf, rs, a.out_r0, out, a.out_nrows, nc, a.ors, a.ocs, (T)a.scale, lgW);
    else
        tile_store<T, TO, NTT>(buf, rs, a.out_r0, out, a.out_nrows, nc, a.ors, a.ocs, (T)a.scale, lgW);
}

// One pencil pass.  A tile is W consecutive columns of one batch entry; it is
// loaded into LDS (rows placed as the input mode needs), transformed along
// its rows and stored.  Generic widths (WC = 0): one tile per block.  With a
// compile-time width WC and EPT fetch registers per thread, the grid holds as
// many blocks as are resident on the device at once, each block walks the
// tiles with the grid size as stride and fetches the next tile into
// registers while the current one is transformed.  The thread index is made
// opaque inside that loop so that the compiler recomputes per-thread index
// values instead of holding them in registers for the whole loop.
template <typename T, typename TI, typename TO, int MAXE, int KD, int NTT, int WC, int EPT>
__global__ __launch_bounds__(NTT) void k_pass(PassArgs a, int ntiles)
{
    constexpr bool PF = WC > 0;
    if constexpr (!PF) {
        // one tile per block
        pass_tile<T, TI, TO, MAXE, KD, NTT>(a, xcd_remap(blockIdx.x, ntiles));
        return;
    }
    constexpr bool BIG = NTT != NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const FftDesc &fd = a.fd;
    const int N = fd.N, M = fd.M, W = PF ? WC : a.W, rs = BIG ? W : W + 1;
    const int lgW = 31 - __clz(W), lgs = lgW - 1;
    const cx<T> *tw = tw_table<T, BIG>(smem, a.tw, a.twf);
    T *buf = reinterpret_cast<T *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<T>)));
    const int ncb = (a.ncols + W - 1) / W;
    const int grid = gridDim.x;
    const int lb = xcd_remap(blockIdx.x, grid);
    const int mode = a.in_mode;
    // first tile row of the loaded rows
    const int row0 = mode == IN_ZPAD ? 1 : (mode == IN_SPECS ? M + 1 : 0);
    const bool rcont = a.irs == 1 && a.ics != 1;
    const TI *in0 = static_cast<const TI *>(a.in);
    TO *out0 = static_cast<TO *>(a.out);
    auto tile_at = [&](int it, int &c0, int &nc, int64_t &ioff, int64_t &ooff) {
        int cb, bt;
        tile_of(a, ncb, it, cb, bt);
        c0 = cb * W;
        nc = min(W, a.ncols - c0);
        ioff = bt * a.ibs + c0 * a.ics;
        ooff = bt * a.obs + c0 * a.ocs;
    };
    if (!BIG) load_twiddles<T, NTT>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    TI pf[PF ? EPT : 1];
    if constexpr (PF) {
        if (lb < ntiles) {
            int c0, nc;
            int64_t io, oo;
            tile_at(lb, c0, nc, io, oo);
            fetch_pair<TI, NTT, WC, EPT, false>(pf, in0 + io, a.nrows_in, a.irs, a.ics, 0, nc, 0, 0, threadIdx.x);
        }
    }
    for (int it = lb; it < ntiles; it += grid) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        tid &= NTT - 1; // the range (known bits) of the thread index
        int c0, nc;
        int64_t io, oo;
        tile_at(it, c0, nc, io, oo);
        if (mode == IN_ZPAD) {
            zero_rows<T, NTT>(buf, rs, lgW, 0, 1, tid);
            zero_rows<T, NTT>(buf, rs, lgW, 1 + a.nrows_in, N, tid);
        } else if (mode == IN_ZPAD0) {
            zero_rows<T, NTT>(buf, rs, lgW, a.nrows_in, N, tid);
        }
        if constexpr (PF) {
            put_pair<T, TI, NTT, WC, EPT>(buf, rs, row0, pf, a.nrows_in, rcont, tid);
            const int nx = it + grid;
            if (nx < ntiles) {
                int c1, n1;
                int64_t i1, o1;
                tile_at(nx, c1, n1, i1, o1);
                fetch_pair<TI, NTT, WC, EPT, false>(pf, in0 + i1, a.nrows_in, a.irs, a.ics, 0, n1, 0, 0, tid);
            }
        }
        __syncthreads();
        bool inv = false;
        if (mode == IN_EVEN) {
            pre_even<T, NTT>(buf, rs, lgW, M, tid);
        } else if (mode == IN_HERM) {
            pre_herm<T, MAXE, NTT>(buf, rs, lgs, M, false, tid);
            inv = true;
        } else if (mode == IN_SPECS) {
            pre_herm<T, MAXE, NTT>(buf, rs, lgs, M, true, tid);
            inv = true;
        }
        fft_tile<T, MAXE, NTT, KD>(buf, rs, lgs, fd, tw, inv, tid);
        if (mode == IN_ZPAD || mode == IN_ZPAD0) post_cs<T, MAXE, NTT>(buf, rs, lgs, M, tid);
        if (a.accum)
            tile_store_acc<T, TO, NTT>(buf, rs, a.out_r0, out0 + oo, a.out_nrows, nc, a.ors, a.ocs, (T)a.scale, lgW,
                                       tid);
        else
            tile_store<T, TO, NTT>(buf, rs, a.out_r0, out0 + oo, a.out_nrows, nc, a.ors, a.ocs, (T)a.scale, lgW,
                                   tid);
        __syncthreads();
    }
}

// A pass in register tiles (see RegTile): inputs straight from global memory into
// the first stage, results straight from the last one. MODE: IN_ZPAD (forward
// cosine/sine, or the sine rows alone), IN_SPECS (sine synthesis: the first stage's
// upper rows are the mirror lane's, negated) or IN_HERM. One tile per block: resident
// blocks that walk the tiles and fetch the next one's inputs ahead measured slower
// (257^3 FP64 1392 -> 1443 us), the blocks of a CU overlap by themselves. Bound by
// the latency and the partial cache lines of its strided rows: 257^3 FP64 rho_z 140 ->
// 90 us, rho_y 123 -> 85, inv_y 97 -> 62, inv_z 98 -> 60 us (4.4 TB/s), FP32 rho_z 103 ->
// 90, rho_y 94 -> 66, inv_y 50 -> 35, inv_z 53 -> 44 us; 513^3 FP32 rho_z 1127 -> 591,
// rho_y 1124 -> 504, inv_z 522 us (3.1 TB/s).
template <typename T, typename TI, typename TO, typename R, int MODE>
__global__ __launch_bounds__(R::NTH) void k_pass_rt(PassArgs a, int ntiles)
{
    constexpr int N = R::N, M = N / 2, W = R::W, P = R::P, NV = MODE == IN_HERM ? 16 : 8;
    extern __shared__ __align__(16) unsigned char smem[];
    const cx<T> *tw = tw_table<T, !R::LTW>(smem, a.tw, a.twf);
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem) + (R::LTW ? N : 0);
    const int ncb = (a.ncols + W - 1) / W;
    const int tid = threadIdx.x;
    int cb, bt, j, s;
    tile_of(a, ncb, xcd_remap(blockIdx.x, ntiles), cb, bt);
    const int c0 = cb * W, nc = min(W, a.ncols - c0);
    const TI *in = static_cast<const TI *>(a.in) + bt * a.ibs + c0 * a.ics;
    TO *out = static_cast<TO *>(a.out) + bt * a.obs + c0 * a.ocs;
    if constexpr (MODE == IN_ZPAD)
        rt_plain<R>(tid, j, s);
    else
        rt_paired<R>(tid, j, s);
    TI x[NV];
    {
        const int c = 2 * s, ics = (int)a.ics;
        const int o0 = c < nc ? c * ics : -1, o1 = c + 1 < nc ? (c + 1) * ics : -1, dir = nc == W && ics == 1;
        if constexpr (MODE == IN_HERM) {
            // cosine rows k and sine rows M + k (row M of k = 0: the last cosine row)
            TI y[8], z[8];
            rt_fetch<TI, R>(y, in, a.irs, o0, o1, dir, j, 0);
            rt_fetch<TI, R>(z, in + M * a.irs, a.irs, o0, o1, dir, j, 0);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                x[r] = y[r];
                x[8 + r] = z[r];
            }
        } else {
            rt_fetch<TI, R>(x, in, a.irs, o0, o1, dir, j, 1);
        }
    }
    if constexpr (R::LTW) load_twiddles<T, R::NTH>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    cx<T> v[8];
    if constexpr (MODE == IN_ZPAD) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = cx<T>{(T)x[2 * r], (T)x[2 * r + 1]};
    } else if constexpr (MODE == IN_SPECS) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = cx<T>{(T)x[2 * r + 1], -(T)x[2 * r]};
        rt_unfold_odd<T, R>(v, j);
    } else {
        cx<T> C[4], S[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            C[r] = cx<T>{(T)x[2 * r], (T)x[2 * r + 1]};
            S[r] = cx<T>{(T)x[8 + 2 * r], (T)x[9 + 2 * r]};
        }
        rt_unfold_herm<T, R>(C, S, j, v);
    }
    if constexpr (MODE == IN_ZPAD)
        rt_first_zpad<T, R>(buf, v, j, s);
    else
        rt_first<T, R, true>(buf, v, j, s);
    rt_middle<T, R, MODE != IN_ZPAD>(buf, tw, tid);
    if constexpr (MODE == IN_ZPAD)
        rt_paired<R>(tid, j, s);
    else
        rt_plain<R>(tid, j, s);
    rt_last<T, R, MODE != IN_ZPAD>(buf, tw, v, j, s);
    const T scale = (T)a.scale;
    const int c = 2 * s, ocs = (int)a.ocs, ors = (int)a.ors;
    auto put = [&](int row, cx<T> w) {
        const int t = row - a.out_r0;
        if (t < 0 || t >= a.out_nrows) return;
        TO *p = out + toff(t, ors, c, ocs);
        if (nc == W && ocs == 1 && !a.accum) {
            *reinterpret_cast<pair_t<TO> *>(p) = pair_t<TO>{(TO)(scale * w.x), (TO)(scale * w.y)};
        } else if (a.accum) {
            if (c < nc) p[0] += (TO)(scale * w.x);
            if (c + 1 < nc) p[ocs] += (TO)(scale * w.y);
        } else {
            if (c < nc) p[0] = (TO)(scale * w.x);
            if (c + 1 < nc) p[ocs] = (TO)(scale * w.y);
        }
    };
    if constexpr (MODE == IN_ZPAD) {
        cx<T> C[4], S[4];
        rt_slots<T, R>(v, j, C, S);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            put(j + r * P, C[r]);
            put(M + j + r * P, S[r]);
        }
    } else {
        // rows beyond M are not kept (row M itself: j = 0 of r = 4)
#pragma unroll
        for (int r = 0; r < 4; ++r) put(j + r * P, v[r]);
        if (j == 0) put(M, v[4]);
    }
}

template <typename T, typename TI, typename TO, typename R, int MODE>
static void launch_pass_rt_m(const PassArgs &a, int ntiles, hipStream_t st)
{
    const void *fn = (const void *)&k_pass_rt<T, TI, TO, R, MODE>;
    const size_t lds = rt_lds<T, R>();
    set_lds(fn, lds);
    hipLaunchKernelGGL((k_pass_rt<T, TI, TO, R, MODE>), dim3((unsigned)ntiles), dim3(R::NTH), lds, st, a, ntiles);
}

// Full register tiles of the modes k_pass_rt takes; whether the pass is one.
template <typename T, typename TI, typename TO>
static bool launch_pass_rt(const PassArgs &a, int ntiles, hipStream_t st)
{
    const int M = a.fd.M;
    const int mode = a.in_mode;
    if (mode == IN_HERM ? a.nsum > 1 || a.nrows_in != 2 * M : mode == IN_ZPAD || mode == IN_SPECS ? a.nrows_in != M - 1 : true)
        return false;
    // synthesis keeps rows 0..M
    if (mode != IN_ZPAD && a.out_r0 + a.out_nrows > M + 1) return false;
    return rt_tile<kWide512 + (sizeof(T) == 4 ? kWide1024 + kQuad1024 : kWide1024)>(a.fd.N, a.W, [&](auto tile) {
        using R = decltype(tile);
        if (mode == IN_ZPAD)
            launch_pass_rt_m<T, TI, TO, R, IN_ZPAD>(a, ntiles, st);
        else if (mode == IN_SPECS)
            launch_pass_rt_m<T, TI, TO, R, IN_SPECS>(a, ntiles, st);
        else
            launch_pass_rt_m<T, TI, TO, R, IN_HERM>(a, ntiles, st);
    });
}

template <typename T, typename TI, typename TO, int MAXE, int KD, int NTT = NT, int WC = 0, int EPT = 0>
static void launch_pass_k(const PassArgs &a, int ntiles, size_t lds, hipStream_t st)
{
    const void *fn = (const void *)&k_pass<T, TI, TO, MAXE, KD, NTT, WC, EPT>;
    set_lds(fn, lds);
    int grid = ntiles;
    if (WC > 0) {
        const int r = resident_blocks(fn, NTT, lds);
        if (r > 0 && r < ntiles) grid = r;
    }
    hipLaunchKernelGGL((k_pass<T, TI, TO, MAXE, KD, NTT, WC, EPT>), dim3((unsigned)grid), dim3(NTT), lds, st,
                       a, ntiles);
}

// Compile-time tile widths W = 4, 8, 16 (lengths near 2M = 1024, 512, 256) with
// plain loads get the register prefetch when EPT registers per thread cover the
// loaded rows. FP32 tiles: only the forward zero-padded transforms (EPT = MAXE);
// for the inverse passes the prefetching loop measured slower than one tile per
// block.
template <int WC, int EPT>
static bool pass_fits(const PassArgs &a)
{
    return a.W == WC && PairMap<NT, WC, EPT>::covers(a.nrows_in, a.irs == 1 && a.ics != 1);
}

template <typename T, typename TI, typename TO, int MAXE, int KD>
static void launch_pass_m(const PassArgs &a, int ntiles, size_t lds, hipStream_t st)
{
    // other lengths from 2M = 512 up (the small uneven boxes of a batch measured
    // faster with one tile per block)
    if constexpr (MAXE == 8) {
        constexpr bool wide = sizeof(T) == 8; // FP64 tiles: every mode, EPT up to 2 MAXE
        // (FP32 passes of the powers of two are register tiles or narrow)
        if constexpr (wide || KD != kPow2) {
            if (!(a.in_mode == IN_HERM && a.nsum > 1) && (KD == kPow2 || a.fd.N >= 512) &&
                (wide || a.in_mode == IN_ZPAD || a.in_mode == IN_ZPAD0)) {
                if (pass_fits<8, 8>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 8, 8>(a, ntiles, lds, st);
                if (pass_fits<16, 8>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 16, 8>(a, ntiles, lds, st);
                if (pass_fits<4, 8>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 4, 8>(a, ntiles, lds, st);
                if constexpr (wide) {
                    if (pass_fits<8, 16>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 8, 16>(a, ntiles, lds, st);
                    if (pass_fits<16, 16>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 16, 16>(a, ntiles, lds, st);
                    if (pass_fits<4, 16>(a)) return launch_pass_k<T, TI, TO, 8, KD, NT, 4, 16>(a, ntiles, lds, st);
                }
            }
        }
    }
    launch_pass_k<T, TI, TO, MAXE, KD>(a, ntiles, lds, st);
}

template <typename T, typename TI, typename TO>
hipError_t launch_pass_t(const PassArgs &a, hipStream_t st)
{
    const int ncb = (a.ncols + a.W - 1) / a.W;
    const int64_t ntl = (int64_t)ncb * a.nbatch;
    const size_t lds = tile_lds<T>(a.fd.N, a.W);
    const int work = (a.W / 2) * a.fd.N;
    if (ntl <= 0) return hipSuccess;
    if (ntl > INT32_MAX) return hipErrorInvalidValue;
    const int ntiles = (int)ntl;
    if (launch_pass_rt<T, TI, TO>(a, ntiles, st)) return hipGetLastError();
    if (big_fft(a.fd.N)) {
        if (a.W != 2 || work > 8 * NTB) return hipErrorInvalidValue;
        auto go = [&](auto kd) {
            constexpr int KD = decltype(kd)::value;
            if (work <= 4 * NTB)
                launch_pass_k<T, TI, TO, 4, KD, NTB>(a, ntiles, lds, st);
            else
                launch_pass_k<T, TI, TO, 8, KD, NTB>(a, ntiles, lds, st);
        };
        // (FP32 passes of the powers of two are register tiles)
        if constexpr (sizeof(T) == 4)
            go(std::integral_constant<int, kAnyLen>());
        else
            by_pow2(a.fd.N, go);
        return hipGetLastError();
    }
    if (work > 16 * NT) return hipErrorInvalidValue;
    if (work > 8 * NT)
        by_pow2(a.fd.N, [&](auto kd) { launch_pass_m<T, TI, TO, 16, decltype(kd)::value>(a, ntiles, lds, st); });
    else
        by_kind(a.fd.N, [&](auto kd) {
            constexpr int KD = decltype(kd)::value;
            if (work <= 4 * NT)
                launch_pass_m<T, TI, TO, 4, KD>(a, ntiles, lds, st);
            else
                launch_pass_m<T, TI, TO, 8, KD>(a, ntiles, lds, st);
        });
    return hipGetLastError();
}

inline bool pass_strides_ok(const PassArgs &a)
{
    // loads address rows [0, nrows_in) of the input, stores rows [0, out_nrows) of the output
    return tile_strides_ok(a.nrows_in, a.irs, a.ncols, a.ics) && tile_strides_ok(a.out_nrows, a.ors, a.ncols, a.ocs);
}

// Several independent passes in one launch, one tile per block: block b runs
// tile b - first[i] of pass i (first[i] <= b < first[i + 1]).  The passes
// share the element types; the tile budget and the LDS are those of the
// largest tile.  Used where the passes are small (the per-family transforms
// of uneven boxes), so that they fill the device together.
template <typename T, typename TI, typename TO, int MAXE, int KD>
__global__ __launch_bounds__(NT) void k_pass_multi(MultiPassArgs m)
{
    const int b = xcd_remap(blockIdx.x, m.first[m.n]);
    int i = 0;
    while (i + 1 < m.n && b >= m.first[i + 1]) ++i;
    pass_tile<T, TI, TO, MAXE, KD, NT>(m.p[i], b - m.first[i]);
}

template <typename T, typename TI, typename TO>
hipError_t launch_multi_t(MultiPassArgs &m, hipStream_t st)
{
    size_t lds = 0;
    int work = 0, tot = 0;
    bool p2 = true, smooth = true;
    for (int i = 0; i < m.n; ++i) {
        const PassArgs &a = m.p[i];
        if (big_fft(a.fd.N) || a.W < 2 || !pass_strides_ok(a)) return hipErrorInvalidValue;
        const int64_t ntl = (int64_t)((a.ncols + a.W - 1) / a.W) * a.nbatch;
        if (ntl < 0 || tot + ntl > INT32_MAX) return hipErrorInvalidValue;
        m.first[i] = tot;
        tot += (int)ntl;
        lds = std::max(lds, tile_lds<T>(a.fd.N, a.W));
        work = std::max(work, (a.W / 2) * a.fd.N);
        p2 = p2 && is_pow2(a.fd.N);
        smooth = smooth && len_kind(a.fd.N) != kAnyLen;
    }
    m.first[m.n] = tot;
    if (tot == 0) return hipSuccess;
    if (work > 16 * NT) return hipErrorInvalidValue;
    auto go = [&](const void *fn, auto kern) {
        set_lds(fn, lds);
        hipLaunchKernelGGL(kern, dim3((unsigned)tot), dim3(NT), lds, st, m);
    };
    with_kind(p2 ? kPow2 : smooth && work <= 8 * NT ? kSmooth : kAnyLen, [&](auto kd) {
        constexpr int KD = decltype(kd)::value;
        constexpr int KL = KD == kSmooth ? kAnyLen : KD; // the largest budget: no instance of its own
        if (work <= 4 * NT)
            go((const void *)&k_pass_multi<T, TI, TO, 4, KD>, k_pass_multi<T, TI, TO, 4, KD>);
        else if (work <= 8 * NT)
            go((const void *)&k_pass_multi<T, TI, TO, 8, KD>, k_pass_multi<T, TI, TO, 8, KD>);
        else
            go((const void *)&k_pass_multi<T, TI, TO, 16, KL>, k_pass_multi<T, TI, TO, 16, KL>);
    });
    return hipGetLastError();
}

} // namespace ips
