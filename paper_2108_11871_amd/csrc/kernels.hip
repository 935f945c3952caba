// HIP kernels of the infinite-domain Poisson solver (gfx950).
//
// Stage map (paper sections):
//   k_pass    (pass.h) pencil transforms: DST-I / zero-padded cos+sin / even (DCT-I) /
//             hermitian synthesis along one axis (Sections 3, 4, 5)
//   k_cc      (conv.h) boundary values as sums over slices of 2D (3D problems) or 1D
//             (2D problems) discrete convolutions, accumulated in Fourier
//             space with the kernel spectra (Section 4, eqs. Trap2D,
//             Trap2Dconvolution, convolution)
//   k_gtilde  transfer of the boundary values of the compact operator to the
//             right-hand side next to the boundary (eq. harmonic4thOrderNH2D)
//   k_r6t     sixth-order right-hand side on the layers near the boundary,
//             from its sine coefficients (eqs. 6thOrderRelation2D/3D)
//   k_rcore,  boundary terms of that right-hand side and its cubic
//   k_dcorr   extrapolation next to the boundary (Section 5)
//   k_final   spectral combination phi_star + phi_H and first inverse pass
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <type_traits>
#include <mutex>
#include <tuple>

#include "common.h"
#include "kernels.h"

namespace ips {

// Allow more than 64 KiB of dynamic LDS where a tile needs it (gfx950 has
// 160 KiB).  Each kernel's limit is raised once per process, to the largest
// size requested so far, so that launches inside a stream capture make no
// further attribute calls.
void set_lds(const void *fn, size_t bytes)
{
    if (bytes <= 65536) return;
    static std::mutex mu;
    static std::map<const void *, size_t> done;
    std::lock_guard<std::mutex> lk(mu);
    auto it = done.find(fn);
    if (it != done.end() && it->second >= bytes) return;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess)
        done[fn] = bytes;
    else
        (void)hipGetLastError();
}


// Blocks of a kernel that fit on the device at once (occupancy times the
// number of compute units), cached per kernel, block size and LDS size.
int resident_blocks(const void *fn, int nthreads, size_t lds)
{
    static std::mutex mu;
    static std::map<std::tuple<const void *, int, size_t, int>, int> done;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_tuple(fn, nthreads, lds, dev);
    auto it = done.find(key);
    if (it != done.end()) return it->second;
    int per = 0, ncu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, nthreads, lds) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const int r = per * ncu;
    done[key] = r;
    return r;
}

// ---------------------------------------------------------------------------
// Domain extension: the caller's block of n nodes at offset off inside the
// extended grid ne (one block row of threads per grid line of the last axis).
//   extract = false: ext[off + i] = a[i]    (embed)
//   extract = true : a[i] = ext[off + i]    (restrict; a is the output)
// ---------------------------------------------------------------------------
__global__ void k_embed(const double *src, double *dst, int64_t line0, int64_t n1, int64_t n2, int64_t e1,
                        int64_t e2, int64_t o0, int64_t o1, int64_t o2, int extract)
{
    const int64_t line = line0 + blockIdx.y; // i0 * n1 + i1
    const int64_t i0 = line / n1, i1 = line % n1;
    const int64_t ebase = ((i0 + o0) * e1 + (i1 + o1)) * e2 + o2, cbase = line * n2;
    for (int64_t i2 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i2 < n2; i2 += (int64_t)gridDim.x * blockDim.x) {
        if (extract)
            dst[cbase + i2] = src[ebase + i2];
        else
            dst[ebase + i2] = src[cbase + i2];
    }
}

hipError_t launch_embed(const double *src, double *dst, int d, const int64_t *n, const int64_t *ne,
                        const int64_t *off, bool extract, hipStream_t st)
{
    int64_t c[3] = {1, 1, 1}, e[3] = {1, 1, 1}, o[3] = {0, 0, 0};
    for (int a = 0; a < d; ++a) {
        c[3 - d + a] = n[a];
        e[3 - d + a] = ne[a];
        o[3 - d + a] = off[a];
    }
    const int64_t lines = c[0] * c[1];
    const unsigned gx = (unsigned)std::min<int64_t>((c[2] + NT - 1) / NT, 64);
    // grid.y covers at most 65535 lines per launch
    for (int64_t l0 = 0; l0 < lines; l0 += 65535) {
        const unsigned nl = (unsigned)std::min<int64_t>(65535, lines - l0);
        hipLaunchKernelGGL(k_embed, dim3(gx, nl), dim3(NT), 0, st, src, dst, l0, c[1], c[2], e[1], e[2], o[0], o[1],
                           o[2], extract ? 1 : 0);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small element-wise kernels
// ---------------------------------------------------------------------------
// out[s][i] = sum over c of part[s][c][i] (i < len, s < nset, c < nchunk): the
// lanes take 64 consecutive i, the 16 waves of a block every 16th chunk with
// eight loads in flight, combined in LDS in a fixed order.
constexpr int kRedWaves = 16;

__global__ __launch_bounds__(64 * kRedWaves) void k_reduce(ReduceArgs a)
{
    const ReduceJob &jb = a.job[blockIdx.z];
    const int64_t len = jb.len;
    const int nchunk = jb.nchunk;
    __shared__ double red[kRedWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = blockIdx.x * (int64_t)64 + lane;
    const double *src = jb.part + (int64_t)blockIdx.y * nchunk * len + i;
    double s = 0.0;
    if (i < len) {
        for (int c0 = wave; c0 < nchunk; c0 += 8 * kRedWaves) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = c0 + u * kRedWaves;
                v[u] = c < nchunk ? src[(int64_t)c * len] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && i < len) {
        for (int w = 1; w < kRedWaves; ++w) s += red[w][lane];
        jb.out[(int64_t)blockIdx.y * len + i] = s;
    }
}

hipError_t launch_reduce(const ReduceArgs &a, hipStream_t st)
{
    int64_t nb = 0;
    for (int j = 0; j < a.njobs; ++j) nb = std::max(nb, (a.job[j].len + 63) / 64);
    if (nb > INT32_MAX || a.nset < 1 || a.nset > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reduce, dim3((unsigned)nb, (unsigned)a.nset, (unsigned)a.njobs), dim3(64 * kRedWaves), 0, st,
                       a);
    return hipGetLastError();
}

__global__ void k_fill(double *p, int64_t n, double v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_to_f32(const double *src, float *dst, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (float)src[i];
}

hipError_t launch_to_f32(const double *src, float *dst, int64_t n, hipStream_t st)
{
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>((n + NT - 1) / NT, 8192));
    hipLaunchKernelGGL(k_to_f32, dim3(nb), dim3(NT), 0, st, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_fill(double *p, int64_t n, double v, hipStream_t st)
{
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>((n + NT - 1) / NT, 8192));
    hipLaunchKernelGGL(k_fill, dim3(nb), dim3(NT), 0, st, p, n, v);
    return hipGetLastError();
}

// Node index helpers ---------------------------------------------------------
__device__ __forceinline__ int64_t node_off(const int64_t *n, int d, const int *i)
{
    int64_t o = 0;
    for (int a = 0; a < d; ++a) o = o * n[a] + i[a];
    return o;
}

__device__ __forceinline__ bool on_boundary(const Geo &g, const int *i)
{
    for (int a = 0; a < g.d; ++a)
        if (i[a] == 0 || i[a] == g.M[a]) return true;
    return false;
}

// Boundary value at a face node, rounded as it is stored in phi (never the product
// of a fused multiply-add).
__device__ __forceinline__ double face_val(const FaceVals &v, int fam, int f, int jlo, int jhi)
{
    double g = v.scale[fam] * v.F[fam][f * v.fs[fam][0] + jlo * v.fs[fam][1] + jhi * v.fs[fam][2]];
    asm volatile("" : "+v"(g));
    return g;
}

// ---------------------------------------------------------------------------
// Boundary values -> phi (faces, then edges and corners by lowest axis)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void write_boundary(const GtArgs &a, int64_t e)
{
    const Geo &g = a.geo;
    const int d = g.d;
    for (int fam = 0; fam < d; ++fam) {
        // ranges of the in-face axes: lower axes exclude their end nodes
        int lo[2] = {0, 0}, len[2] = {1, 1}, ax[2] = {0, 0}, na = 0;
        for (int b = 0; b < d; ++b) {
            if (b == fam) continue;
            ax[na] = b;
            lo[na] = b < fam ? 1 : 0;
            len[na] = b < fam ? g.M[b] - 1 : g.M[b] + 1;
            ++na;
        }
        const int64_t cnt = 2 * (int64_t)len[0] * len[1];
        if (e < cnt) {
            const int f = (int)(e / ((int64_t)len[0] * len[1]));
            const int64_t r = e % ((int64_t)len[0] * len[1]);
            int j[2];
            j[0] = lo[0] + (int)(na == 2 ? r / len[1] : r);
            j[1] = na == 2 ? lo[1] + (int)(r % len[1]) : 0;
            int idx[3];
            idx[fam] = f ? g.M[fam] : 0;
            for (int q = 0; q < na; ++q) idx[ax[q]] = j[q];
            a.phi[node_off(a.n, d, idx)] = face_val(a.face, fam, f, j[0], na == 2 ? j[1] : 0);
            return;
        }
        e -= cnt;
    }
}

static int64_t boundary_nodes(const Geo &g)
{
    int64_t tot = 0;
    for (int fam = 0; fam < g.d; ++fam) {
        int64_t c = 2;
        for (int b = 0; b < g.d; ++b)
            if (b != fam) c *= b < fam ? g.M[b] - 1 : g.M[b] + 1;
        tot += c;
    }
    return tot;
}

// ---------------------------------------------------------------------------
// Shell layer sizes
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ int64_t shell_size(const Geo &g, int a)
{
    int64_t s = 1;
    for (int b = 0; b < g.d; ++b)
        if (b != a) s *= g.M[b] - 1;
    return s;
}

// ---------------------------------------------------------------------------
// Parity packing of the shell spectra (see ShellSpec)
// ---------------------------------------------------------------------------
// A block takes one 16 x 16 tile of a family's (k_lo, k_hi) plane, an element per
// thread; the transposed copies go through LDS, so that every write is a run of 16.
// The g~ part (t = 0) is packed by the call without D layers, the D parts by the
// one with them. 257^3: 8 + 13 -> 6 + 7 us, 513^3 13 + 41 -> 11 + 18 us (one element
// per thread with strided copies before); bound by launch latency below. The last call
// also writes the final pass's row table from the values in hand (257^3 7 + 7 us for
// two launches -> 11); of families 1 and 2 only the call before k_r6t stores P and P1T,
// which nothing else reads (513^3 21 -> 18 us for the last call).
constexpr int kPackTile = 16;

// Row i of batch index kB - 1 of the final pass's row table [batch][M0 - 1][12] (see
// k_final for the layout), from family 1's packed spectra v = (even t = 1, 2, odd
// t = 1, 2, even t = 0, odd t = 0).
template <typename TR>
__device__ __forceinline__ void final_row_t(const PackArgs &a, int i, int b, const double *v, int64_t e)
{
    const Geo &geo = a.geo;
    const int d = geo.d, I0 = geo.M[0] - 1;
    const double lamB = d == 3 ? a.tab[2].lam[b] : 0.0, qB = d == 3 ? a.tab[2].q[b] : 0.0;
    const double c2xz = d == 3 ? geo.c2[0][2] : 0.0;
    const double c4xz = d == 3 ? geo.c4[0][2] : 0.0, c4zx = d == 3 ? geo.c4[2][0] : 0.0;
    const double lx = a.tab[0].lam[i];
    TR *r = static_cast<TR *>(a.rowtab) + e * 12;
    r[0] = (TR)lx;
    r[1] = (TR)(a.tab[0].q[i] + qB);
    r[2] = (TR)a.tab[0].s[i];
    r[3] = (TR)a.tab[0].s[I0 + i];
    r[4] = (TR)v[4];
    r[5] = (TR)v[0];
    r[6] = (TR)v[1];
    r[7] = (TR)v[5];
    r[8] = (TR)v[2];
    r[9] = (TR)v[3];
    r[10] = (TR)(lx + c2xz * lx * lamB);
    r[11] = (TR)(lx * lamB * (c4xz * lx + c4zx * lamB));
}
__device__ __forceinline__ void final_row(const PackArgs &a, int i, int b, const double *v, int64_t e)
{
    if (a.mixed)
        final_row_t<float>(a, i, b, v, e);
    else
        final_row_t<double>(a, i, b, v, e);
}

__global__ __launch_bounds__(kPackTile *kPackTile) void k_pack(PackArgs a)
{
    __shared__ double tile[6][kPackTile][kPackTile + 1];
    const Geo &g = a.geo;
    int fam = 0, blk = blockIdx.x;
    while (fam < g.d - 1 && blk >= a.nblk[fam]) blk -= a.nblk[fam++];
    const int lo = fam == 0 ? 1 : 0, hi = fam == 2 ? 1 : 2;
    const int Il = g.d == 3 ? g.M[lo] - 1 : 1, Ih = (g.d == 3 ? g.M[hi] : g.M[1 - fam]) - 1;
    const int nbh = (Ih + kPackTile - 1) / kPackTile;
    const int r0 = blk / nbh * kPackTile, c0 = blk % nbh * kPackTile;
    const int64_t ss = (int64_t)Il * Ih;
    const int tx = threadIdx.x & (kPackTile - 1), ty = threadIdx.x / kPackTile;
    const bool tr = g.d == 3 && fam > 0;
    const bool rows = fam == 1 && a.rowtab; // (the last call: all parts are known)
    const int nk = a.withD ? 4 : 2; // values per element, of kind (parity, t)
    const bool keep = !a.withD && !a.rowtab; // k_r6t follows
    auto kind = [&](int q) { return a.withD ? (q >> 1) * 3 + 1 + (q & 1) : 3 * q; };
    if (r0 + ty < Il && c0 + tx < Ih) {
        const int64_t e = (int64_t)(r0 + ty) * Ih + c0 + tx;
        double v[6];
        if (!a.withD || rows) {
            const double g0 = a.G[fam][e], g1 = a.G[fam][ss + e];
            v[0] = v[4] = g0 - g1; // even k, t = 0
            v[1] = v[5] = g0 + g1; // odd k, t = 0
        }
        if (a.withD) {
            const double *D = a.D[fam];
            const double d1 = D[e], d2 = D[ss + e], d3 = D[2 * ss + e], d4 = D[3 * ss + e];
            v[0] = d1 - d4; // even k, t = 1
            v[1] = d2 - d3; // even k, t = 2
            v[2] = d1 + d4; // odd k, t = 1
            v[3] = d2 + d3; // odd k, t = 2
        } else {
            v[2] = v[3] = 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= nk) break;
            if (fam == 0 || keep) a.P[fam][kind(q) * ss + e] = v[q];
            if (tr) tile[q][ty][tx] = v[q];
        }
        if (tr && rows) {
            tile[4][ty][tx] = v[4];
            tile[5][ty][tx] = v[5];
        }
        if (!tr && rows) {
            if (!a.withD) v[0] = v[1] = 0.0;
            final_row(a, c0 + tx, 0, v, e);
        }
    }
    if (!tr) return;
    __syncthreads();
    // (k_lo, k_hi) -> [k_hi][k_lo]: lo is axis 0 of families 1 and 2
    if (c0 + ty >= Ih || r0 + tx >= Il) return;
    const int64_t et = (int64_t)(c0 + ty) * Il + r0 + tx;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q >= nk) break;
        const double v = tile[q][tx][ty];
        if (fam == 1) {
            if (keep) a.P1T[kind(q) * ss + et] = v;
        } else if (a.p2t_f32)
            static_cast<float *>(a.P2T)[kind(q) * ss + et] = (float)v;
        else
            static_cast<double *>(a.P2T)[kind(q) * ss + et] = v;
    }
    if (rows) {
        double v[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) v[q] = q < 4 && !a.withD ? 0.0 : tile[q][tx][ty];
        final_row(a, r0 + tx, c0 + ty, v, et);
    }
}

hipError_t launch_pack(PackArgs a, hipStream_t st)
{
    const Geo &g = a.geo;
    int tot = 0;
    for (int fam = 0; fam < g.d; ++fam) {
        const int lo = fam == 0 ? 1 : 0, hi = fam == 2 ? 1 : 2;
        const int Il = g.d == 3 ? g.M[lo] - 1 : 1, Ih = (g.d == 3 ? g.M[hi] : g.M[1 - fam]) - 1;
        a.nblk[fam] = (Il + kPackTile - 1) / kPackTile * ((Ih + kPackTile - 1) / kPackTile);
        tot += a.nblk[fam];
    }
    hipLaunchKernelGGL(k_pack, dim3((unsigned)tot), dim3(kPackTile * kPackTile), 0, st, a);
    return hipGetLastError();
}

// 1/x from the hardware reciprocal refined by two Newton steps
// (each doubles the correct bits: the result is within an ulp or two of 1/x).
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// FP32: one Newton step on the hardware reciprocal.
__device__ __forceinline__ float recip(float x)
{
    float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}


// ---------------------------------------------------------------------------
// Sixth-order right-hand side of the harmonic part, interior contribution.
// The stencils applied to the interior part of u1 act on its sine
// coefficients as the symbol m_R(k); so the coefficients of that part of the
// right-hand side are
//     V(k) = prod(2/M) * m_R(k) * gt_hat(k) / Lambda(k).
// Its values on the layers j = 1..5 and M-5..M-1 of every axis a are
//     T_a[j][k_other] = sum_{k_a} sin(pi k_a j / M_a) V(k)
// (followed by an inverse sine transform over the other axes).  Parity:
// sin(pi k (M-j)/M) = (-1)^(k+1) sin(pi k j / M).
//
// k_r6t computes the three (two in 2D) contractions in one launch and never
// stores V: each thread owns one position (k_b, k_c) and sums over a quarter
// of the k_a, rebuilding V(k) from the packed shell spectra:
//   gt_hat = sin(pi k_a/M_a) G_a(k_b, k_c) + sin(pi k_l/M_l) G_l(.., k_a, ..)
//            + sin(pi k_w/M_w) G_w(.., k_a, ..)
// where l is the axis that varies across the lanes of a wave and w the
// other one.  The lanes read G_w contiguously (3D: for a = 2 from the
// transposed family-1 copy) and G_l at one of two addresses (parity of
// k_l).  With lambda_a the only varying eigenvalue,
//   Lambda = A0 + A1 lambda_a,  m_R = B0 + lambda_a (B1 + B2 lambda_a).
// Block: 64 PPT positions x 4 wave groups; group g takes k_a = 1 + g + 4t,
// so its parity is fixed and the layer pairs split into odd and even sums.
// Each thread carries PPT positions (64 apart) through the k_a loop: their
// loads and reciprocals are independent, which hides more latency per wave.
// ---------------------------------------------------------------------------
template <int D, int PPT, int KU>
__global__ __launch_bounds__(NT) void k_r6t(R6Args a)
{
    constexpr int PB = 64 * PPT, NG = NT / 64;
    __shared__ double red[NG][5][PB];
    const Geo &g = a.geo;
    int ax = 0, blk = blockIdx.x;
    while (ax < D - 1 && blk >= a.nblk[ax]) {
        blk -= a.nblk[ax];
        ++ax;
    }
    const int lane = threadIdx.x & 63;
    const int grp = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int Ia = g.M[ax] - 1;
    int la, wa;
    if (D == 3) {
        la = ax == 2 ? 0 : 2;
        wa = ax == 1 ? 0 : 1;
    } else {
        la = 1 - ax;
        wa = -1;
    }
    const int Il = g.M[la] - 1;
    const int Iw = D == 3 ? g.M[wa] - 1 : 1;
    const int npos = Il * Iw;
    const int para = (grp & 1) ? 0 : 1; // parity of k_a in this group
    const int64_t ssa = shell_size(g, ax), ssl = shell_size(g, la);
    // per position q (PPT independent positions per thread, 64 apart)
    double A0[PPT], A1[PPT], B0[PPT], B1[PPT], B2[PPT], gown[PPT], sbl[PPT], scw[PPT];
    const double *pb[PPT], *pc[PPT];
    int64_t bs = 1, cs = 0;
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int p = blk * PB + q * 64 + lane;
        const int pp = p < npos ? p : 0;
        const int kl = 1 + pp % Il;
        const int kw = 1 + pp / Il;
        // symbols as polynomials in lambda_a
        const double lamL = a.tab[la].lam[kl - 1];
        A0[q] = lamL;
        A1[q] = 1.0 + g.c2[ax][la] * lamL;
        B0[q] = 0.0;
        B1[q] = g.c4[la][ax] * lamL * lamL;
        B2[q] = g.c4[ax][la] * lamL;
        if (D == 3) {
            const double lamW = a.tab[wa].lam[kw - 1];
            A0[q] += lamW + g.c2[la][wa] * lamL * lamW;
            A1[q] += g.c2[ax][wa] * lamW;
            B0[q] = g.c4[la][wa] * lamL * lamL * lamW + g.c4[wa][la] * lamL * lamW * lamW;
            B1[q] += g.c4[wa][ax] * lamW * lamW;
            B2[q] += g.c4[ax][wa] * lamW;
        }
        // own family (normal to a): fixed value for this group's parity
        int64_t oown;
        if (D == 3)
            oown = ax == 2 ? (int64_t)(kl - 1) * Iw + (kw - 1) : (int64_t)(kw - 1) * Il + (kl - 1);
        else
            oown = kl - 1;
        gown[q] = a.P[ax][(int64_t)para * 3 * ssa + oown];
        // family normal to the lane axis: two addresses per wave
        sbl[q] = a.tab[la].s[kl - 1];
        pb[q] = a.P[la] + (int64_t)(kl & 1) * 3 * ssl;
        if (D == 3) {
            if (ax == 0) {
                pb[q] += kw - 1; // G_2[k0][k1], k0 = k_a
                bs = Iw;
            } else if (ax == 1) {
                pb[q] += (int64_t)(kw - 1) * (g.M[1] - 1); // G_2[k0][k1], k1 = k_a
            } else {
                pb[q] += (int64_t)(kw - 1) * (g.M[2] - 1); // G_0[k1][k2], k2 = k_a
            }
        }
        // family normal to the wave axis (3D): contiguous across the lanes
        pc[q] = nullptr;
        scw[q] = 0.0;
        if (D == 3) {
            const int64_t ssw = shell_size(g, wa);
            scw[q] = a.tab[wa].s[kw - 1];
            const double *base = ax == 2 ? a.P1T : a.P[wa];
            pc[q] = base + (int64_t)(kw & 1) * 3 * ssw + (kl - 1);
            cs = ax == 2 ? (g.M[0] - 1) : (g.M[2] - 1);
        }
    }
    const double *tl = a.tab[ax].lam;
    const double *ts = a.tab[ax].s;
    double acc[PPT][5];
#pragma unroll
    for (int q = 0; q < PPT; ++q)
#pragma unroll
        for (int j = 0; j < 5; ++j) acc[q][j] = 0.0;
    // split s of gridDim.y: every gridDim.y-th wavenumber of this group's
    // residue (the parity of k_a stays that of the group)
    const int ks = gridDim.y, sp = blockIdx.y, step = NG * ks;
    // one wavenumber: pbv, pcv are the family values at (position q, ka)
    auto term = [&](int ka, const double *pbv, const double *pcv) {
        const double lk = tl[ka - 1], sk = ts[ka - 1];
        double sj[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) sj[j] = ts[j * Ia + ka - 1];
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            double gt = sk * gown[q] + sbl[q] * pbv[q];
            if (D == 3) gt += scw[q] * pcv[q];
            const double L = fma(A1[q], lk, A0[q]);
            const double R = fma(fma(B2[q], lk, B1[q]), lk, B0[q]);
            const double v = R * gt * recip(L);
#pragma unroll
            for (int j = 0; j < 5; ++j) acc[q][j] = fma(sj[j], v, acc[q][j]);
        }
    };
    // KU wavenumbers per iteration, their strided family loads issued first
    // (more loads in flight per wave)
    int ka = 1 + grp + NG * sp;
    for (; ka + (KU - 1) * step <= Ia; ka += KU * step) {
        double pbv[KU][PPT], pcv[KU][PPT];
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const int64_t k1 = ka - 1 + u * step;
                pbv[u][q] = pb[q][k1 * bs];
                pcv[u][q] = D == 3 ? pc[q][k1 * cs] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < KU; ++u) term(ka + u * step, pbv[u], pcv[u]);
    }
    for (; ka <= Ia; ka += step) {
        double pbv[PPT], pcv[PPT];
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            pbv[q] = pb[q][(int64_t)(ka - 1) * bs];
            pcv[q] = D == 3 ? pc[q][(int64_t)(ka - 1) * cs] : 0.0;
        }
        term(ka, pbv, pcv);
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q)
#pragma unroll
        for (int j = 0; j < 5; ++j) red[grp][j][q * 64 + lane] = acc[q][j];
    __syncthreads();
    // group g finishes positions g*64/...: every thread of the block writes
    // its share of the PB positions
    // several splits: FP64 partials [split][10][positions] of this axis,
    // summed into T by k_r6t_sum
    double *Td = ks > 1 ? a.part + a.part_off[ax] + (int64_t)sp * 10 * npos : static_cast<double *>(a.T[ax]);
    float *Tf = static_cast<float *>(a.T[ax]);
    for (int i = threadIdx.x; i < PB; i += NT) {
        const int p = blk * PB + i;
        if (p >= npos) continue;
        const int kl = 1 + p % Il, kw = 1 + p / Il;
        const int64_t pout = (D == 3 && ax == 2) ? (int64_t)(kl - 1) * Iw + (kw - 1) : p;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const double od = red[0][j][i] + red[2][j][i];
            const double ev = red[1][j][i] + red[3][j][i];
            const double v1 = g.pref * (od + ev), v2 = g.pref * (od - ev);
            if (a.t_f32 && ks == 1) {
                Tf[j * (int64_t)npos + pout] = (float)v1;
                Tf[(5 + j) * (int64_t)npos + pout] = (float)v2;
            } else {
                Td[j * (int64_t)npos + pout] = v1;
                Td[(5 + j) * (int64_t)npos + pout] = v2;
            }
        }
    }
}

// T[ax][l][p] = sum over the splits of part[ax][s][l][p] (10 layers of npos)
__global__ void k_r6t_sum(R6Args a, int ks)
{
    const int ax = blockIdx.y;
    const int64_t len = 10 * shell_size(a.geo, ax);
    const double *src = a.part + a.part_off[ax];
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len; i += (int64_t)gridDim.x * blockDim.x) {
        double v = 0.0;
        for (int sp = 0; sp < ks; ++sp) v += src[(int64_t)sp * len + i];
        if (a.t_f32)
            static_cast<float *>(a.T[ax])[i] = (float)v;
        else
            static_cast<double *>(a.T[ax])[i] = v;
    }
}

template <int PPT, int KU>
static hipError_t launch_r6t_p(R6Args a, hipStream_t st)
{
    const int d = a.geo.d;
    int tot = 0;
    for (int ax = 0; ax < d; ++ax) {
        const int np = (int)shell_size(a.geo, ax);
        a.nblk[ax] = (np + 64 * PPT - 1) / (64 * PPT);
        tot += a.nblk[ax];
    }
    const int ks = r6t_splits(a.geo);
    if (ks > 1 && !a.part) return hipErrorInvalidValue;
    if (d == 3)
        hipLaunchKernelGGL((k_r6t<3, PPT, KU>), dim3(tot, ks), dim3(NT), 0, st, a);
    else
        hipLaunchKernelGGL((k_r6t<2, PPT, KU>), dim3(tot, ks), dim3(NT), 0, st, a);
    hipError_t e = hipGetLastError();
    if (ks > 1 && e == hipSuccess) {
        int64_t len = 0;
        for (int ax = 0; ax < d; ++ax) len = std::max(len, 10 * shell_size(a.geo, ax));
        const unsigned nb = (unsigned)std::min<int64_t>((len + NT - 1) / NT, 4096);
        hipLaunchKernelGGL(k_r6t_sum, dim3(nb, (unsigned)d), dim3(NT), 0, st, a, ks);
        e = hipGetLastError();
    }
    return e;
}

// two positions per thread, two wavenumbers per iteration (measured against
// one and four of each)
hipError_t launch_r6t(R6Args a, hipStream_t st) { return launch_r6t_p<2, 2>(a, st); }

int r6t_splits(const Geo &g)
{
    int tot = 0, mina = 1 << 30;
    for (int ax = 0; ax < g.d; ++ax) {
        tot += (int)((shell_size(g, ax) + 127) / 128);
        mina = std::min(mina, g.M[ax] - 1);
    }
    const int want = (1024 + tot - 1) / tot;
    const int cap = std::max(1, mina / 128);
    return std::max(1, std::min(want, cap));
}

// ---------------------------------------------------------------------------
// D = R - R_spec on the nodes with an index in {1, 2, M-2, M-1}, in two steps.
//   k_rcore: R on the core nodes with an index along axis a in
//            {2..5, M-5..M-2}:  R = R_spec + boundary terms, where a
//            D2^2 D2 stencil centred on index 2 or M-2 of some axis x reaches
//            the face of x: c4[x][y] D2_y g / h_x^4 for every y != x.
//            C[a][l][other], l = 0..7 for the layers 2,3,4,5,M-5,..,M-2.
//   k_dcorr: R at the shell nodes by tensor-product cubic extrapolation
//            (index 1 <- 4,-6,4,-1 times indices 2..5, mirrored at M-1),
//            minus R_spec.  A node belongs to the lowest axis that has an
//            index in {1, 2, M-2, M-1} there; other layers hold 0.
// Both read R_spec only from the layers of their own axis.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int layer5(int i, int M)
{
    return i <= 5 ? i - 1 : 5 + (M - 1 - i);
}

template <int D>
__device__ __forceinline__ void other_axes(int a, int *ob)
{
    int q = 0;
    for (int b = 0; b < D; ++b)
        if (b != a) ob[q++] = b;
}

// R_spec value (FP32 or FP64 storage)
__device__ __forceinline__ double rs_at(const DcorrArgs &a, int fam, int64_t o)
{
    return a.rs_f32 ? (double)static_cast<const float *>(a.RS[fam])[o] : static_cast<const double *>(a.RS[fam])[o];
}

template <int D>
__global__ __launch_bounds__(NT) void k_rcore(DcorrArgs a)
{
    const Geo &g = a.geo;
    const int fam = blockIdx.y >> 3, l = blockIdx.y & 7;
    const int64_t ss = shell_size(g, fam);
    const int e = blockIdx.x * NT + threadIdx.x;
    if (e >= ss) return;
    int ob[2] = {0, 0};
    other_axes<D>(fam, ob);
    int i[3] = {0, 0, 0};
    const int Mf = g.M[fam];
    i[fam] = l < 4 ? 2 + l : Mf - 2 - (7 - l);
    if (D == 3) {
        const int Ic = g.M[ob[1]] - 1;
        i[ob[0]] = 1 + e / Ic;
        i[ob[1]] = 1 + e % Ic;
    } else {
        i[ob[0]] = 1 + e;
    }
    bool core = true;
    for (int b = 0; b < D; ++b) core = core && i[b] >= 2 && i[b] <= g.M[b] - 2;
    double v = 0.0;
    if (core) {
        v = rs_at(a, fam, (int64_t)layer5(i[fam], Mf) * ss + e);
#pragma unroll
        for (int x = 0; x < D; ++x) {
            if (i[x] != 2 && i[x] != g.M[x] - 2) continue;
            int q[3] = {i[0], i[1], i[2]};
            q[x] = i[x] == 2 ? 0 : g.M[x];
            double t = 0.0;
#pragma unroll
            for (int y = 0; y < D; ++y) {
                if (y == x) continue;
                int qm[3] = {q[0], q[1], q[2]}, qp[3] = {q[0], q[1], q[2]};
                qm[y] -= 1;
                qp[y] += 1;
                const double f0 = a.phi[node_off(a.n, D, q)];
                const double fm = a.phi[node_off(a.n, D, qm)];
                const double fp = a.phi[node_off(a.n, D, qp)];
                t += g.c4[x][y] * (fm - 2.0 * f0 + fp) / (g.h[y] * g.h[y]);
            }
            const double h2 = g.h[x] * g.h[x];
            v += t / (h2 * h2);
        }
    }
    a.C[fam][(int64_t)l * ss + e] = v;
}

template <int D>
__global__ __launch_bounds__(NT) void k_dcorr(DcorrArgs a)
{
    const Geo &g = a.geo;
    const int fam = blockIdx.y >> 2, jj = blockIdx.y & 3;
    const int64_t ss = shell_size(g, fam);
    const int e = blockIdx.x * NT + threadIdx.x;
    if (e >= ss) return;
    int ob[2] = {0, 0};
    other_axes<D>(fam, ob);
    const int Mf = g.M[fam];
    const int L4[4] = {1, 2, Mf - 2, Mf - 1};
    int i[3] = {0, 0, 0};
    i[fam] = L4[jj];
    int Ic = 1;
    if (D == 3) {
        Ic = g.M[ob[1]] - 1;
        i[ob[0]] = 1 + e / Ic;
        i[ob[1]] = 1 + e % Ic;
    } else {
        i[ob[0]] = 1 + e;
    }
    bool owned = true;
    for (int b = 0; b < fam; ++b) {
        const int m = g.M[b];
        if (i[b] == 1 || i[b] == 2 || i[b] == m - 2 || i[b] == m - 1) owned = false;
    }
    double out = 0.0;
    if (owned) {
        const double *C = a.C[fam];
        // along the family axis (uniform over the block)
        const bool exa = jj == 0 || jj == 3;
        int l0;
        if (jj == 0)
            l0 = 0;
        else if (jj == 3)
            l0 = 7;
        else
            l0 = jj == 1 ? 0 : 7;
        const int dl = jj == 3 ? -1 : 1;
        // in-face axes: 1 or 4 taps each
        int nt[2] = {1, 1}, p0[2] = {0, 0}, dp[2] = {0, 0};
        for (int q = 0; q < D - 1; ++q) {
            const int b = ob[q], m = g.M[b];
            if (i[b] == 1) {
                nt[q] = 4;
                p0[q] = 2;
                dp[q] = 1;
            } else if (i[b] == m - 1) {
                nt[q] = 4;
                p0[q] = m - 2;
                dp[q] = -1;
            } else {
                p0[q] = i[b];
            }
        }
        const double wt[4] = {4.0, -6.0, 4.0, -1.0};
        double R = 0.0;
        for (int t0 = 0; t0 < nt[0]; ++t0) {
            const double w0 = nt[0] == 1 ? 1.0 : wt[t0];
            const int pb = p0[0] + dp[0] * t0;
            for (int t1 = 0; t1 < (D == 3 ? nt[1] : 1); ++t1) {
                const double w1 = (D == 3 && nt[1] == 4) ? wt[t1] : 1.0;
                const int pc = D == 3 ? p0[1] + dp[1] * t1 : 1;
                const int64_t o = D == 3 ? (int64_t)(pb - 1) * Ic + (pc - 1) : pb - 1;
                double v;
                if (exa) {
                    const double c0 = C[(int64_t)(l0)*ss + o], c1 = C[(int64_t)(l0 + dl) * ss + o];
                    const double c2 = C[(int64_t)(l0 + 2 * dl) * ss + o], c3 = C[(int64_t)(l0 + 3 * dl) * ss + o];
                    v = 4.0 * c0 - 6.0 * c1 + 4.0 * c2 - c3;
                } else {
                    v = C[(int64_t)l0 * ss + o];
                }
                R += w0 * w1 * v;
            }
        }
        out = R - rs_at(a, fam, (int64_t)layer5(i[fam], Mf) * ss + e);
    }
    a.D[fam][(int64_t)jj * ss + e] = out;
}

hipError_t launch_dcorr(const DcorrArgs &a, hipStream_t st)
{
    const int d = a.geo.d;
    int64_t mx = 1;
    for (int fam = 0; fam < d; ++fam) mx = std::max(mx, shell_size(a.geo, fam));
    const unsigned nb = (unsigned)((mx + NT - 1) / NT);
    if (d == 3) {
        hipLaunchKernelGGL(k_rcore<3>, dim3(nb, 8 * d), dim3(NT), 0, st, a);
        hipLaunchKernelGGL(k_dcorr<3>, dim3(nb, 4 * d), dim3(NT), 0, st, a);
    } else {
        hipLaunchKernelGGL(k_rcore<2>, dim3(nb, 8 * d), dim3(NT), 0, st, a);
        hipLaunchKernelGGL(k_dcorr<2>, dim3(nb, 4 * d), dim3(NT), 0, st, a);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// g~ = -(L_h B) on the interior nodes next to the boundary, split into one
// layer pair per axis (a node belongs to the lowest axis whose index is 1 or
// M-1 there; other layers hold 0 at that node). Nodes away from the edges read their
// five neighbours from the face array; the others all 18 at once (bound by the latency
// of these loads: one after the other 12 us on the smallest grid; 513^3 113 -> 41 us,
// whose z faces are a row apart per node in phi). FACES: boundary values come from the
// face arrays, and the block rows from 2 D on write them to phi, in one launch (257^3
// 11 + 15 -> 14 us, 33^3 4 + 11 -> 5 us and a launch less); else they are in phi.
// ---------------------------------------------------------------------------
template <int D, bool FACES>
__global__ __launch_bounds__(NT) void k_gtilde(GtArgs a)
{
    if (FACES && blockIdx.y >= 2 * D) {
        write_boundary(a, ((int64_t)(blockIdx.y - 2 * D) * gridDim.x + blockIdx.x) * NT + threadIdx.x);
        return;
    }
    const Geo &g = a.geo;
    const int fam = blockIdx.y >> 1, f = blockIdx.y & 1;
    const int64_t ss = shell_size(g, fam);
    const int e = blockIdx.x * NT + threadIdx.x;
    if (e >= ss) return;
    int ob[2] = {0, 0};
    other_axes<D>(fam, ob);
    int i[3] = {0, 0, 0};
    i[fam] = f ? g.M[fam] - 1 : 1;
    if (D == 3) {
        const int Ic = g.M[ob[1]] - 1;
        i[ob[0]] = 1 + e / Ic;
        i[ob[1]] = 1 + e % Ic;
    } else {
        i[ob[0]] = 1 + e;
    }
    // with M = 2 both layers are the same nodes: keep only the first
    bool owned = !(f == 1 && g.M[fam] == 2);
    for (int b = 0; b < fam; ++b)
        if (i[b] == 1 || i[b] == g.M[b] - 1) owned = false;
    double s = 0.0;
    bool bulk = FACES && g.M[fam] > 2;
#pragma unroll
    for (int q = 0; q < D - 1; ++q) bulk = bulk && i[ob[q]] >= 2 && i[ob[q]] <= g.M[ob[q]] - 2;
    auto add = [&](double w, double v) { // (no fused multiply-add)
        double t = w * v;
        asm volatile("" : "+v"(t));
        s += t;
    };
    if (bulk) {
        // only the node's own face is near: its neighbours there, from the face array
        // (contiguous across the lanes), in the order of the general sum below
        const int jl = i[ob[0]], jh = D == 3 ? i[ob[1]] : 0;
        double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        const double *F = a.face.F[fam] + f * a.face.fs[fam][0] + jl * a.face.fs[fam][1] + jh * a.face.fs[fam][2];
        v[0] = F[0];
#pragma unroll
        for (int q = 0; q < D - 1; ++q) {
            v[1 + 2 * q] = F[-a.face.fs[fam][1 + q]];
            v[2 + 2 * q] = F[a.face.fs[fam][1 + q]];
        }
        asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]));
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            v[q] = a.face.scale[fam] * v[q];
            asm volatile("" : "+v"(v[q])); // as stored in phi
        }
        add(a.wf[fam], v[0]);
#pragma unroll
        for (int q = 0; q < D - 1; ++q) {
            add(a.we[fam][ob[q]], v[1 + 2 * q]);
            add(a.we[fam][ob[q]], v[2 + 2 * q]);
        }
        s = -s;
    } else if (owned) {
        // every neighbour is a grid node: all are loaded at once, those off the
        // boundary dropped
        double v[2 * D + 2 * D * (D - 1)];
        double scl[FACES ? 2 * D + 2 * D * (D - 1) : 1];
        bool on[2 * D + 2 * D * (D - 1)];
        int m = 0;
        auto get = [&](int p, int sp, int q, int sq) {
            int j[3] = {i[0], i[1], i[2]};
            j[p] += sp;
            j[q] += sq;
            bool any = false;
            if constexpr (FACES) {
                // the face of the lowest axis at its end, as in phi
                const double *F = nullptr;
                double sc = 0.0;
                int o = 0;
#pragma unroll
                for (int b = D - 1; b >= 0; --b) {
                    const bool at = j[b] == 0 || j[b] == g.M[b];
                    const int lo = b == 0 ? 1 : 0, hi = b == 2 ? 1 : 2;
                    const int ob = (j[b] ? (int)a.face.fs[b][0] : 0) + j[lo] * (int)a.face.fs[b][1] +
                                   (D == 3 ? j[hi] * (int)a.face.fs[b][2] : 0);
                    const bool take = at || b == D - 1; // (of no face: any address)
                    F = take ? a.face.F[b] : F;
                    sc = take ? a.face.scale[b] : sc;
                    o = take ? ob : o;
                    any = any || at;
                }
                v[m] = F[any ? o : 0];
                scl[m] = sc;
            } else {
                v[m] = a.phi[node_off(a.n, D, j)];
                any = on_boundary(g, j);
            }
            on[m++] = any;
        };
#pragma unroll
        for (int p = 0; p < D; ++p) {
            get(p, -1, p, 0);
            get(p, 1, p, 0);
        }
#pragma unroll
        for (int p = 0; p < D; ++p)
#pragma unroll
            for (int q = p + 1; q < D; ++q) {
                get(p, -1, q, -1);
                get(p, -1, q, 1);
                get(p, 1, q, -1);
                get(p, 1, q, 1);
            }
        // (one use of all of them: the loads are in flight together)
        if constexpr (D == 3) {
            asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),
                         "+v"(v[7]), "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]), "+v"(v[12]), "+v"(v[13]),
                         "+v"(v[14]), "+v"(v[15]), "+v"(v[16]), "+v"(v[17]));
        } else {
            asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),
                         "+v"(v[7]));
        }
        m = 0;
        auto use = [&](double w) {
            double t = v[m];
            if constexpr (FACES) {
                t = scl[m] * t;
                asm volatile("" : "+v"(t)); // as stored in phi
            }
            add(w, on[m] ? t : 0.0);
            ++m;
        };
#pragma unroll
        for (int p = 0; p < D; ++p) {
            use(a.wf[p]);
            use(a.wf[p]);
        }
#pragma unroll
        for (int p = 0; p < D; ++p)
#pragma unroll
            for (int q = p + 1; q < D; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) use(a.we[p][q]);
        s = -s;
    }
    a.G[fam][(int64_t)f * ss + e] = s;
}

hipError_t launch_gtilde(GtArgs a, hipStream_t st)
{
    const int d = a.geo.d;
    const Geo &g = a.geo;
    // weights of L_h's face and edge neighbours
    for (int p = 0; p < d; ++p) {
        a.wf[p] = 1.0 / (g.h[p] * g.h[p]);
        for (int q = 0; q < d; ++q) {
            if (q == p) continue;
            a.wf[p] -= 2.0 * g.c2[p][q] / (g.h[p] * g.h[p] * g.h[q] * g.h[q]);
            const int lo = std::min(p, q), hi = std::max(p, q);
            a.we[p][q] = g.c2[lo][hi] / (g.h[lo] * g.h[lo] * g.h[hi] * g.h[hi]);
        }
    }
    int64_t mx = 1;
    for (int fam = 0; fam < d; ++fam) mx = std::max(mx, shell_size(a.geo, fam));
    const unsigned nb = (unsigned)((mx + NT - 1) / NT);
    const bool faces = a.face.F[0] != nullptr;
    const unsigned nw = faces ? (unsigned)((boundary_nodes(g) + (int64_t)nb * NT - 1) / ((int64_t)nb * NT)) : 0;
    const dim3 grid(nb, 2 * d + nw);
    if (d == 3 && faces)
        hipLaunchKernelGGL((k_gtilde<3, true>), grid, dim3(NT), 0, st, a);
    else if (d == 3)
        hipLaunchKernelGGL((k_gtilde<3, false>), grid, dim3(NT), 0, st, a);
    else if (faces)
        hipLaunchKernelGGL((k_gtilde<2, true>), grid, dim3(NT), 0, st, a);
    else
        hipLaunchKernelGGL((k_gtilde<2, false>), grid, dim3(NT), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Final pass along axis 0: raw DST of B along axis 0 -> beta (raw DST of rho),
// spectral combination
//   c(k) = prod(2/M) [ -beta / (pi^2 sum k^2/L^2)
//                      + (gt_hat (1 + m_R/Lambda) + D_hat) / Lambda ]   (order 6)
//   c(k) = prod(2/M) [ -beta / (pi^2 sum k^2/L^2) + gt_hat / Lambda ]     (order 4)
// then the inverse sine transform along axis 0, written back in place.
// ---------------------------------------------------------------------------
// The 12 staged values of one row or column of the final pass, read as
// 16-byte vectors (records are 16-byte aligned in both spaces).
__device__ __forceinline__ void load12(const float *p, float *r)
{
    const float4 *v = reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float4 t = v[i];
        r[4 * i] = t.x;
        r[4 * i + 1] = t.y;
        r[4 * i + 2] = t.z;
        r[4 * i + 3] = t.w;
    }
}
__device__ __forceinline__ void load12(const double *p, double *r)
{
    const double2 *v = reinterpret_cast<const double2 *>(p);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const double2 t = v[i];
        r[2 * i] = t.x;
        r[2 * i + 1] = t.y;
    }
}

// Tile lb of the final pass -> (column block, batch entry), in the logical order:
// groups of a.group neighbouring column blocks (together 256 bytes of every row),
// then the batch, then the group index -- the blocks that share a line run side
// by side on one XCD, and each XCD sweeps all batches over a narrow band of columns,
// so the per-element shell data of that band stays in its L2.
__device__ __forceinline__ void final_tile(const FinalArgs &a, int ncb, int lb, int &cb, int &bt)
{
    const int G = a.group;
    const int full = ncb / G;
    if (lb < G * full * a.nbatch) {
        const int pr = lb / (G * a.nbatch), rem = lb % (G * a.nbatch);
        bt = rem / G;
        cb = G * pr + rem % G;
    } else {
        const int left = ncb - G * full; // the last, partial group
        const int rem = lb - G * full * a.nbatch;
        bt = rem / left;
        cb = G * full + rem % left;
    }
}

// Staged column j = k1 - 1 of the final pass at batch index kB = k2: 12 values
// (layout below, in k_final).
template <typename T>
__device__ __forceinline__ void final_col(const FinalArgs &a, int j, int kB, T *r)
{
    const Geo &geo = a.geo;
    const int d = geo.d, I1 = geo.M[1] - 1, I2 = d == 3 ? geo.M[2] - 1 : 1;
    const int nt = a.order == 6 ? 3 : 1;
    const double lamB = d == 3 ? a.tab[2].lam[kB - 1] : 0.0;
    const double c2yz = d == 3 ? geo.c2[1][2] : 0.0;
    const double c4yz = d == 3 ? geo.c4[1][2] : 0.0, c4zy = d == 3 ? geo.c4[2][1] : 0.0;
    const double ly = a.tab[1].lam[j];
    r[0] = (T)ly;
    r[1] = (T)a.tab[1].q[j];
    r[2] = (T)a.tab[1].s[j];
    r[3] = (T)a.tab[1].s[I1 + j];
    r[10] = (T)(ly + c2yz * ly * lamB);
    r[11] = (T)(ly * lamB * (c4yz * ly + c4zy * lamB));
    // family 0: other index (k1, k2) in 3D, (k1) in 2D
    const int64_t ss0 = shell_size(geo, 0), o = d == 3 ? (int64_t)j * I2 + (kB - 1) : j;
    for (int par = 0; par < 2; ++par)
        for (int t = 0; t < nt; ++t) r[4 + par * 3 + t] = (T)a.sh.P0[(par * 3 + t) * ss0 + o];
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One coefficient of the combination: row record r and column record q (layout in
// k_final), kxodd / kyodd the parities of the wavenumbers, Pe the family-2 values of
// the element (stride ss2), beta the raw sine coefficient of rho. The fused
// operations are written out, so that every kernel rounds alike.
template <typename T>
struct FinalConst {
    T c2xy, c4xy, c4yx, pref, lamB, s1B, s2B;
    int64_t ss2;
    bool six, d3;
};

template <typename T>
__device__ __forceinline__ T final_value(const FinalConst<T> &f, const T *r, const T *q, bool kxodd, bool kyodd,
                                         const T *Pe, T beta)
{
    const T *Pr = r + (kyodd ? 7 : 4), *Pc = q + (kxodd ? 7 : 4);
    const T lxy = r[0] * q[0];
    const T L = fma_t(f.c2xy, lxy, r[10] + q[10] + f.lamB);
    T h = fma_t(q[2], Pr[0], r[2] * Pc[0]);
    T dh = (T)0;
    if (f.six) dh = fma_t(q[3], Pr[2], fma_t(q[2], Pr[1], fma_t(r[2], Pc[1], r[3] * Pc[2])));
    if (f.d3) {
        h = fma_t(f.s1B, Pe[0], h);
        if (f.six) dh += fma_t(f.s1B, Pe[f.ss2], f.s2B * Pe[2 * f.ss2]);
    }
    const T iL = recip(L);
    if (f.six) {
        const T R = fma_t(lxy, fma_t(f.c4yx, q[0], f.c4xy * r[0]), r[11] + q[11]);
        h = fma_t(h, fma_t(R, iL, (T)1), dh);
    }
    return f.pref * fma_t(h, iL, -(beta * recip(r[1] + q[1])));
}

template <typename T>
__device__ __forceinline__ FinalConst<T> final_const(const FinalArgs &a, int kB)
{
    const Geo &g = a.geo;
    FinalConst<T> f;
    f.c2xy = (T)g.c2[0][1];
    f.c4xy = (T)g.c4[0][1];
    f.c4yx = (T)g.c4[1][0];
    f.pref = (T)g.pref;
    f.six = a.order == 6;
    f.d3 = g.d == 3;
    f.lamB = f.s1B = f.s2B = (T)0;
    f.ss2 = 0;
    if (f.d3) {
        f.lamB = (T)a.tab[2].lam[kB - 1];
        f.s1B = (T)a.tab[2].s[kB - 1];
        f.s2B = (T)a.tab[2].s[g.M[2] - 1 + kB - 1];
        f.ss2 = shell_size(g, 2);
    }
    return f;
}

template <typename T, int MAXE, int KD, int WC, int NTT>
__global__ __launch_bounds__(NTT) void k_final(FinalArgs a, int ntiles)
{
    constexpr bool BIG = NTT != NT;
    // FP64 tiles of a compile-time width (short transforms): persistent blocks
    // that fetch the next tile into registers while the current one is processed
    // (for FP32 tiles one tile per block measured faster)
    constexpr bool PF = WC > 0 && !BIG && sizeof(T) == 8;
    extern __shared__ __align__(16) unsigned char smem[];
    // WC > 0: tile width known at compile time (row offsets become shifts)
    const FftDesc &fd = a.fd;
    const int N = fd.N, M = fd.M, W = WC > 0 ? WC : a.W, rs = BIG ? W : W + 1;
    const int lgW = WC > 0 ? __builtin_ctz(WC > 0 ? WC : 1) : 31 - __clz(W), lgs = lgW - 1;
    const cx<T> *tw = tw_table<T, BIG>(smem, a.tw, a.twf);
    const size_t twb = BIG ? 0 : (size_t)N * sizeof(cx<T>);
    T *buf = reinterpret_cast<T *>(smem + twb);
    const int ncb = (a.ncols + W - 1) / W;
    const int grid = gridDim.x;
    const int lb0 = xcd_remap(blockIdx.x, grid);
    const bool rcont = a.irs == 1 && a.ics != 1;
    if (!BIG) load_twiddles<T, NTT>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    T pf[PF ? MAXE : 1];
    if constexpr (PF) {
        if (lb0 < ntiles) {
            int cb, bt;
            final_tile(a, ncb, lb0, cb, bt);
            const int c0 = cb * W;
            fetch_pair<T, NTT, (PF ? WC : 2), MAXE, false>(pf, static_cast<const T *>(a.buf) + bt * a.ibs + c0 * a.ics,
                                                          a.nrows_in, a.irs, a.ics, 0, min(W, a.ncols - c0), 0, 0,
                                                          threadIdx.x);
        }
    }
    for (int it = lb0; it < ntiles; it += grid) {
    int tid = threadIdx.x;
    if constexpr (PF) {
        asm volatile("" : "+v"(tid));
        tid &= NTT - 1;
    }
    int cb, bt;
    final_tile(a, ncb, it, cb, bt);
    const int c0 = cb * W;
    const int nc = min(W, a.ncols - c0);
    T *g = static_cast<T *>(a.buf) + bt * a.ibs + c0 * a.ics;
    zero_rows<T, NTT>(buf, rs, lgW, 0, 1, tid);
    zero_rows<T, NTT>(buf, rs, lgW, 1 + a.nrows_in, N, tid);
    if constexpr (PF) {
        put_pair<T, T, NTT, (PF ? WC : 2), MAXE>(buf, rs, 1, pf, a.nrows_in, rcont, tid);
        const int nx = it + grid;
        if (nx < ntiles) {
            int cb1, bt1;
            final_tile(a, ncb, nx, cb1, bt1);
            const int c1 = cb1 * W;
            fetch_pair<T, NTT, (PF ? WC : 2), MAXE, false>(pf, static_cast<const T *>(a.buf) + bt1 * a.ibs + c1 * a.ics,
                                                          a.nrows_in, a.irs, a.ics, 0, min(W, a.ncols - c1), 0, 0,
                                                          tid);
        }
    } else {
        tile_load<T, T, NTT>(buf, rs, 1, g, a.nrows_in, nc, a.irs, a.ics, lgW, tid);
    }
    const Geo &geo = a.geo;
    const int d = geo.d;
    const bool six = a.order == 6;
    const int nt = six ? 3 : 1;
    // Staged per row kx and per column ky (12 doubles each):
    //   [0] lambda  [1] q (rows: + q_z)  [2] sin(pi k/M)  [3] sin(2 pi k/M)
    //   [4..9] packed shell values of the family whose other index is fixed
    //          along the row/column, parity 0 then 1, three kinds each
    //   [10] lambda + c2[.][2] lambda lambda_z   (part of Lambda)
    //   [11] c4[.][2] lambda^2 lambda_z + c4[2][.] lambda lambda_z^2   (part of m_R)
    // so that per element Lambda = r10 + c10 + lambda_z + c2[0][1] lx ly and
    // m_R = r11 + c11 + lx ly (c4[0][1] lx + c4[1][0] ly).
    constexpr int SV = 12;
    // The row invariants come from the per-solve table in global memory
    // (written by k_pack); the column invariants are staged in LDS after
    // the tile, 16-byte aligned and addressed from smem, so that every access
    // to them is an LDS instruction (a pointer that may point to either space
    // would make every access a flat one). Staged values and the per-element
    // combination are in the transform type (FP32 in the mixed modes).
    const size_t soff = (twb + (size_t)N * rs * sizeof(T) + 15) & ~(size_t)15;
    const T *__restrict__ rv = static_cast<const T *>(a.rowtab) + (int64_t)bt * (M - 1) * SV;
    T *cv = reinterpret_cast<T *>(smem + soff);
    const int I0 = geo.M[0] - 1;
    const int kB = bt + 1;
    for (int i = tid; i < nc; i += NTT) final_col(a, c0 + i, kB, cv + i * SV);
    __syncthreads();
    // forward transform of the zero-padded rows 1..M0-1 (unless B already holds the spectrum)
    if (!a.pre) fft_tile<T, MAXE, NTT, KD, false>(buf, rs, lgs, fd, tw, false, tid);
    // One sweep over the row pairs (k, N-k) of every complex sequence s
    // (real columns 2s and 2s+1):
    //   sine coefficients  S_a = (z(N-k).y - z(k).y)/2,  S_b = (z(k).x - z(N-k).x)/2
    //   (raw DST of rho along axis 0 at kx = k; the cosine part is not needed),
    //   spectral combination of each column into its coefficient c(k),
    //   and the hermitian input of the inverse sine transform:
    //   z(k) = (c_b, -c_a), z(N-k) = (-c_b, c_a), rows 0 and M zero.
    // Each thread owns both rows of its pair, so no barrier is needed between
    // the reads and the writes.
    const FinalConst<T> f = final_const<T>(a, kB);
    const int nseq = 1 << lgs;
    // Row k per thread (consecutive k across the lanes): the row invariants
    // are read once and serve every column of the tile; the family-2 values
    // come from the transposed copy [par][t][k1][k0], contiguous in k0 = kx.
    const T *Pt = f.d3 ? static_cast<const T *>(a.sh.P2T) + ((kB & 1) ? 3 * f.ss2 : 0) : nullptr;
    // Fewer than NTT / 2 rows would leave threads over: 2^lgG groups of M - 1
    // threads then share the sequences of a row (33^3 FP64 solve 226 -> 209 us,
    // 65^3 261 -> 250 us: this loop is a chain of FP64 operations per column).
    int lgG = 0;
    while (lgG < lgs && ((M - 1) << (lgG + 1)) <= NTT) ++lgG;
    const int kstep = lgG > 0 ? M - 1 : NTT, grp = lgG > 0 ? tid / kstep : 0;
    const int sq0 = grp << (lgs - lgG), sq1 = sq0 + (nseq >> lgG);
    for (int z = tid; z < 2 * nseq; z += NTT) lds_cs(buf, rs, (z & 1) ? M : 0, z >> 1, cx<T>{(T)0, (T)0});
    for (int k = 1 + tid - grp * kstep; k < M && grp < (1 << lgG); k += kstep) {
        T r[SV];
        load12(rv + (k - 1) * SV, r);
        const int kx = k;
        const bool kodd = (kx & 1) != 0; // family 0 at (ky, kz): parity of kx
        for (int sq = sq0; sq < sq1; ++sq) {
            const cx<T> z1 = lds_c(buf, rs, k, sq), z2 = lds_c(buf, rs, N - k, sq);
            T cab[2];
            // the spectrum as loaded (pre), or from the forward transform
            const T beta2[2] = {a.pre ? z1.x : (T)0.5 * (z2.y - z1.y), a.pre ? z1.y : (T)0.5 * (z1.x - z2.x)};
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const int c = 2 * sq + h2;
                T cval = (T)0;
                if (c < nc) {
                    const int ky = 1 + c0 + c; // c0 is even: ky is odd for h2 = 0
                    T q1[SV];
                    load12(cv + c * SV, q1);
                    const T *Pe = f.d3 ? Pt + (int64_t)(ky - 1) * I0 + (kx - 1) : nullptr;
                    cval = final_value(f, r, q1, kodd, h2 == 0, Pe, beta2[h2]);
                }
                cab[h2] = cval;
            }
            lds_cs(buf, rs, k, sq, cx<T>{cab[1], -cab[0]});
            lds_cs(buf, rs, N - k, sq, cx<T>{-cab[1], cab[0]});
        }
    }
    __syncthreads();
    fft_tile<T, MAXE, NTT, KD, false>(buf, rs, lgs, fd, tw, true, tid);
    tile_store<T, T, NTT>(buf, rs, 1, g, a.nrows_in, nc, a.irs, a.ics, (T)0.5, lgW, tid);
    if constexpr (!PF) break; // one tile per block: no loop for the compiler to hoist out of
    __syncthreads();          // the next tile reuses the LDS
    }
}

// The value of lane i of the NL lanes (1, 2 or 4) a lane belongs to.
template <int NL, int I>
__device__ __forceinline__ float quad_get(float v)
{
    constexpr int ctrl = NL == 4 ? I * 0x55 : I ? 0xF5 : 0xA0;
    if constexpr (NL == 1) return v;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xF, 0xF, true));
}

template <int NL, int I>
__device__ __forceinline__ double quad_get(double v)
{
    constexpr int ctrl = NL == 4 ? I * 0x55 : I ? 0xF5 : 0xA0;
    if constexpr (NL == 1) return v;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// The final pass in register tiles (full tiles of the power-of-two lengths): the first
// forward and the last inverse stage read and write B directly, and the spectral
// combination works on the registers between the last forward and the first inverse
// stage (see RegTile): thread (j, s) combines rows k = j + r N/8, r < 4, of its two columns;
// its inverse inputs are these and its mirror's. 8 instead of 12 passes over the tile in
// LDS, six barriers less. Its row records are read a part per lane (whole records per lane:
// 117 us) and its columns in pairs. Bound by VALU issue (FP32 75% busy) and the latency of
// B and the shell spectra. 257^3: FP32 102 -> 97 us, FP64 191 -> 178; 513^3 FP32 1243 -> 847.
template <typename T, typename R>
__global__ __launch_bounds__(R::NTH) void k_final_rt(FinalArgs a, int ntiles)
{
    constexpr int N = R::N, M = N / 2, W = R::W, SV = 12, P = R::P, NL = R::NSEQ < 4 ? R::NSEQ : 4;
    extern __shared__ __align__(16) unsigned char smem[];
    const cx<T> *tw = tw_table<T, !R::LTW>(smem, a.tw, a.twf);
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem) + (R::LTW ? N : 0);
    T *cv = reinterpret_cast<T *>(buf + R::ELEMS);
    const int tid = threadIdx.x;
    const int ncb = (a.ncols + W - 1) / W;
    int cb, bt;
    final_tile(a, ncb, xcd_remap(blockIdx.x, ntiles), cb, bt);
    const int c0 = cb * W, nc = min(W, a.ncols - c0);
    T *g = static_cast<T *>(a.buf) + bt * a.ibs + c0 * a.ics;
    if constexpr (R::LTW) load_twiddles<T, R::NTH>(reinterpret_cast<cx<T> *>(smem), a.tw, N);
    const int kB = bt + 1;
    for (int i = tid; i < nc; i += R::NTH) final_col(a, c0 + i, kB, cv + i * SV);
    __syncthreads();
    cx<T> v[8];
    int j, s;
    const int c = 2 * (tid & (R::NSEQ - 1));
    T x[8];
    auto load = [&]() {
        const int cc = 2 * s;
        rt_fetch<T, R>(x, g, a.irs, cc < nc ? cc * (int)a.ics : -1, cc + 1 < nc ? (cc + 1) * (int)a.ics : -1,
                       nc == W && a.ics == 1, j, 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = cx<T>{x[2 * r], x[2 * r + 1]};
    };
    if (!a.pre) {
        rt_plain<R>(tid, j, s);
        load();
        rt_first_zpad<T, R>(buf, v, j, s);
        rt_middle<T, R, false>(buf, tw, tid);
        rt_paired<R>(tid, j, s);
        rt_last<T, R, false>(buf, tw, v, j, s);
    } else {
        // B holds the spectrum
        rt_paired<R>(tid, j, s);
        load();
    }
    {
        cx<T> z2[4];
        if (!a.pre) {
            rt_reflect<T, R>(v, j, z2);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = cx<T>{(T)0.5 * (z2[r].y - v[r].y), (T)0.5 * (v[r].x - z2[r].x)};
        }
    }
    // v[r]: the raw sine coefficients of columns 2s and 2s + 1 at kx = k
    const FinalConst<T> f = final_const<T>(a, kB);
    const int I0 = M - 1;
    const T *Pt = f.d3 ? static_cast<const T *>(a.sh.P2T) + ((kB & 1) ? 3 * f.ss2 : 0) : nullptr;
    const T *__restrict__ rv = static_cast<const T *>(a.rowtab) + (int64_t)bt * (M - 1) * SV;
    const bool kodd = (j & 1) != 0; // parity of every k of the thread
    auto combine = [&](int k, cx<T> beta) -> cx<T> {
        if (k == 0) return cx<T>{(T)0, (T)0};
        // the NL neighbouring lanes that hold this row read a part of its record
        // each and pass it on (whole records per lane: NL times the L1 traffic)
        T rr[SV], part[SV / NL];
#pragma unroll
        for (int i = 0; i < SV / NL; ++i) part[i] = rv[(k - 1) * SV + (tid & (NL - 1)) * (SV / NL) + i];
#pragma unroll
        for (int i = 0; i < SV / NL; ++i) {
            rr[i] = quad_get<NL, 0>(part[i]);
            if constexpr (NL >= 2) rr[SV / NL + i] = quad_get<NL, 1>(part[i]);
            if constexpr (NL == 4) {
                rr[2 * (SV / NL) + i] = quad_get<NL, 2>(part[i]);
                rr[3 * (SV / NL) + i] = quad_get<NL, 3>(part[i]);
            }
        }
        T out[2];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const int c = 2 * s + h2; // ky = 1 + c0 + c; c0 is even: odd for h2 = 0
            out[h2] = (T)0;
            if (c < nc) {
                T q1[SV];
                load12(cv + c * SV, q1);
                const T *Pe = f.d3 ? Pt + (int64_t)(c0 + c) * I0 + (k - 1) : nullptr;
                out[h2] = final_value(f, rr, q1, kodd, h2 == 0, Pe, h2 ? beta.y : beta.x);
            }
        }
        return cx<T>{out[0], out[1]};
    };
    const cx<T> cab[4] = {combine(j, v[0]), combine(j + P, v[1]), combine(j + 2 * P, v[2]), combine(j + 3 * P, v[3])};
    // hermitian input: z(k) = (c_b, -c_a), z(N - k) = (-c_b, c_a), rows 0 and M zero
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = cx<T>{cab[r].y, -cab[r].x};
    rt_unfold_odd<T, R>(v, j);
    __syncthreads(); // every wave has read the forward transform
    rt_first<T, R, true>(buf, v, j, s);
    rt_middle<T, R, true>(buf, tw, tid);
    rt_plain<R>(tid, j, s);
    rt_last<T, R, true>(buf, tw, v, j, s);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = j + r * P;
        if (t < 1 || t > a.nrows_in) continue;
        T *p = g + toff(t - 1, a.irs, c, a.ics);
        const T y0 = (T)0.5 * v[r].x, y1 = (T)0.5 * v[r].y;
        if (nc == W && a.ics == 1) {
            *reinterpret_cast<pair_t<T> *>(p) = pair_t<T>{y0, y1};
        } else {
            if (c < nc) p[0] = y0;
            if (c + 1 < nc) p[a.ics] = y1;
        }
    }
}

template <typename T, int MAXE, int KD, int WC, int NTT = NT>
static void launch_final_w(const FinalArgs &a, int nblk, size_t lds, hipStream_t st)
{
    const void *fn = (const void *)&k_final<T, MAXE, KD, WC, NTT>;
    set_lds(fn, lds);
    int grid = nblk;
    if (WC > 0 && NTT == NT && sizeof(T) == 8) { // persistent blocks (PF in k_final)
        const int r = resident_blocks(fn, NTT, lds);
        if (r > 0 && r < nblk) grid = r;
    }
    hipLaunchKernelGGL((k_final<T, MAXE, KD, WC, NTT>), dim3(grid), dim3(NTT), lds, st, a, nblk);
}

template <typename T, typename R>
static void launch_final_rt(const FinalArgs &a, int nblk, hipStream_t st)
{
    const size_t lds = rt_lds<T, R>() + (size_t)R::W * 12 * sizeof(T);
    set_lds((const void *)&k_final_rt<T, R>, lds);
    hipLaunchKernelGGL((k_final_rt<T, R>), dim3(nblk), dim3(R::NTH), lds, st, a, nblk);
}

template <typename T, int MAXE, int KD>
static void launch_final_k(const FinalArgs &a, int nblk, hipStream_t st)
{
    // tile + staged column (W) invariants, 12 values of type T each (the row
    // invariants are in the global row table)
    const size_t lds = tile_lds<T>(a.fd.N, a.W) + 16 + (size_t)a.W * 12 * sizeof(T);
    // compile-time widths also prefetch the next tile: MAXE registers per
    // thread must cover the tile's rows
    const bool rc = a.irs == 1 && a.ics != 1;
    // (8 and 16 columns of more than 4 NT elements, powers of two: register tiles)
    if constexpr (KD != kPow2 || MAXE != 8) {
        if (a.W == 8 && PairMap<NT, 8, MAXE>::covers(a.nrows_in, rc))
            return launch_final_w<T, MAXE, KD, 8>(a, nblk, lds, st);
        if (a.W == 16 && PairMap<NT, 16, MAXE>::covers(a.nrows_in, rc))
            return launch_final_w<T, MAXE, KD, 16>(a, nblk, lds, st);
    }
    if (a.W == 32 && PairMap<NT, 32, MAXE>::covers(a.nrows_in, rc))
        launch_final_w<T, MAXE, KD, 32>(a, nblk, lds, st);
    else
        launch_final_w<T, MAXE, KD, 0>(a, nblk, lds, st);
}

template <typename T>
static void launch_final_t(const FinalArgs &a, int nblk, int work, hipStream_t st)
{
    // full tiles of the power-of-two lengths (narrowed tiles of small grids keep the
    // generic stages)
    if (rt_tile<0>(a.fd.N, a.W, [&](auto tile) { launch_final_rt<T, decltype(tile)>(a, nblk, st); })) return;
    if (big_fft(a.fd.N)) {
        // tile + staged columns only (the rows come from the global table)
        const size_t lds = tile_lds<T>(a.fd.N, a.W) + 16 + (size_t)a.W * 12 * sizeof(T);
        if (work <= 4 * NTB)
            launch_final_w<T, 4, kAnyLen, 2, NTB>(a, nblk, lds, st);
        else
            launch_final_w<T, 8, kAnyLen, 2, NTB>(a, nblk, lds, st);
        return;
    }
    by_kind(a.fd.N, [&](auto kd) {
        constexpr int KD = decltype(kd)::value;
        if (work <= 4 * NT)
            launch_final_k<T, 4, KD>(a, nblk, st);
        else
            launch_final_k<T, 8, KD>(a, nblk, st);
    });
}

hipError_t launch_final(const FinalArgs &a, hipStream_t st)
{
    const int ncb = (a.ncols + a.W - 1) / a.W;
    const int nblk = ncb * a.nbatch;
    const int work = (a.W / 2) * a.fd.N;
    if (!a.rowtab) return hipErrorInvalidValue; // the row invariants are read from it
    if (big_fft(a.fd.N) && (a.geo.d != 2 || a.W != 2 || work > 8 * NTB))
        return hipErrorInvalidValue;
    if (!big_fft(a.fd.N) && work > 8 * NT) return hipErrorInvalidValue;
    if (!tile_strides_ok(a.nrows_in, a.irs, a.ncols, a.ics)) return hipErrorInvalidValue;
    if (a.mixed)
        launch_final_t<float>(a, nblk, work, st);
    else
        launch_final_t<double>(a, nblk, work, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Kernel samples for the boundary convolutions: for faces normal to axis a,
// K[dd][ib][ic] = G(sqrt(((dd+1) h_a)^2 + (ib h_b)^2 + (ic h_c)^2)),
// dd = 0..M_a-2, ib = 0..M_b, ic = 0..M_c  (2D: K[dd][ib]).
// ---------------------------------------------------------------------------
__global__ void k_ksample(double *out, int d, int a, int b, int c, int Ma, int Mb, int Mc,
                          double ha, double hb, double hc)
{
    const int64_t nb = Mb + 1, ncn = d == 3 ? Mc + 1 : 1;
    const int64_t tot = (int64_t)(Ma - 1) * nb * ncn;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int ic = (int)(e % ncn);
        const int ib = (int)((e / ncn) % nb);
        const int dd = (int)(e / (ncn * nb));
        const double x = (dd + 1) * ha, y = ib * hb, z = ic * hc;
        const double r = sqrt(x * x + y * y + (d == 3 ? z * z : 0.0));
        double G;
        if (d == 3)
            G = -1.0 / (4.0 * M_PI * r);
        else
            G = log(r) / (2.0 * M_PI);
        out[e] = G;
    }
}

hipError_t launch_ksample(double *out, int d, int a, int b, int c, const int *M, const double *h,
                          hipStream_t st)
{
    const int64_t tot = (int64_t)(M[a] - 1) * (M[b] + 1) * (d == 3 ? M[c] + 1 : 1);
    const int nb = (int)std::min<int64_t>((tot + NT - 1) / NT, 65536);
    hipLaunchKernelGGL(k_ksample, dim3(nb), dim3(NT), 0, st, out, d, a, b, c, M[a], M[b],
                       d == 3 ? M[c] : 0, h[a], h[b], d == 3 ? h[c] : 0.0);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 1D: phi* by one sine-transform pencil, end values by direct sums of
// G(r) = r/2, phi_H linear between them.
// ---------------------------------------------------------------------------
// screen != 0: the end values come from the screening charge instead: with the
// sine coefficients alpha_k of phi*, sigma_lo = -sum (pi k/L) alpha_k and
// sigma_hi = sum (pi k/L)(-1)^k alpha_k are the outward derivatives at the two
// ends and g(x) = sum over both ends of G(|x - end|) sigma, i.e.
// g_0 = (L/2) sigma_hi and g_M = (L/2) sigma_lo (G = r/2 vanishes at r = 0).
template <int MAXE, int KD, int NTT>
__global__ __launch_bounds__(NTT) void k_1d(const double *rho, double *phi, int M, double h,
                                            FftDesc fd, const cx<double> *twg, AxisTabs tab, int screen)
{
    constexpr bool BIG = NTT != NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = fd.N, rs = BIG ? 2 : 3, lgW = 1;
    const cx<double> *tw = BIG ? twg : reinterpret_cast<const cx<double> *>(smem);
    double *buf = reinterpret_cast<double *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<double>)));
    __shared__ double red[2][NTT];
    if (!BIG) load_twiddles<double, NTT>(reinterpret_cast<cx<double> *>(smem), twg, N);
    // end values
    double s0 = 0.0, s1 = 0.0;
    for (int j = 1 + threadIdx.x; j < M; j += NTT) {
        s0 += (0.5 * j * h) * rho[j];
        s1 += (0.5 * (M - j) * h) * rho[j];
    }
    red[0][threadIdx.x] = s0;
    red[1][threadIdx.x] = s1;
    zero_rows<double, NTT>(buf, rs, lgW, 0, 1);
    zero_rows<double, NTT>(buf, rs, lgW, M, N);
    tile_load<double, double, NTT>(buf, rs, 1, rho + 1, M - 1, 1, 1, 1, lgW);
    __syncthreads();
    for (int w = NTT / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            red[0][threadIdx.x] += red[0][threadIdx.x + w];
            red[1][threadIdx.x] += red[1][threadIdx.x + w];
        }
        __syncthreads();
    }
    double g0 = h * red[0][0], g1 = h * red[1][0];
    fft_tile<double, MAXE, NTT, KD, false>(buf, rs, 0, fd, tw, false);
    post_cs<double, MAXE, NTT>(buf, rs, 0, M);
    __syncthreads();
    double slo = 0.0, shi = 0.0;
    const double L = M * h, piL = 3.14159265358979323846264338327950288 / L;
    for (int k = 1 + threadIdx.x; k < M; k += NTT) {
        const double al = -(2.0 / M) * buf[(M + k) * rs] / tab.q[k - 1];
        buf[(M + k) * rs] = al;
        const double t = (k * piL) * al;
        slo -= t;
        shi += (k & 1) ? -t : t;
    }
    if (screen) {
        red[0][threadIdx.x] = slo;
        red[1][threadIdx.x] = shi;
        __syncthreads();
        for (int w = NTT / 2; w > 0; w >>= 1) {
            if (threadIdx.x < w) {
                red[0][threadIdx.x] += red[0][threadIdx.x + w];
                red[1][threadIdx.x] += red[1][threadIdx.x + w];
            }
            __syncthreads();
        }
        g0 = 0.5 * L * red[1][0];
        g1 = 0.5 * L * red[0][0];
    }
    __syncthreads();
    pre_herm<double, MAXE, NTT>(buf, rs, 0, M, true);
    fft_tile<double, MAXE, NTT, KD, false>(buf, rs, 0, fd, tw, true);
    for (int j = threadIdx.x; j <= M; j += NTT) {
        double v;
        if (j == 0)
            v = g0;
        else if (j == M)
            v = g1;
        else
            v = 0.5 * buf[j * rs] + g0 + (g1 - g0) * ((double)j / M);
        phi[j] = v;
    }
}

hipError_t launch_1d(const double *rho, double *phi, int M, double h, const FftDesc &fd,
                     const cx<double> *tw, const AxisTabs &tab, int screen, hipStream_t st)
{
    const size_t lds = tile_lds<double>(fd.N, 2);
    auto go = [&](auto maxe, auto ntt) {
        constexpr int MAXE = decltype(maxe)::value, NTT = decltype(ntt)::value;
        by_kind(fd.N, [&](auto kd) {
            constexpr int KD = decltype(kd)::value;
            set_lds((const void *)&k_1d<MAXE, KD, NTT>, lds);
            hipLaunchKernelGGL((k_1d<MAXE, KD, NTT>), dim3(1), dim3(NTT), lds, st, rho, phi, M, h, fd, tw, tab, screen);
        });
        return hipGetLastError();
    };
    return by_length(fd.N, go);
}

} // namespace ips
