// HIP kernels of the adjoint map rho_bar = A^T phi_bar (gfx950, FP64).
//
// The forward solve is linear, phi = A rho; each of its steps is transposed
// here in reverse order:
//   phi_I = phi_star_I + u_I,  phi_boundary = g,  g = B rho  (Sections 2, 4)
//   u_I   = L0^-1 (T g)                                        (order 4)
//   u_I   = L0^-1 (T g + E R_core(u1, g)),  u1_I = L0^-1 T g   (order 6)
// with T the transfer of boundary values to the right-hand side (eq.
// harmonic4thOrderNH2D), R_core the sixth-order stencils on the core and E
// the cubic extrapolation next to the boundary (eqs. 6thOrderRelation2D/3D).
// The phi_star map and L0^-1 are symmetric.  Writing w = phi_bar:
//   a      = L0^-1 w_I
//   f      = E^T a                    (core nodes; order 6)
//   U      = S f, S = sum_{x != y} c4[x][y] D2_x D2_x D2_y on every node
//   b      = L0^-1 U_I                (order 6)
//   lambda = w_boundary + T^T (a + b) + U_boundary
//   rho_bar_I = phi_star(w_I) + B^T lambda,  rho_bar_boundary = 0
// FP64 plans evaluate this on the shell, as the forward solve does (launch_adj_*
// below: volume transforms of w alone); the mixed modes by whole-volume transforms
// and stencils (their FP32 tiles' rounding is kept).
// B^T spreads boundary values back over the interior with the same Green's
// function sums, evaluated by FFT convolutions with the plan's kernel
// spectra: for every slice s normal to a face family,
//   slice(s) = IFFT2[ K_hat(s - 1) . FFT2(lambda_face0)
//                     + K_hat(M - 1 - s) . FFT2(lambda_faceM) ].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ips {

constexpr int NTA = 256;

__device__ __forceinline__ int64_t grid_off(const int64_t *n, int d, const int *i)
{
    int64_t o = 0;
    for (int a = 0; a < d; ++a) o = o * n[a] + i[a];
    return o;
}

// Lambda(k) of L0 and the continuous eigenvalue sum q(k) for one mode.
template <int D>
__device__ __forceinline__ void mode_symbols(const AdjArgs &a, const int *k, double &L, double &q)
{
    double lam[3];
    L = 0.0;
    q = 0.0;
#pragma unroll
    for (int x = 0; x < D; ++x) {
        lam[x] = a.tab[x].lam[k[x] - 1];
        L += lam[x];
        q += a.tab[x].q[k[x] - 1];
    }
#pragma unroll
    for (int x = 0; x < D; ++x)
#pragma unroll
        for (int y = x + 1; y < D; ++y) L += a.geo.c2[x][y] * lam[x] * lam[y];
}

// X holds raw sine coefficients over the interior modes ([k0][k1][k2], last
// fastest).  Y (if given) <- -pref X / q  (the phi_star map);  X <- pref X / Lambda.
// A wave per 256 elements of a row of the last axis: contiguous, no index divisions
// per element, four loads in flight (257^3, 267 MB: 89 -> 73 us; a position of the last
// axes per thread, walking along the first: 92).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_spec(AdjArgs a, double *X, double *Y)
{
    constexpr int U = 4;
    const Geo &g = a.geo;
    const int I1 = g.M[D - 2] - 1, n = g.M[D - 1] - 1, lane = threadIdx.x & 63;
    const uint32_t row = __builtin_amdgcn_readfirstlane(blockIdx.x * (NTA / 64) + (threadIdx.x >> 6));
    int k[3] = {1 + (int)row, 0, 0};
    if (D == 3) {
        k[0] = 1 + (int)(row / (uint32_t)I1);
        k[1] = 1 + (int)(row % (uint32_t)I1);
    }
    if (k[0] >= g.M[0]) return;
    double *Xr = X + (int64_t)row * n, *Yr = Y ? Y + (int64_t)row * n : nullptr;
    const int i = blockIdx.y * 64 * U + lane;
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = Xr[min(i + 64 * u, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = i + 64 * u;
        if (c >= n) break;
        double L, q;
        k[D - 1] = 1 + c;
        mode_symbols<D>(a, k, L, q);
        if (Yr) Yr[c] = -g.pref * v[u] / q;
        Xr[c] = g.pref * v[u] / L;
    }
}

hipError_t launch_adj_spec(const AdjArgs &a, double *X, double *Y, hipStream_t st)
{
    int64_t rows = 1;
    for (int x = 0; x + 1 < a.geo.d; ++x) rows *= a.geo.M[x] - 1;
    const dim3 grid((unsigned)((rows + NTA / 64 - 1) / (NTA / 64)), (unsigned)((a.geo.M[a.geo.d - 1] + 254) / 256));
    if (a.geo.d == 3)
        hipLaunchKernelGGL(k_adj_spec<3>, grid, dim3(NTA), 0, st, a, X, Y);
    else
        hipLaunchKernelGGL(k_adj_spec<2>, grid, dim3(NTA), 0, st, a, X, Y);
    return hipGetLastError();
}

// f = E^T a on the core (all indices in [2, M-2]), 0 on every other node of
// the grid-shaped array F.  E is the tensor product of one-axis maps
//   e(i, p) = [i == p] for i in [2, M-2],
//   e(1, p) = (4, -6, 4, -1)[p - 2]        for p in 2..5,
//   e(M-1, p) = (4, -6, 4, -1)[M - 2 - p]  for p in M-5..M-2,
// so E^T a at p sums a at (p or 1 or M-1 per axis) with the product weights.
// a is packed over the interior ([i0-1][i1-1][i2-1]).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_etrans(AdjArgs a, const double *A, double *F)
{
    const Geo &g = a.geo;
    int64_t tot = 1;
    for (int x = 0; x < D; ++x) tot *= a.n[x];
    const double wt[4] = {4.0, -6.0, 4.0, -1.0};
    for (int64_t e = blockIdx.x * (int64_t)NTA + threadIdx.x; e < tot; e += (int64_t)gridDim.x * NTA) {
        int i[3] = {0, 0, 0};
        int64_t r = e;
#pragma unroll
        for (int x = D - 1; x >= 0; --x) {
            i[x] = (int)(r % a.n[x]);
            r /= a.n[x];
        }
        bool core = true;
#pragma unroll
        for (int x = 0; x < D; ++x) core = core && i[x] >= 2 && i[x] <= g.M[x] - 2;
        double v = 0.0;
        if (core) {
            // per axis: up to three (source index, weight) options
            int src[3][3];
            double w[3][3];
            int cnt[3] = {1, 1, 1};
#pragma unroll
            for (int x = 0; x < D; ++x) {
                const int M = g.M[x], p = i[x];
                src[x][0] = p;
                w[x][0] = 1.0;
                if (p <= 5) {
                    src[x][cnt[x]] = 1;
                    w[x][cnt[x]] = wt[p - 2];
                    ++cnt[x];
                }
                if (p >= M - 5) {
                    src[x][cnt[x]] = M - 1;
                    w[x][cnt[x]] = wt[M - 2 - p];
                    ++cnt[x];
                }
            }
            const int c1 = D >= 2 ? cnt[1] : 1, c2 = D == 3 ? cnt[2] : 1;
            for (int t0 = 0; t0 < cnt[0]; ++t0)
                for (int t1 = 0; t1 < c1; ++t1)
                    for (int t2 = 0; t2 < c2; ++t2) {
                        int64_t o = src[0][t0] - 1;
                        double ww = w[0][t0];
                        if (D >= 2) {
                            o = o * (g.M[1] - 1) + (src[1][t1] - 1);
                            ww *= w[1][t1];
                        }
                        if (D == 3) {
                            o = o * (g.M[2] - 1) + (src[2][t2] - 1);
                            ww *= w[2][t2];
                        }
                        v += ww * A[o];
                    }
        }
        F[e] = v;
    }
}

// U = sum_{x != y} c4[x][y] D2_x D2_x D2_y F on every grid node, with F = 0
// off the core (the stencil is symmetric, so this is also its transpose).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_sop(AdjArgs a, const double *F, double *U)
{
    const Geo &g = a.geo;
    int64_t tot = 1;
    for (int x = 0; x < D; ++x) tot *= a.n[x];
    const double a4[5] = {1.0, -4.0, 6.0, -4.0, 1.0};
    const double a2[3] = {1.0, -2.0, 1.0};
    for (int64_t e = blockIdx.x * (int64_t)NTA + threadIdx.x; e < tot; e += (int64_t)gridDim.x * NTA) {
        int i[3] = {0, 0, 0};
        int64_t r = e;
#pragma unroll
        for (int x = D - 1; x >= 0; --x) {
            i[x] = (int)(r % a.n[x]);
            r /= a.n[x];
        }
        double v = 0.0;
#pragma unroll
        for (int x = 0; x < D; ++x)
#pragma unroll
            for (int y = 0; y < D; ++y) {
                if (y == x) continue;
                double s = 0.0;
#pragma unroll
                for (int dx = -2; dx <= 2; ++dx)
#pragma unroll
                    for (int dy = -1; dy <= 1; ++dy) {
                        int j[3] = {i[0], i[1], i[2]};
                        j[x] += dx;
                        j[y] += dy;
                        bool core = true;
#pragma unroll
                        for (int z = 0; z < D; ++z) core = core && j[z] >= 2 && j[z] <= g.M[z] - 2;
                        if (core) s += a4[dx + 2] * a2[dy + 1] * F[grid_off(a.n, D, j)];
                    }
                const double hx2 = g.h[x] * g.h[x];
                v += g.c4[x][y] * s / (hx2 * hx2 * g.h[y] * g.h[y]);
            }
        U[e] = v;
    }
}

// 3D: the same sums in separable form, one axis x at a time,
//   T_x = sum_{y != x} c4[x][y] / (h_x^4 h_y^2) D2_y F      (k_adj_d2y)
//   U  += D4_x T_x                                         (k_adj_d4x)
// with F and T_x taken as zero off the grid (F is zero outside the core: the
// extrapolation writes every node), which is the tap set of k_adj_sop.  One
// thread per node; the threads of a block take consecutive nodes of one plane
// of the first axis (grid.y), so every lane is busy whatever the line length.
__global__ __launch_bounds__(NTA) void k_adj_d2y(AdjArgs a, int x, const double *F, double *T)
{
    const Geo &g = a.geo;
    const int n[3] = {(int)a.n[0], (int)a.n[1], (int)a.n[2]};
    const int pl = blockIdx.x * NTA + threadIdx.x;
    if (pl >= n[1] * n[2]) return;
    const int i0 = blockIdx.y, i1 = pl / n[2], i2 = pl - i1 * n[2];
    const int64_t st[3] = {(int64_t)n[1] * n[2], n[2], 1};
    const double hx2 = g.h[x] * g.h[x];
    {
        const int i[3] = {i0, i1, i2};
        const int64_t e = i0 * st[0] + pl;
        double v = 0.0;
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            if (y == x) continue;
            const double fm = i[y] > 0 ? F[e - st[y]] : 0.0;
            const double fp = i[y] < n[y] - 1 ? F[e + st[y]] : 0.0;
            v += g.c4[x][y] / (hx2 * hx2 * g.h[y] * g.h[y]) * (fm - 2.0 * F[e] + fp);
        }
        T[e] = v;
    }
}

__global__ __launch_bounds__(NTA) void k_adj_d4x(AdjArgs a, int x, const double *T, double *U)
{
    const int n[3] = {(int)a.n[0], (int)a.n[1], (int)a.n[2]};
    const int pl = blockIdx.x * NTA + threadIdx.x;
    if (pl >= n[1] * n[2]) return;
    const int i0 = blockIdx.y, i1 = pl / n[2], i2 = pl - i1 * n[2];
    const int64_t st[3] = {(int64_t)n[1] * n[2], n[2], 1};
    const double a4[5] = {1.0, -4.0, 6.0, -4.0, 1.0};
    {
        const int i[3] = {i0, i1, i2};
        const int64_t e = i0 * st[0] + pl;
        double v = 0.0;
#pragma unroll
        for (int dx = -2; dx <= 2; ++dx) {
            const int j = i[x] + dx;
            if (j >= 0 && j < n[x]) v += a4[dx + 2] * T[e + dx * st[x]];
        }
        U[e] = x == 0 ? v : U[e] + v;
    }
}

hipError_t launch_adj_r6(const AdjArgs &a, const double *A, double *F, double *U, double *T, hipStream_t st)
{
    const int nb = 4096;
    if (a.geo.d == 3) {
        hipLaunchKernelGGL(k_adj_etrans<3>, dim3(nb), dim3(NTA), 0, st, a, A, F);
        const dim3 grid((unsigned)((a.n[1] * a.n[2] + NTA - 1) / NTA), (unsigned)a.n[0]);
        for (int x = 0; x < 3; ++x) {
            hipLaunchKernelGGL(k_adj_d2y, grid, dim3(NTA), 0, st, a, x, F, T);
            hipLaunchKernelGGL(k_adj_d4x, grid, dim3(NTA), 0, st, a, x, T, U);
        }
    } else {
        hipLaunchKernelGGL(k_adj_etrans<2>, dim3(nb), dim3(NTA), 0, st, a, A, F);
        hipLaunchKernelGGL(k_adj_sop<2>, dim3(nb), dim3(NTA), 0, st, a, F, U);
    }
    return hipGetLastError();
}

// lambda on the face nodes of every family (faces own their edges and
// corners with precedence axis 0 > axis 1 > axis 2; other entries 0):
//   lambda = w + U - sum over interior neighbours i of the L_h stencil
//            weight times (y1 + y2)(i)
// y1, y2 packed over the interior (y2 and U may be NULL).
// LF[fam][f][j_b][j_c] over (M_b + 1) x (M_c + 1), (b, c) = a.fb[fam], a.fc[fam].
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_lambda(AdjArgs a, const double *w, const double *y1,
                                                    const double *y2, const double *U)
{
    const Geo &g = a.geo;
    int fam = 0;
    int64_t e = blockIdx.x * (int64_t)NTA + threadIdx.x;
    while (fam < D && e >= a.lf_size[fam]) {
        e -= a.lf_size[fam];
        ++fam;
    }
    if (fam >= D) return;
    const int b = a.fb[fam], c = a.fc[fam];
    const int nb = g.M[b] + 1, ncn = D == 3 ? g.M[c] + 1 : 1;
    const int per = nb * ncn;
    const int f = (int)(e / per);
    const int rem = (int)(e % per);
    int i[3] = {0, 0, 0};
    i[fam] = f ? g.M[fam] : 0;
    i[b] = rem / ncn;
    if (D == 3) i[c] = rem % ncn;
    bool owned = true;
    for (int x = 0; x < fam; ++x)
        if (i[x] == 0 || i[x] == g.M[x]) owned = false;
    double lam = 0.0;
    if (owned) {
        const int64_t go = grid_off(a.n, D, i);
        lam = w[go];
        if (U) lam += U[go];
        double s = 0.0;
        // face-neighbour offsets
#pragma unroll
        for (int p = 0; p < D; ++p) {
            double wf = 1.0 / (g.h[p] * g.h[p]);
#pragma unroll
            for (int q = 0; q < D; ++q)
                if (q != p) wf -= 2.0 * g.c2[p][q] / (g.h[p] * g.h[p] * g.h[q] * g.h[q]);
#pragma unroll
            for (int sg = -1; sg <= 1; sg += 2) {
                int j[3] = {i[0], i[1], i[2]};
                j[p] += sg;
                bool in = true;
#pragma unroll
                for (int z = 0; z < D; ++z) in = in && j[z] >= 1 && j[z] <= g.M[z] - 1;
                if (in) {
                    int64_t o = 0;
#pragma unroll
                    for (int z = 0; z < D; ++z) o = o * (g.M[z] - 1) + (j[z] - 1);
                    s += wf * (y1[o] + (y2 ? y2[o] : 0.0));
                }
            }
        }
        // edge-neighbour offsets
#pragma unroll
        for (int p = 0; p < D; ++p)
#pragma unroll
            for (int q = p + 1; q < D; ++q) {
                const double we = g.c2[p][q] / (g.h[p] * g.h[p] * g.h[q] * g.h[q]);
#pragma unroll
                for (int sp = -1; sp <= 1; sp += 2)
#pragma unroll
                    for (int sq = -1; sq <= 1; sq += 2) {
                        int j[3] = {i[0], i[1], i[2]};
                        j[p] += sp;
                        j[q] += sq;
                        bool in = true;
#pragma unroll
                        for (int z = 0; z < D; ++z) in = in && j[z] >= 1 && j[z] <= g.M[z] - 1;
                        if (in) {
                            int64_t o = 0;
#pragma unroll
                            for (int z = 0; z < D; ++z) o = o * (g.M[z] - 1) + (j[z] - 1);
                            s += we * (y1[o] + (y2 ? y2[o] : 0.0));
                        }
                    }
            }
        lam -= s;
    }
    a.LF[fam][e] = lam;
}

hipError_t launch_adj_lambda(const AdjArgs &a, const double *w, const double *y1, const double *y2,
                             const double *U, hipStream_t st)
{
    int64_t tot = 0;
    for (int fam = 0; fam < a.geo.d; ++fam) tot += a.lf_size[fam];
    const unsigned nb = (unsigned)((tot + NTA - 1) / NTA);
    if (a.geo.d == 3)
        hipLaunchKernelGGL(k_adj_lambda<3>, dim3(nb), dim3(NTA), 0, st, a, w, y1, y2, U);
    else
        hipLaunchKernelGGL(k_adj_lambda<2>, dim3(nb), dim3(NTA), 0, st, a, w, y1, y2, U);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The shell form of the adjoint (FP64). With W the raw sine spectrum of w_I and
// gt_hat, D_hat, V as in the forward solve, c(k) = pref [(gt_hat (1 + m_R/Lambda) +
// D_hat)/Lambda - beta/q] transposes to
//   D layers:    D_hat_l(k_o)  = sum over k_a of sin(pi k_a l/M_a) X(k),  X = pref W/Lambda
//   their values by sine sums, the extrapolation and the sixth-order stencils
//   transposed on the layers (R_spec layers, boundary terms Z), back to spectra T,
//   g~ layers:   the same sums over k_a of X (1 + m_R/Lambda) + pref m_R/Lambda V,
//                V(k) = sum over the layers of all families of sin(pi k_f l/M_f) T_l(k_o)
// and lambda collects g~ and Z. Three volume transforms instead of twelve and no
// volume stencils: 257^3 forward and backward 5.03 -> 3.93 ms, 4097^2 5.52 -> 4.29 ms.
// The sums over k_a read X once per family (257^3, three families: 67 us for two layers,
// 96 for four, 12 and 23 to add the splits); k_adj_x (150 to 159 us in the runs measured)
// is bound by its ten cached loads per element.
// ---------------------------------------------------------------------------
struct ContractJob {
    const double *s;      // s[(j-1)*Ia + k-1] = sin(pi k j/M)
    int Ia;
    int64_t np, st;       // positions, stride of k_a
    int64_t inner, outer; // position p starts at (p / inner) * outer + p % inner
    double *out;          // [splits][nl][np]
    int nblk, splits;     // blocks, of which nblk / splits per split
};
struct ContractArgs {
    const double *X;
    ContractJob job[3]; // the last one's axis is contiguous
    int d;
};

// Layer sums from the odd and the even wavenumbers' sums of weights 1 (and 2).
template <int NW>
__device__ __forceinline__ void layer_out(double *out, int64_t np, int64_t p, const double (&o)[NW], const double (&e)[NW])
{
    out[p] = o[0] + e[0];
    out[(2 * NW - 1) * np + p] = o[0] - e[0];
    if constexpr (NW == 2) {
        out[np + p] = o[1] + e[1];
        out[2 * np + p] = o[1] - e[1];
    }
}

// Strided axis: one position per thread, neighbouring positions side by side.
template <int NW>
__device__ __forceinline__ void contract_strided(const ContractJob &a, const double *Xv, int blk)
{
    const int nb = a.nblk / a.splits, sp = blk / nb, ns = a.splits;
    const int64_t p = (int64_t)(blk % nb) * NTA + threadIdx.x;
    if (p >= a.np) return;
    // whole pairs of wavenumbers (odd, even) per split
    const int pairs = (a.Ia + 1) / 2;
    const int i0 = 2 * (int)((int64_t)pairs * sp / ns), i1 = min(a.Ia, 2 * (int)((int64_t)pairs * (sp + 1) / ns));
    const double *X = Xv + p / a.inner * a.outer + p % a.inner;
    double o[NW], e[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) o[w] = e[w] = 0.0;
    int i = i0;
    for (; i + 8 <= i1; i += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = X[(i + u) * a.st];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                double &t = u & 1 ? e[w] : o[w];
                t = fma(a.s[w * a.Ia + i + u], v[u], t);
            }
    }
    for (; i < i1; ++i) {
        const double v = X[i * a.st];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const double t = a.s[w * a.Ia + i] * v;
            o[w] += i & 1 ? 0.0 : t;
            e[w] += i & 1 ? t : 0.0;
        }
    }
    layer_out<NW>(a.out + sp * (2 * NW) * a.np, a.np, p, o, e);
}

// Contiguous axis: one position (row) per wave; lane parity is wavenumber parity.
template <int NW>
__device__ __forceinline__ void contract_rows(const ContractJob &a, const double *Xv, int blk)
{
    const int lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blk * (NTA / 64) + (threadIdx.x >> 6);
    if (p >= a.np) return;
    const double *X = Xv + p * a.outer;
    double t[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) t[w] = 0.0;
    for (int i = lane; i < a.Ia; i += 64) {
        const double v = X[i];
#pragma unroll
        for (int w = 0; w < NW; ++w) t[w] = fma(a.s[w * a.Ia + i], v, t[w]);
    }
    double o[NW], e[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
#pragma unroll
        for (int m = 2; m < 64; m <<= 1) t[w] += __shfl_xor(t[w], m);
        o[w] = t[w];
        e[w] = __shfl_xor(t[w], 1);
    }
    if (lane == 0) layer_out<NW>(a.out, a.np, p, o, e);
}

// The families' sums in one launch: small grids are bound by the number of dependent
// launches (with k_adj_rs_z below: adjoint of 14^2 103 -> 99 us, 33^3 207 -> 191, 257^3
// 2024 -> 2003).
template <int NW>
__global__ __launch_bounds__(NTA) void k_adj_contract(ContractArgs a)
{
    int fam = 0, blk = blockIdx.x;
    while (fam < a.d - 1 && blk >= a.job[fam].nblk) blk -= a.job[fam++].nblk;
    if (fam < a.d - 1)
        contract_strided<NW>(a.job[fam], a.X, blk);
    else
        contract_rows<NW>(a.job[fam], a.X, blk);
}

// Splits of the sums along axis a (1: none).
static int adj_splits(const Geo &g, int a)
{
    if (a == g.d - 1) return 1; // rows
    int64_t np = 1;
    for (int b = 0; b < g.d; ++b)
        if (b != a) np *= g.M[b] - 1;
    const int Ia = g.M[a] - 1;
    const int64_t want = ((int64_t)512 * 1024 + np - 1) / np; // threads of a full device
    // (the partials of two families, up to 4 layers per split, fit one volume)
    return (int)std::max<int64_t>(1, std::min<int64_t>(want, Ia / 16));
}

hipError_t launch_adj_contract(const AdjArgs &a, int nl, const double *X, double *part, double *const *out,
                               hipStream_t st)
{
    const Geo &g = a.geo;
    if (nl != 2 && nl != 4) return hipErrorInvalidValue;
    ContractArgs c{};
    ReduceArgs r{};
    c.X = X;
    c.d = g.d;
    r.nset = 1;
    int64_t tot = 0;
    for (int ax = 0; ax < g.d; ++ax) {
        ContractJob &j = c.job[ax];
        j.s = a.tab[ax].s;
        j.Ia = g.M[ax] - 1;
        j.np = 1;
        j.st = 1;
        for (int b = 0; b < g.d; ++b) {
            if (b != ax) j.np *= g.M[b] - 1;
            if (b > ax) j.st *= g.M[b] - 1;
        }
        j.inner = j.st;
        j.outer = j.st * j.Ia;
        j.splits = adj_splits(g, ax);
        j.out = out[ax];
        if (j.splits > 1) {
            j.out = part;
            r.job[r.njobs++] = {part, out[ax], nl * j.np, j.splits};
            part += j.splits * nl * j.np;
        }
        const int per = ax == g.d - 1 ? NTA / 64 : NTA; // positions per block
        j.nblk = (int)((j.np + per - 1) / per) * j.splits;
        tot += j.nblk;
    }
    if (nl == 2)
        hipLaunchKernelGGL(k_adj_contract<1>, dim3((unsigned)tot), dim3(NTA), 0, st, c);
    else
        hipLaunchKernelGGL(k_adj_contract<2>, dim3((unsigned)tot), dim3(NTA), 0, st, c);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && r.njobs > 0) e = launch_reduce(r, st);
    return e;
}

// ---- transposed extrapolation and stencils on the shell ---------------------------
__device__ __forceinline__ int64_t adj_shell_size(const Geo &g, int a)
{
    int64_t s = 1;
    for (int b = 0; b < g.d; ++b)
        if (b != a) s *= g.M[b] - 1;
    return s;
}

// Position e of family fam -> the indices of the other axes.
template <int D>
__device__ __forceinline__ void shell_pos(const Geo &g, int fam, int e, int *ob, int *i)
{
    int q = 0;
    ob[1] = 0;
#pragma unroll
    for (int b = 0; b < D; ++b)
        if (b != fam) ob[q++] = b;
    if (D == 3) {
        const int Ic = g.M[ob[1]] - 1;
        i[ob[0]] = 1 + e / Ic;
        i[ob[1]] = 1 + e % Ic;
    } else {
        i[ob[0]] = 1 + e;
    }
}

// Index along the family axis of core layer l (2..5, M-5..M-2) and R_spec slot of
// index i (1..5, then M-1..M-5).
__device__ __forceinline__ int core_index(int l, int M) { return l < 4 ? 2 + l : M - 9 + l; }
__device__ __forceinline__ int rs_slot(int i, int M) { return i <= 5 ? i - 1 : 5 + (M - 1 - i); }

// Whether family fam owns the D values at index i of a lower axis.
__device__ __forceinline__ bool d_owned(int i, int M) { return i > 2 && i < M - 2; }

// Cb[fam][l] = transposed cubic extrapolation of the owned D layers: core node p of
// an axis feeds the shell nodes p, 1 (p <= 5) and M-1 (p >= M-5).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_core(AdjArgs a, AdjShell s)
{
    const Geo &g = a.geo;
    const int fam = blockIdx.y >> 3, l = blockIdx.y & 7;
    const int64_t ss = adj_shell_size(g, fam);
    const int e = blockIdx.x * NTA + threadIdx.x;
    if (e >= ss) return;
    int ob[2], i[3] = {0, 0, 0};
    shell_pos<D>(g, fam, e, ob, i);
    const int Mf = g.M[fam];
    i[fam] = core_index(l, Mf);
    bool core = true;
    for (int b = 0; b < D; ++b) core = core && i[b] >= 2 && i[b] <= g.M[b] - 2;
    double v = 0.0;
    if (core) {
        const double wt[4] = {4.0, -6.0, 4.0, -1.0};
        const double *Db = s.Db[fam];
        const double wf = wt[l < 4 ? l : 7 - l];
        const int jx = l < 4 ? 0 : 3, j1 = l == 0 ? 1 : l == 7 ? 2 : -1;
        const int Ic = D == 3 ? g.M[ob[1]] - 1 : 1;
        // sources along each other axis: itself, node 1, node M-1 (weight 0: none)
        int src[2][3];
        double w[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            src[q][0] = src[q][1] = src[q][2] = 1;
            w[q][0] = q < D - 1 ? 0.0 : 1.0;
            w[q][1] = w[q][2] = 0.0;
            if (q >= D - 1) continue;
            const int b = ob[q], M = g.M[b], p = i[b];
            src[q][0] = p;
            src[q][2] = M - 1;
            w[q][0] = b > fam || d_owned(p, M) ? 1.0 : 0.0;
            if (b > fam) { // a lower axis owns its own shell nodes
                w[q][1] = p <= 5 ? wt[p - 2] : 0.0;
                w[q][2] = p >= M - 5 ? wt[M - 2 - p] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int t = 0; t < (D == 3 ? 3 : 1); ++t) {
                const double ww = w[0][u] * w[1][t];
                if (ww == 0.0) continue;
                const int64_t o = D == 3 ? (int64_t)(src[0][u] - 1) * Ic + (src[1][t] - 1) : src[0][u] - 1;
                double d = wf * Db[jx * ss + o];
                if (j1 >= 0) d += Db[j1 * ss + o];
                v += ww * d;
            }
    }
    s.Cb[fam][(int64_t)l * ss + e] = v;
}

// Rb[fam][r] = core layers' part minus the owned D layers (D = R - R_spec).
template <int D>
__device__ __forceinline__ void adj_rs(const AdjArgs &a, const AdjShell &s, int fam, int r)
{
    const Geo &g = a.geo;
    const int64_t ss = adj_shell_size(g, fam);
    const int e = blockIdx.x * NTA + threadIdx.x;
    if (e >= ss) return;
    int ob[2], i[3] = {0, 0, 0};
    shell_pos<D>(g, fam, e, ob, i);
    const int Mf = g.M[fam];
    bool owned = true;
    for (int b = 0; b < fam; ++b) owned = owned && d_owned(i[b], g.M[b]);
    const int L4[4] = {1, 2, Mf - 2, Mf - 1};
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (owned && rs_slot(L4[j], Mf) == r) v -= s.Db[fam][j * ss + e];
#pragma unroll
    for (int l = 0; l < 8; ++l)
        if (rs_slot(core_index(l, Mf), Mf) == r) v += s.Cb[fam][l * ss + e];
    s.Rb[fam][(int64_t)r * ss + e] = v;
}

// Z[x][side]: the transposed core values at the nodes with index 2 (M-2) along x,
// of every family whose core layers hold the node, over h_x^4.
template <int D>
__device__ __forceinline__ void adj_z(const AdjArgs &a, const AdjShell &s, int x, int f)
{
    const Geo &g = a.geo;
    const int64_t ss = adj_shell_size(g, x);
    const int e = blockIdx.x * NTA + threadIdx.x;
    if (e >= ss) return;
    int ob[2], i[3] = {0, 0, 0};
    shell_pos<D>(g, x, e, ob, i);
    i[x] = f ? g.M[x] - 2 : 2;
    bool core = true;
    for (int b = 0; b < D; ++b) core = core && i[b] >= 2 && i[b] <= g.M[b] - 2;
    double v = 0.0;
    if (core) {
#pragma unroll
        for (int fam = 0; fam < D; ++fam) {
            if (i[fam] > 5 && i[fam] < g.M[fam] - 5) continue;
            int64_t o = 0;
#pragma unroll
            for (int b = 0; b < D; ++b)
                if (b != fam) o = o * (g.M[b] - 1) + (i[b] - 1);
            const int64_t sf = adj_shell_size(g, fam);
            for (int l = 0; l < 8; ++l)
                if (core_index(l, g.M[fam]) == i[fam]) v += s.Cb[fam][l * sf + o];
        }
        const double h2 = g.h[x] * g.h[x];
        v /= h2 * h2;
    }
    s.Z[x][(int64_t)f * ss + e] = v;
}

// Both from the core layers: block rows 0 .. 10 D - 1 and 10 D .. 12 D - 1.
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_rs_z(AdjArgs a, AdjShell s)
{
    const int y = blockIdx.y;
    if (y < 10 * D)
        adj_rs<D>(a, s, y / 10, y % 10);
    else
        adj_z<D>(a, s, (y - 10 * D) >> 1, y & 1);
}

hipError_t launch_adj_shell(const AdjArgs &a, const AdjShell &s, hipStream_t st)
{
    const Geo &g = a.geo;
    int64_t mx = 1;
    for (int f = 0; f < g.d; ++f) {
        int64_t ss = 1;
        for (int b = 0; b < g.d; ++b)
            if (b != f) ss *= g.M[b] - 1;
        mx = std::max(mx, ss);
    }
    const unsigned nb = (unsigned)((mx + NTA - 1) / NTA), d = (unsigned)g.d;
    if (d == 3) {
        hipLaunchKernelGGL(k_adj_core<3>, dim3(nb, 8 * d), dim3(NTA), 0, st, a, s);
        hipLaunchKernelGGL(k_adj_rs_z<3>, dim3(nb, 12 * d), dim3(NTA), 0, st, a, s);
    } else {
        hipLaunchKernelGGL(k_adj_core<2>, dim3(nb, 8 * d), dim3(NTA), 0, st, a, s);
        hipLaunchKernelGGL(k_adj_rs_z<2>, dim3(nb, 12 * d), dim3(NTA), 0, st, a, s);
    }
    return hipGetLastError();
}

// Tp[fam][par][j] = T_{j+1} + sg T_{M-1-j}, sg = +1 for odd wavenumbers (par = 1).
__global__ __launch_bounds__(NTA) void k_adj_tpack(AdjArgs a, AdjShell s)
{
    const int fam = blockIdx.y;
    const int64_t len = 5 * adj_shell_size(a.geo, fam);
    for (int64_t e = blockIdx.x * (int64_t)NTA + threadIdx.x; e < len; e += (int64_t)gridDim.x * NTA) {
        const double lo = s.Rb[fam][e], hi = s.Rb[fam][len + e];
        s.Tp[fam][e] = lo - hi;
        s.Tp[fam][len + e] = lo + hi;
    }
}

// One position of the axes after the first per thread (neighbours side by side), a
// range of k0 per block row: the family-0 values of the position stay in registers.
// Bound by the ten loads of the other families' values per element, two elements' at
// once in flight (257^3, one run: 159 -> 148 us).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_x(AdjArgs a, AdjShell s, double *X)
{
    constexpr int U = 2;
    const Geo &g = a.geo;
    const int I0 = g.M[0] - 1, I1 = g.M[1] - 1, I2 = D == 3 ? g.M[2] - 1 : 1;
    const int64_t np = (int64_t)I1 * I2, p = blockIdx.x * (int64_t)NTA + threadIdx.x;
    if (p >= np) return;
    const int i1 = D == 3 ? (int)(p / I2) : (int)p, i2 = D == 3 ? (int)(p % I2) : 0;
    const int k0 = (int)((int64_t)I0 * blockIdx.y / gridDim.y), k1 = (int)((int64_t)I0 * (blockIdx.y + 1) / gridDim.y);
    const double l1 = a.tab[1].lam[i1], l2 = D == 3 ? a.tab[2].lam[i2] : 0.0;
    double T0[2][5], s1[5], s2[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        T0[0][j] = s.Tp[0][j * np + p];
        T0[1][j] = s.Tp[0][(5 + j) * np + p];
        s1[j] = a.tab[1].s[j * I1 + i1];
        s2[j] = D == 3 ? a.tab[2].s[j * I2 + i2] : 0.0;
    }
    const int64_t n1 = (int64_t)I0 * I2, n2 = (int64_t)I0 * I1;
    const double *T1 = s.Tp[1] + ((i1 + 1) & 1) * 5 * n1 + i2, *T2 = D == 3 ? s.Tp[2] + ((i2 + 1) & 1) * 5 * n2 + i1 : nullptr;
    // Lambda and m_R as polynomials of lambda_0
    double A0 = l1, A1 = 1.0 + g.c2[0][1] * l1, B0 = 0.0, B1 = g.c4[1][0] * l1 * l1, B2 = g.c4[0][1] * l1;
    if (D == 3) {
        A0 += l2 + g.c2[1][2] * l1 * l2;
        A1 += g.c2[0][2] * l2;
        B0 = g.c4[1][2] * l1 * l1 * l2 + g.c4[2][1] * l1 * l2 * l2;
        B1 += g.c4[2][0] * l2 * l2;
        B2 += g.c4[0][2] * l2;
    }
    for (int i0 = k0; i0 < k1; i0 += U) {
        double x[U], t1[U][5], t2[U][5];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = min(i0 + u, k1 - 1);
            x[u] = X[i * np + p];
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                t1[u][j] = T1[j * n1 + i * I2];
                t2[u][j] = D == 3 ? T2[j * n2 + i * I1] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u;
            if (i >= k1) break;
            const bool odd = (i & 1) == 0;
            double V = 0.0;
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                V = fma(a.tab[0].s[j * I0 + i], odd ? T0[1][j] : T0[0][j], V);
                V = fma(s1[j], t1[u][j], V);
                if (D == 3) V = fma(s2[j], t2[u][j], V);
            }
            const double l0 = a.tab[0].lam[i];
            const double L = fma(A1, l0, A0), R = fma(fma(B2, l0, B1), l0, B0);
            const double q = R / L;
            X[i * np + p] = fma(x[u], q, x[u]) + g.pref * q * V;
        }
    }
}

hipError_t launch_adj_x(const AdjArgs &a, const AdjShell &s, double *X, hipStream_t st)
{
    const Geo &g = a.geo;
    const int I0 = g.M[0] - 1;
    int64_t np = 1;
    for (int b = 1; b < g.d; ++b) np *= g.M[b] - 1;
    hipLaunchKernelGGL(k_adj_tpack, dim3(512, (unsigned)g.d), dim3(NTA), 0, st, a, s);
    const int64_t want = ((int64_t)512 * 1024 + np - 1) / np;
    const unsigned ks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, (I0 + 7) / 8));
    const dim3 grid((unsigned)((np + NTA - 1) / NTA), ks);
    if (g.d == 3)
        hipLaunchKernelGGL(k_adj_x<3>, grid, dim3(NTA), 0, st, a, s, X);
    else
        hipLaunchKernelGGL(k_adj_x<2>, grid, dim3(NTA), 0, st, a, s, X);
    return hipGetLastError();
}

// As k_adj_lambda, with the transfer's transpose taken on the g~ layers (an interior
// neighbour belongs to the lowest axis with index 1 or M-1 there) and the boundary
// terms of the sixth-order stencils from Z (zero off the core).
template <int D>
__global__ __launch_bounds__(NTA) void k_adj_lambda_shell(AdjArgs a, AdjShell sh, const double *w, int six)
{
    const Geo &g = a.geo;
    int fam = 0;
    int64_t e = blockIdx.x * (int64_t)NTA + threadIdx.x;
    while (fam < D && e >= a.lf_size[fam]) {
        e -= a.lf_size[fam];
        ++fam;
    }
    if (fam >= D) return;
    const int b = a.fb[fam], c = a.fc[fam];
    const int nb = g.M[b] + 1, ncn = D == 3 ? g.M[c] + 1 : 1;
    const int per = nb * ncn;
    const int f = (int)(e / per);
    const int rem = (int)(e % per);
    int i[3] = {0, 0, 0};
    i[fam] = f ? g.M[fam] : 0;
    i[b] = rem / ncn;
    if (D == 3) i[c] = rem % ncn;
    bool owned = true;
    for (int x = 0; x < fam; ++x)
        if (i[x] == 0 || i[x] == g.M[x]) owned = false;
    double lam = 0.0;
    if (owned) {
        lam = w[grid_off(a.n, D, i)];
        // g~ layer value of an interior node next to the boundary
        auto gt = [&](const int *j) -> double {
            int x = 0;
            while (x < D - 1 && j[x] != 1 && j[x] != g.M[x] - 1) ++x;
            int64_t o = 0;
#pragma unroll
            for (int z = 0; z < D; ++z)
                if (z != x) o = o * (g.M[z] - 1) + (j[z] - 1);
            return sh.Gb[x][(j[x] == 1 ? 0 : adj_shell_size(g, x)) + o];
        };
        auto inside = [&](const int *j) {
            bool in = true;
#pragma unroll
            for (int z = 0; z < D; ++z) in = in && j[z] >= 1 && j[z] <= g.M[z] - 1;
            return in;
        };
        double s = 0.0;
#pragma unroll
        for (int p = 0; p < D; ++p) {
            double wf = 1.0 / (g.h[p] * g.h[p]);
#pragma unroll
            for (int q = 0; q < D; ++q)
                if (q != p) wf -= 2.0 * g.c2[p][q] / (g.h[p] * g.h[p] * g.h[q] * g.h[q]);
#pragma unroll
            for (int sg = -1; sg <= 1; sg += 2) {
                int j[3] = {i[0], i[1], i[2]};
                j[p] += sg;
                if (inside(j)) s += wf * gt(j);
            }
        }
#pragma unroll
        for (int p = 0; p < D; ++p)
#pragma unroll
            for (int q = p + 1; q < D; ++q) {
                const double we = g.c2[p][q] / (g.h[p] * g.h[p] * g.h[q] * g.h[q]);
#pragma unroll
                for (int sp = -1; sp <= 1; sp += 2)
#pragma unroll
                    for (int sq = -1; sq <= 1; sq += 2) {
                        int j[3] = {i[0], i[1], i[2]};
                        j[p] += sp;
                        j[q] += sq;
                        if (inside(j)) s += we * gt(j);
                    }
            }
        lam -= s;
        if (six) {
            // in-face axes in storage order of Z (increasing)
            const int o0 = fam == 0 ? 1 : 0, o1 = D == 3 ? (fam == 2 ? 1 : 2) : o0;
            const double *Z = sh.Z[fam] + (f ? adj_shell_size(g, fam) : 0);
            auto z = [&](int j0, int j1) {
                if (j0 < 2 || j0 > g.M[o0] - 2) return 0.0;
                if (D == 3 && (j1 < 2 || j1 > g.M[o1] - 2)) return 0.0;
                return Z[D == 3 ? (int64_t)(j0 - 1) * (g.M[o1] - 1) + (j1 - 1) : j0 - 1];
            };
            const int j0 = i[o0], j1 = D == 3 ? i[o1] : 0;
            const double z0 = z(j0, j1);
            lam += g.c4[fam][o0] / (g.h[o0] * g.h[o0]) * (z(j0 - 1, j1) - 2.0 * z0 + z(j0 + 1, j1));
            if (D == 3) lam += g.c4[fam][o1] / (g.h[o1] * g.h[o1]) * (z(j0, j1 - 1) - 2.0 * z0 + z(j0, j1 + 1));
        }
    }
    a.LF[fam][e] = lam;
}

hipError_t launch_adj_lambda_shell(const AdjArgs &a, const AdjShell &s, const double *w, bool six, hipStream_t st)
{
    int64_t tot = 0;
    for (int fam = 0; fam < a.geo.d; ++fam) tot += a.lf_size[fam];
    const unsigned nb = (unsigned)((tot + NTA - 1) / NTA);
    if (a.geo.d == 3)
        hipLaunchKernelGGL(k_adj_lambda_shell<3>, dim3(nb), dim3(NTA), 0, st, a, s, w, six ? 1 : 0);
    else
        hipLaunchKernelGGL(k_adj_lambda_shell<2>, dim3(nb), dim3(NTA), 0, st, a, s, w, six ? 1 : 0);
    return hipGetLastError();
}

// Zero the boundary nodes of a grid-shaped array, a wave per row of the last axis:
// whole rows on the faces of the others, else the two ends (257^3: 33 us for a walk
// over all nodes -> 10).
template <int D>
__global__ __launch_bounds__(NTA) void k_zero_boundary(AdjArgs a, double *out, int64_t rows)
{
    const int lane = threadIdx.x & 63, n = (int)a.n[D - 1];
    const int64_t row = blockIdx.x * (int64_t)(NTA / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    int64_t r = row;
    bool face = false;
#pragma unroll
    for (int x = D - 2; x >= 0; --x) {
        const int ix = (int)(r % a.n[x]);
        r /= a.n[x];
        face = face || ix == 0 || ix == a.geo.M[x];
    }
    double *p = out + row * n;
    if (face) {
        for (int i = lane; i < n; i += 64) p[i] = 0.0;
    } else if (lane < 2) {
        p[lane == 0 ? 0 : n - 1] = 0.0;
    }
}

hipError_t launch_zero_boundary(const AdjArgs &a, double *out, hipStream_t st)
{
    int64_t rows = 1;
    for (int x = 0; x + 1 < a.geo.d; ++x) rows *= a.n[x];
    const unsigned nb = (unsigned)((rows + NTA / 64 - 1) / (NTA / 64));
    if (a.geo.d == 3)
        hipLaunchKernelGGL(k_zero_boundary<3>, dim3(nb), dim3(NTA), 0, st, a, out, rows);
    else
        hipLaunchKernelGGL(k_zero_boundary<2>, dim3(nb), dim3(NTA), 0, st, a, out, rows);
    return hipGetLastError();
}

// Face-to-slice expansion, first transform.  Tile rows = slots r of the
// transform axis (length N), tile columns = W consecutive column indices.
// Input element (r, q, s), q = slot of the other in-face axis (2D: 0), s = slice:
//   K_hat[s-1][kb(q)][kc(r)] LH0[q][r] + K_hat[M-1-s][kb][kc] LH1[q][r],
// (column, batch) = (q, s - 1), or (s - 1, q) with scol;
// followed by the hermitian synthesis along the rows.  Rows 1..M-1 of the
// result, times `scale`, are stored or (accum) added to out[(row-1)*ors +
// col*ocs + batch*obs].
template <int MAXE, int KD, int NTT>
__global__ __launch_bounds__(NTT) void k_expand(ExpandArgs a)
{
    constexpr bool BIG = NTT != NTA;
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = a.fd.N, M = a.fd.M, W = a.W, rs = BIG ? W : W + 1;
    const int lgW = 31 - __clz(W), lgs = lgW - 1;
    const cx<double> *tw = BIG ? a.tw : reinterpret_cast<const cx<double> *>(smem);
    double *buf = reinterpret_cast<double *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<double>)));
    const int ncb = (a.ncols + W - 1) / W;
    const int cb = blockIdx.x % ncb, bt = blockIdx.x / ncb;
    const int c0 = cb * W;
    const int nc = min(W, a.ncols - c0);
    if (!BIG) load_twiddles<double, NTT>(reinterpret_cast<cx<double> *>(smem), a.tw, N);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c = wave; c < W; c += NTT / 64) {
        const int col = c0 + c;
        int s, kb;
        const double *l0, *l1;
        const int q = a.scol ? bt : col; // column of the face spectra
        s = (a.scol ? col : bt) + 1;
        kb = q <= a.Mb ? q : q - a.Mb;
        l0 = a.LH0 + (int64_t)q * N;
        l1 = a.LH1 + (int64_t)q * N;
        const double *k0 = a.K + (int64_t)(s - 1) * a.Kd + (int64_t)kb * a.Kb;
        const double *k1 = a.K + (int64_t)(a.Ms - 1 - s) * a.Kd + (int64_t)kb * a.Kb;
        for (int r = lane; r < N; r += 64) {
            double v = 0.0;
            if (c < nc) {
                const int kc = r <= M ? r : r - M;
                v = k0[kc] * l0[r] + k1[kc] * l1[r];
            }
            buf[r * rs + c] = v;
        }
    }
    __syncthreads();
    pre_herm<double, MAXE, NTT>(buf, rs, lgs, M, false);
    fft_tile<double, MAXE, NTT, KD, false>(buf, rs, lgs, a.fd, tw, true);
    double *out = a.out + (int64_t)bt * a.obs + (int64_t)c0 * a.ocs;
    if (a.accum)
        tile_store_acc<double, double, NTT>(buf, rs, 1, out, M - 1, nc, a.ors, a.ocs, a.scale, lgW);
    else
        tile_store<double, double, NTT>(buf, rs, 1, out, M - 1, nc, a.ors, a.ocs, a.scale, lgW);
}

// The expansion in register tiles (see RegTile): a thread forms the products of the
// rows that its first butterfly takes, results go straight to global memory. Columns
// that are slices (SCOL) share the rows of the face spectra. Slices s and M - s, and the
// cosine and the sine column of one frequency, read the same rows of K, so blocks that
// share them run next to each other. 257^3, per family: 283 -> 187 to 198 us (of it 80 for K and
// the result at 5.1 TB/s; the rest is the latency of the loads before each transform);
// with the other slots as columns 320 us (36 loads per thread -> 52); 4097^2: 820 -> 230 and 270.
// All loads issued before their first use measured 3% slower.
template <typename R, bool SCOL>
__global__ __launch_bounds__(R::NTH) void k_expand_rt(ExpandArgs a, int nblk)
{
    constexpr int N = R::N, M = N / 2, W = R::W, P = R::P;
    extern __shared__ __align__(16) unsigned char smem[];
    const cx<double> *tw = R::LTW ? reinterpret_cast<const cx<double> *>(smem) : a.tw;
    cx<double> *buf = reinterpret_cast<cx<double> *>(smem) + (R::LTW ? N : 0);
    const int ncb = (a.ncols + W - 1) / W, tid = threadIdx.x;
    const int lb = xcd_remap(blockIdx.x, nblk);
    // index i of n as 0, n-1, 1, n-2, ..
    auto ends = [](int i, int n) { return i & 1 ? n - 1 - (i >> 1) : i >> 1; };
    // index i of n (even) as 0, n/2, 1, n/2 + 1, ..
    auto halves = [](int i, int n) { return n & 1 ? i : (i & 1) * (n >> 1) + (i >> 1); };
    int cb, bt;
    if constexpr (SCOL) {
        cb = ends(lb % ncb, ncb);
        bt = halves(lb / ncb, a.nbatch);
    } else {
        cb = lb % ncb;
        bt = ends(lb / ncb, a.nbatch);
    }
    const int c0 = cb * W, nc = min(W, a.ncols - c0);
    int j, s;
    rt_paired<R>(tid, j, s);
    double l[2][8]; // face spectra, rows k and N/2 + k (SCOL: of both columns)
    auto fetch_l = [&](int q) {
        const double *l0 = a.LH0 + (int64_t)q * N + j, *l1 = a.LH1 + (int64_t)q * N + j;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            l[0][r] = l0[r * P];
            l[1][r] = l1[r * P];
        }
    };
    cx<double> C[4], S[4];
    if (SCOL) fetch_l(bt);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const bool in = 2 * s + c < nc;
        const int col = c0 + (in ? 2 * s + c : 0);
        const int q = SCOL ? bt : col, sl = (SCOL ? col : bt) + 1;
        const int kb = q <= a.Mb ? q : q - a.Mb;
        if (!SCOL) fetch_l(q);
        const double *k0 = a.K + (int64_t)(sl - 1) * a.Kd + (int64_t)kb * a.Kb + j;
        const double *k1 = a.K + (int64_t)(a.Ms - 1 - sl) * a.Kd + (int64_t)kb * a.Kb + j;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double a0 = k0[r * P], a1 = k1[r * P];
            // (row N/2 in the place of the sine row of k = 0)
            const double b0 = r == 0 ? k0[j == 0 ? M : 0] : a0, b1 = r == 0 ? k1[j == 0 ? M : 0] : a1;
            const double cv = a0 * l[0][r] + a1 * l[1][r], sv = b0 * l[0][4 + r] + b1 * l[1][4 + r];
            (c == 0 ? C[r].x : C[r].y) = in ? cv : 0.0;
            (c == 0 ? S[r].x : S[r].y) = in ? sv : 0.0;
        }
    }
    if constexpr (R::LTW) load_twiddles<double, R::NTH>(reinterpret_cast<cx<double> *>(smem), a.tw, N);
    cx<double> v[8];
    rt_unfold_herm<double, R>(C, S, j, v);
    rt_first<double, R, true>(buf, v, j, s);
    rt_middle<double, R, true>(buf, tw, tid);
    rt_plain<R>(tid, j, s);
    rt_last<double, R, true>(buf, tw, v, j, s);
    double *out = a.out + (int64_t)bt * a.obs + (int64_t)c0 * a.ocs;
    const int c = 2 * s, ocs = (int)a.ocs, ors = (int)a.ors;
    const bool both = c + 1 < nc;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = j + r * P - 1;
        if (t < 0 || c >= nc) continue;
        double *p = out + toff(t, ors, c, ocs);
        pair_t<double> w = {a.scale * v[r].x, a.scale * v[r].y};
        if (ocs == 1 && both) {
            pair_t<double> *pp = reinterpret_cast<pair_t<double> *>(p);
            if (a.accum) {
                const pair_t<double> o = *pp;
                w.a += o.a;
                w.b += o.b;
            }
            *pp = w;
        } else if (a.accum) {
            p[0] += w.a;
            if (both) p[ocs] += w.b;
        } else {
            p[0] = w.a;
            if (both) p[ocs] = w.b;
        }
    }
}

template <typename R, bool SCOL>
static void launch_expand_rt(const ExpandArgs &a, int nblk, hipStream_t st)
{
    const size_t lds = rt_lds<double, R>();
    set_lds((const void *)&k_expand_rt<R, SCOL>, lds);
    hipLaunchKernelGGL((k_expand_rt<R, SCOL>), dim3((unsigned)nblk), dim3(R::NTH), lds, st, a, nblk);
}

template <int MAXE, int NTT = NTA>
static void launch_expand_m(const ExpandArgs &a, unsigned nblk, size_t lds, hipStream_t st)
{
    auto go = [&](auto kd) {
        constexpr int KD = decltype(kd)::value;
        set_lds((const void *)&k_expand<MAXE, KD, NTT>, lds);
        hipLaunchKernelGGL((k_expand<MAXE, KD, NTT>), dim3(nblk), dim3(NTT), lds, st, a);
    };
    if constexpr (NTT != NTA)
        go(std::integral_constant<int, kAnyLen>()); // (powers of two: register tiles)
    else if constexpr (MAXE <= 8)
        by_kind(a.fd.N, go);
    else
        by_pow2(a.fd.N, go);
}

hipError_t launch_expand(const ExpandArgs &a, hipStream_t st)
{
    const int ncb = (a.ncols + a.W - 1) / a.W;
    const unsigned nblk = (unsigned)ncb * (unsigned)a.nbatch;
    const int work = (a.W / 2) * a.fd.N;
    if (nblk == 0) return hipSuccess;
    if (!tile_strides_ok(a.fd.M, a.ors, a.ncols, a.ocs)) return hipErrorInvalidValue;
    if (rt_tile<0>(a.fd.N, a.W, [&](auto tile) {
            if (a.scol)
                launch_expand_rt<decltype(tile), true>(a, (int)nblk, st);
            else
                launch_expand_rt<decltype(tile), false>(a, (int)nblk, st);
        }))
        return hipGetLastError();
    if (a.fd.N > 2048) {
        // long transforms: one complex sequence per tile, global twiddles
        const size_t lds = (size_t)a.fd.N * a.W * sizeof(double);
        if (a.W != 2 || work > 8 * 1024) return hipErrorInvalidValue;
        if (work <= 4 * 1024)
            launch_expand_m<4, 1024>(a, nblk, lds, st);
        else
            launch_expand_m<8, 1024>(a, nblk, lds, st);
        return hipGetLastError();
    }
    const size_t lds = (size_t)a.fd.N * sizeof(cx<double>) + (size_t)a.fd.N * (a.W + 1) * sizeof(double);
    if (work <= 4 * NTA)
        launch_expand_m<4>(a, nblk, lds, st);
    else if (work <= 8 * NTA)
        launch_expand_m<8>(a, nblk, lds, st);
    else if (work <= 16 * NTA)
        launch_expand_m<16>(a, nblk, lds, st);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// 1D adjoint in one block: with w = phi_bar on the M+1 nodes,
//   lambda_0 = w_0 + sum_j w_j (1 - j/M),  lambda_M = w_M + sum_j w_j j/M,
//   rho_bar_s = phi_star(w_I)_s + h (G(s h) lambda_0 + G((M - s) h) lambda_M),
// G(r) = r/2, rho_bar on the two end nodes = 0.
template <int MAXE, int KD, int NTT>
__global__ __launch_bounds__(NTT) void k_adj_1d(const double *w, double *out, int M, double h,
                                                FftDesc fd, const cx<double> *twg, AxisTabs tab)
{
    constexpr bool BIG = NTT != NTA;
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = fd.N, rs = BIG ? 2 : 3, lgW = 1;
    const cx<double> *tw = BIG ? twg : reinterpret_cast<const cx<double> *>(smem);
    double *buf = reinterpret_cast<double *>(smem + (BIG ? 0 : (size_t)N * sizeof(cx<double>)));
    __shared__ double red[2][NTT];
    if (!BIG) load_twiddles<double, NTT>(reinterpret_cast<cx<double> *>(smem), twg, N);
    double s0 = 0.0, s1 = 0.0;
    for (int j = 1 + threadIdx.x; j < M; j += NTT) {
        s0 += w[j] * ((double)(M - j) / M);
        s1 += w[j] * ((double)j / M);
    }
    red[0][threadIdx.x] = s0;
    red[1][threadIdx.x] = s1;
    zero_rows<double, NTT>(buf, rs, lgW, 0, 1);
    zero_rows<double, NTT>(buf, rs, lgW, M, N);
    tile_load<double, double, NTT>(buf, rs, 1, w + 1, M - 1, 1, 1, 1, lgW);
    __syncthreads();
    for (int k = NTT / 2; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            red[0][threadIdx.x] += red[0][threadIdx.x + k];
            red[1][threadIdx.x] += red[1][threadIdx.x + k];
        }
        __syncthreads();
    }
    const double l0 = w[0] + red[0][0], l1 = w[M] + red[1][0];
    fft_tile<double, MAXE, NTT, KD, false>(buf, rs, 0, fd, tw, false);
    post_cs<double, MAXE, NTT>(buf, rs, 0, M);
    for (int k = 1 + threadIdx.x; k < M; k += NTT)
        buf[(M + k) * rs] = -(2.0 / M) * buf[(M + k) * rs] / tab.q[k - 1];
    __syncthreads();
    pre_herm<double, MAXE, NTT>(buf, rs, 0, M, true);
    fft_tile<double, MAXE, NTT, KD, false>(buf, rs, 0, fd, tw, true);
    for (int j = threadIdx.x; j <= M; j += NTT) {
        double v = 0.0;
        if (j > 0 && j < M)
            v = 0.5 * buf[j * rs] + h * (0.5 * (j * h) * l0 + 0.5 * ((M - j) * h) * l1);
        out[j] = v;
    }
}

hipError_t launch_adj_1d(const double *w, double *out, int M, double h, const FftDesc &fd,
                         const cx<double> *tw, const AxisTabs &tab, hipStream_t st)
{
    const size_t lds = tile_lds<double>(fd.N, 2);
    auto go = [&](auto maxe, auto ntt) {
        constexpr int MAXE = decltype(maxe)::value, NTT = decltype(ntt)::value;
        by_kind(fd.N, [&](auto kd) {
            constexpr int KD = decltype(kd)::value;
            set_lds((const void *)&k_adj_1d<MAXE, KD, NTT>, lds);
            hipLaunchKernelGGL((k_adj_1d<MAXE, KD, NTT>), dim3(1), dim3(NTT), lds, st, w, out, M, h, fd, tw, tab);
        });
        return hipGetLastError();
    };
    return by_length(fd.N, go);
}

} // namespace ips
