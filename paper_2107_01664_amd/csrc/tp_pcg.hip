// Two-level additive Schwarz preconditioned CG for the cotan Poisson solves (Sec. 5.2).
//
// Unknowns are reordered by (connected component, Morton code of the vertex position on
// the component's bounding cube) and cut into blocks of at most kBS consecutive vertices,
// so every block is a compact patch of the surface.  The preconditioner is
//     M^{-1} r = sum_B R_B^T C_BB^{-1} R_B r  +  Phi C_0^{-1} Phi^T r,
// with C_BB the block's rows and columns of C (dense inverse by register-tiled
// Gauss-Jordan, stored in FP32) and Phi a linear coarse space: aggregates of consecutive
// blocks of one component, each carrying an orthonormalised basis of {1, x, y, z} centred
// and scaled on the aggregate.  C_0 = Phi^T C Phi is assembled from per-row coarse weights;
// per component the rank-one term d e e^T / (e^T e) (e the coefficients of the component's
// constant, d the mean kept diagonal) makes it definite and leaves its action on
// per-component mean-zero vectors equal to the pseudo-inverse.
//
// The solver is the Chronopoulos-Gear form of preconditioned CG: with u = M^{-1} r and
// w = C u, the sums gamma = (r,u) and delta = (w,u) give beta = gamma / gamma_old and
// alpha = gamma / (delta - beta gamma / alpha_old), and p = u + beta p, s = w + beta s (= C p),
// x += alpha p, r -= alpha s.  One workgroup of kPcgThreads threads owns one block and keeps
// C_BB^{-1} in registers for the whole solve.  An iteration has two exchanges between the
// workgroups, of values that carry their own arrival (publish / peek).  In the first, every block
// publishes its block solve v = C_BB^{-1} r_B and its shares Phi_B^T r of the coarse
// right-hand side; after it, every workgroup forms the coarse values of the aggregates its
// rows touch, u = v + Phi c and C u from the neighbours' v.  In the second, the block
// partials of (r,u), (w,u) and (r,r) are added.  All partial sums are added in block order
// by every workgroup, so every workgroup takes the same decisions and the result does not
// depend on scheduling.  (The pipelined form, which folds the sums into the next exchange,
// lost convergence here: relative perturbations of 1e-15 per iteration in its auxiliary
// recurrences already cost 15 % more iterations and 1e-13 stalled it, while this form is
// unchanged up to 1e-13.)  A solve may start from a given x (warm start; the tolerance
// stays relative to |b|).  Every solve ends by checking the true residual b - C x and
// restarts from it when the recursively updated residual has drifted.  Problems with more
// blocks than can be resident at once run the same iteration with two or four blocks per
// workgroup (k_pcg_wide), beyond 1,024 blocks as one launch per phase (k_ml_*).
#include "tp_solver.h"

#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>

namespace tp {

constexpr int kBS = 128;            // vertices per block = row-owning threads of a solver workgroup
constexpr int kThreads = 2 * kBS;   // threads per workgroup of the multi-launch block kernel
constexpr int kMaxAggNbn = 16;      // aggregates touching a block (its own included)
constexpr int kMaxNbPcg = 256;      // blocks (one co-resident workgroup per block)
constexpr int kMaxAggBlocks = 7;    // blocks per aggregate: ceil(4 kMaxNbPcg / kCoarseMax)
constexpr int kMaxNbMulti = 16384;  // blocks of the multi-launch solve (2,097,152 vertices)

// ---------------------------------------------------------------- per-geometry setup

// Permuted ELL values: row inew of the permuted matrix is row perm[inew] of C, entries in
// CSR order (the permuted column indices were built with the pattern).
__global__ void k_perm_ell_vals(int64_t n, int w, const int32_t* __restrict__ perm,
                                const int32_t* __restrict__ off, const double* __restrict__ val,
                                double* __restrict__ pval)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t old = perm[i];
    const int32_t b = off[old], len = off[old + 1] - b;
    for (int e = 0; e < w; ++e) pval[(int64_t)e * n + i] = e < len ? val[b + e] : 0.0;
}

// Dense inverse of each diagonal block (Gauss-Jordan in LDS; the block is symmetric
// positive definite, or made so by the rank-one term, so no pivoting is needed).
// In-place Gauss-Jordan inverse of an n x n symmetric positive definite matrix (no
// pivoting) held in registers.  The matrix is NC x NC (NC = RB * NRB = CB * NCB; rows and
// columns n .. NC-1 zero); thread t < NRB * NCB holds the RB x CB tile a[r][c] =
// A[rb RB + r][cb CB + c] with rb = t % NRB, cb = t / NRB.  Pivot k with d = a_kk and
// g_i = a_ik / d:
//   a_ij -> a_ij - g_i a_kj (i, j != k),  a_kj -> a_kj / d,  a_ik -> -g_i,  a_kk -> 1 / d;
// row k takes the same multiply-add as the others with the multiplier 1 - 1/d.  Per pivot
// the pivot row and column pass through LDS (two copies, alternating, so one workgroup
// barrier per pivot suffices: a copy is written again only two pivots later, after every
// thread has passed the barrier in between); a thread reads CB + RB of their values for
// its RB CB multiply-adds.  The pivot's position within a tile is a compile-time constant
// of the unrolled inner loop (its length L is a multiple of RB and CB), so the tile stays
// in registers.  Threads t >= NRB * NCB only join the barriers.
template <int RB, int CB, int NRB, int NCB>
__device__ __forceinline__ void gj_inverse_tiles(double (&a)[RB][CB], int n, double* prow, double* fcol)
{
    constexpr int NC = RB * NRB;
    static_assert(CB * NCB == NC, "square tiling");
    constexpr int L = RB * CB / (RB % CB == 0 ? CB : (CB % RB == 0 ? RB : 1));   // RB, CB | L
    static_assert(L % RB == 0 && L % CB == 0, "unrolled pivots cover whole tiles");
    const int t = threadIdx.x;
    const bool on = t < NRB * NCB;
    const int rb = t % NRB, cb = t / NRB;
    int buf = 0;
    for (int k0 = 0; k0 < n; k0 += L) {
#pragma unroll
        for (int kk = 0; kk < L; ++kk) {
            const int k = k0 + kk;
            if (k < n) {
                const int rk = kk % RB, ck = kk % CB;   // position of row / column k in a tile
                double* pr = prow + buf * NC;
                double* fc = fcol + buf * NC;
                if (on && rb == k / RB) {
#pragma unroll
                    for (int c = 0; c < CB; ++c) pr[cb * CB + c] = a[rk][c];
                }
                if (on && cb == k / CB) {
#pragma unroll
                    for (int r = 0; r < RB; ++r) fc[rb * RB + r] = a[r][ck];
                }
                __syncthreads();
                const double invd = 1.0 / pr[k];
                if (on) {
                    double p[CB], g[RB], h[RB];
#pragma unroll
                    for (int c = 0; c < CB; ++c) p[c] = pr[cb * CB + c];
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        g[r] = fc[rb * RB + r] * invd;
                        h[r] = rb * RB + r == k ? 1.0 - invd : g[r];
                    }
#pragma unroll
                    for (int r = 0; r < RB; ++r)
#pragma unroll
                        for (int c = 0; c < CB; ++c) a[r][c] = __builtin_fma(-h[r], p[c], a[r][c]);
                    if (cb == k / CB) {
#pragma unroll
                        for (int r = 0; r < RB; ++r) a[r][ck] = rb * RB + r == k ? invd : -g[r];
                    }
                }
                buf ^= 1;
            }
        }
    }
}

// Inverse of block B by one workgroup of kInvThreads threads.
constexpr int kInvThreads = 512;
__device__ __forceinline__ void block_inverse(int B, int64_t n, int w, const int32_t* __restrict__ pcol,
                                              const double* __restrict__ pval, const int32_t* __restrict__ bstart,
                                              const int32_t* __restrict__ whole, float* __restrict__ Binv)
{
    extern __shared__ __align__(16) double A[];   // kBS x kBS, row-major
    __shared__ double prow[2 * kBS], fcol[2 * kBS];
    const int32_t s0 = bstart[B], cnt = bstart[B + 1] - s0;
    for (int t = threadIdx.x; t < kBS * kBS; t += kInvThreads) A[t] = 0.0;
    __syncthreads();
    for (int t = threadIdx.x; t < kBS; t += kInvThreads) {
        if (t < cnt) {
            const int64_t i = s0 + t;
            for (int e = 0; e < w; ++e) {
                const int32_t j = pcol[(int64_t)e * n + i];
                if (j >= s0 && j < s0 + cnt) A[t * kBS + (j - s0)] += pval[(int64_t)e * n + i];
            }
        } else {
            A[t * kBS + t] = 1.0;             // padding rows: identity
        }
    }
    __syncthreads();
    if (whole[B]) {
        // rank-one term (d / cnt) 1 1^T on the block, d = mean diagonal
        __shared__ double dsum;
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int t = 0; t < cnt; ++t) s += A[t * kBS + t];
            dsum = s / cnt;
        }
        __syncthreads();
        const double add = dsum / cnt;
        for (int t = threadIdx.x; t < cnt * cnt; t += kInvThreads) A[(t / cnt) * kBS + (t % cnt)] += add;
        __syncthreads();
    }
    // tiles of 4 rows x 8 columns: 32 row blocks x 16 column blocks
    constexpr int RB = 4, CB = 8, NRB = kBS / RB, NCB = kBS / CB;
    static_assert(NRB * NCB == kInvThreads, "one tile per thread");
    const int rb = threadIdx.x % NRB, cb = threadIdx.x / NRB;
    double a[RB][CB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c) a[r][c] = A[(rb * RB + r) * kBS + cb * CB + c];
    gj_inverse_tiles<RB, CB, NRB, NCB>(a, kBS, prow, fcol);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c) A[(rb * RB + r) * kBS + cb * CB + c] = a[r][c];
    __syncthreads();
    // symmetrize (the elimination leaves rounding-level asymmetry) and round to FP32
    float* dst = Binv + (int64_t)B * kBS * kBS;
    for (int t = threadIdx.x; t < kBS * kBS; t += kInvThreads) {
        const int i = t / kBS, j = t - i * kBS;
        dst[t] = (float)(0.5 * (A[i * kBS + j] + A[j * kBS + i]));
    }
}

// ---- coarse space: per aggregate, an orthonormal basis (in the Euclidean product on the
// aggregate's vertices) of {1, x, y, z}, with x, y, z centred and scaled on the aggregate.
// It is the Cholesky factor L of the 4 x 4 Gram matrix that orthonormalises: phi = V L^-T.
// A function whose remainder after the previous ones is below 1e-6 of its norm (a flat or
// tiny aggregate) is dropped: its values are zero and its coarse row and column are zero
// but for a unit diagonal.

constexpr int kAggThreads = 256;

// Fixed-order sum of M values per thread over a kAggThreads workgroup.
template <int M>
__device__ __forceinline__ void agg_sum(const double (&v)[M], double* sh, double* out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const double s = wave_sum(v[q]);
        if (lane == 0) sh[wave * M + q] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < M) {
        double a = 0.0;
        for (int w = 0; w < kAggThreads / 64; ++w) a += sh[w * M + threadIdx.x];
        out[threadIdx.x] = a;
    }
    __syncthreads();
}

// One workgroup per aggregate: phi[i][0..4) for its rows (block order) and esum[4g + a].
__global__ __launch_bounds__(kAggThreads) void k_agg_basis(const int32_t* __restrict__ perm,
                                                             const double* __restrict__ V,
                                                             const int32_t* __restrict__ astart,
                                                             const int32_t* __restrict__ bstart,
                                                             double* __restrict__ phi, double* __restrict__ esum)
{
    __shared__ double sh[(kAggThreads / 64) * 10];
    __shared__ double tot[10];
    __shared__ double T[16];
    const int g = blockIdx.x;
    const int v0 = bstart[astart[g]], v1 = bstart[astart[g + 1]];
    const double m = (double)(v1 - v0);
    // centroid
    double ps[3] = {0.0, 0.0, 0.0};
    for (int i = v0 + (int)threadIdx.x; i < v1; i += kAggThreads) {
        const int64_t o = (int64_t)perm[i] * 3;
        ps[0] += V[o]; ps[1] += V[o + 1]; ps[2] += V[o + 2];
    }
    agg_sum<3>(ps, sh, tot);
    const double cx = tot[0] / m, cy = tot[1] / m, cz = tot[2] / m;
    __syncthreads();
    // scale: largest coordinate offset (a maximum does not depend on the order)
    double pm[1] = {0.0};
    for (int i = v0 + (int)threadIdx.x; i < v1; i += kAggThreads) {
        const int64_t o = (int64_t)perm[i] * 3;
        pm[0] = fmax(pm[0], fmax(fabs(V[o] - cx), fmax(fabs(V[o + 1] - cy), fabs(V[o + 2] - cz))));
    }
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double w = pm[0];
        for (int off = 32; off > 0; off >>= 1) w = fmax(w, __shfl_xor(w, off));
        if (lane == 0) sh[wave] = w;
        __syncthreads();
        if (threadIdx.x == 0) {
            double a = 0.0;
            for (int q = 0; q < kAggThreads / 64; ++q) a = fmax(a, sh[q]);
            tot[0] = a > 0.0 ? 1.0 / a : 1.0;
        }
        __syncthreads();
    }
    const double is = tot[0];
    __syncthreads();
    // Gram matrix of (1, x', y', z'): entries (0,0) (0,1) (0,2) (0,3) (1,1) (1,2) (1,3) (2,2) (2,3) (3,3)
    double gs[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) gs[q] = 0.0;
    for (int i = v0 + (int)threadIdx.x; i < v1; i += kAggThreads) {
        const int64_t o = (int64_t)perm[i] * 3;
        const double f[4] = {1.0, (V[o] - cx) * is, (V[o + 1] - cy) * is, (V[o + 2] - cz) * is};
        int q = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = a; b < 4; ++b) gs[q++] += f[a] * f[b];
    }
    agg_sum<10>(gs, sh, tot);
    if (threadIdx.x == 0) {
        double G[4][4];
        int q = 0;
        for (int a = 0; a < 4; ++a)
            for (int b = a; b < 4; ++b) G[a][b] = G[b][a] = tot[q++];
        // Cholesky with dropped pivots, then T = L^{-1} (rows of dropped functions zero)
        double L[4][4] = {};
        bool keep[4];
        for (int a = 0; a < 4; ++a) {
            double d = G[a][a];
            for (int c = 0; c < a; ++c) d -= L[a][c] * L[a][c];
            keep[a] = d > 1e-12 * G[a][a] && G[a][a] > 0.0;
            const double la = keep[a] ? sqrt(d) : 0.0;
            L[a][a] = la;
            for (int b = a + 1; b < 4; ++b) {
                double v = G[b][a];
                for (int c = 0; c < a; ++c) v -= L[b][c] * L[a][c];
                L[b][a] = keep[a] ? v / la : 0.0;
            }
        }
        double Ti[4][4] = {};
        for (int a = 0; a < 4; ++a) {
            if (!keep[a]) continue;
            Ti[a][a] = 1.0 / L[a][a];
            for (int b = 0; b < a; ++b) {
                double v = 0.0;
                for (int c = b; c < a; ++c) v += L[a][c] * Ti[c][b];
                Ti[a][b] = -v / L[a][a];
            }
        }
        for (int a = 0; a < 4; ++a)
            for (int b = 0; b < 4; ++b) T[a * 4 + b] = Ti[a][b];
    }
    __syncthreads();
    double es[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = v0 + (int)threadIdx.x; i < v1; i += kAggThreads) {
        const int64_t o = (int64_t)perm[i] * 3;
        const double f[4] = {1.0, (V[o] - cx) * is, (V[o + 1] - cy) * is, (V[o + 2] - cz) * is};
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            double v = 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) v += T[a * 4 + b] * f[b];
            phi[(int64_t)i * 4 + a] = v;
            es[a] += v;
        }
    }
    agg_sum<4>(es, sh, tot);
    if (threadIdx.x < 4) esum[4 * g + threadIdx.x] = tot[threadIdx.x];
}

// Per row i and slot q (an aggregate the row's entries reach): rw[q][a][i] = sum over the
// entries j of that aggregate of C_ij phi_j[a], added in ELL order.
__global__ void k_row_coarse(int64_t n, int w, const int32_t* __restrict__ pcol, const double* __restrict__ pval,
                             const int8_t* __restrict__ eslot, const double* __restrict__ phi, double* __restrict__ rw)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc[kPcgRowSlots][4];
#pragma unroll
    for (int q = 0; q < kPcgRowSlots; ++q)
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[q][a] = 0.0;
    for (int e = 0; e < w; ++e) {
        const int32_t j = pcol[(int64_t)e * n + i];
        const double c = pval[(int64_t)e * n + i];
        const int q = eslot[(int64_t)e * n + i];
#pragma unroll
        for (int qq = 0; qq < kPcgRowSlots; ++qq)
            if (qq == q)
#pragma unroll
                for (int a = 0; a < 4; ++a) acc[qq][a] += c * phi[(int64_t)j * 4 + a];
    }
#pragma unroll
    for (int q = 0; q < kPcgRowSlots; ++q)
#pragma unroll
        for (int a = 0; a < 4; ++a) rw[((int64_t)q * 4 + a) * n + i] = acc[q][a];
}

// Galerkin coarse matrix rows of aggregate g: C0[4g + a][4h + b] = sum over rows i of g of
// phi_i[a] rw[q(h)][b][i].  kAggThreads threads = 16 row groups x 16 (a, b) pairs; each group
// adds a contiguous share of the rows, the groups are added in order.  What bounds it is latency:
// a row's block, slots, list entries and sums are three trips to memory in series, taken for four
// rows at a time.  40 aggregates of 2,500 rows: 265 us row by row, 86 now.
constexpr int kAsmGroups = kAggThreads / 16;
__global__ __launch_bounds__(kAggThreads) void k_coarse_assemble(int64_t n, int na, int nc,
                                                                   const int32_t* __restrict__ astart,
                                                                   const int32_t* __restrict__ bstart,
                                                                   const int32_t* __restrict__ blk,
                                                                   const int32_t* __restrict__ abl_off,
                                                                   const int32_t* __restrict__ abl,
                                                                   const int8_t* __restrict__ rslot,
                                                                   const double* __restrict__ phi,
                                                                   const double* __restrict__ rw,
                                                                   double* __restrict__ C0)
{
    extern __shared__ __align__(16) double acc[];   // [kAsmGroups][na][16]
    const int g = blockIdx.x;
    const int v0 = bstart[astart[g]], v1 = bstart[astart[g + 1]];
    for (int t = threadIdx.x; t < kAsmGroups * na * 16; t += kAggThreads) acc[t] = 0.0;
    __syncthreads();
    const int grp = threadIdx.x / 16, ab = threadIdx.x % 16, a = ab / 4, b = ab % 4;
    const int rows = v1 - v0, chunk = (rows + kAsmGroups - 1) / kAsmGroups;
    const int r0 = v0 + grp * chunk, r1 = min(v1, r0 + chunk);
    double* my = acc + (int64_t)grp * na * 16;
    constexpr int U = 4, Q = kPcgRegSlots;   // rows, and slots of each, with their loads in flight together
    for (int i0 = r0; i0 < r1; i0 += U) {
        int off[U], sl[U][Q], h[U][Q];
        double pa[U], w[U][Q];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u, r1 - 1);
            off[u] = blk[i];
            pa[u] = phi[(int64_t)i * 4 + a];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                sl[u][q] = rslot[(int64_t)q * n + i];
                w[u][q] = rw[((int64_t)q * 4 + b) * n + i];   // (zero in the slots that are not used)
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) off[u] = abl_off[off[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) h[u][q] = abl[off[u] + max(sl[u][q], 0)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u >= r1) break;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (sl[u][q] >= 0) my[h[u][q] * 16 + ab] += pa[u] * w[u][q];
            if (sl[u][Q - 1] < 0) continue;
            for (int q = Q; q < kPcgRowSlots; ++q) {
                const int s = rslot[(int64_t)q * n + i0 + u];
                if (s >= 0) my[abl[off[u] + s] * 16 + ab] += pa[u] * rw[((int64_t)q * 4 + b) * n + i0 + u];
            }
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < na * 16; t += kAggThreads) {
        double v = 0.0;
        for (int q = 0; q < kAsmGroups; ++q) v += acc[(int64_t)q * na * 16 + t];
        const int h = t / 16, aa = (t % 16) / 4, bb = t % 4;
        C0[(int64_t)(4 * g + aa) * nc + 4 * h + bb] = v;
    }
}

// Inverse of the nc x nc coarse matrix (nc <= kCoarseMax) after the regularisation of each
// component's constants: with e the coefficients of the component's constant function in the
// coarse basis (e_d = sum of coarse function d), the term dmean e e^T / (e^T e) is added,
// dmean the mean of the kept diagonal entries; the action on per-component mean-zero vectors
// is that of the pseudo-inverse.  The matrix is symmetric positive definite, so no pivoting
// is needed.
constexpr int kCoarseThreads = 512;
constexpr int kCoarseMax = 160;
// tiles of 5 rows x 10 columns: 32 row blocks x 16 column blocks
constexpr int kCoarseRB = 5, kCoarseCB = 10;
constexpr int kCoarseNRB = kCoarseMax / kCoarseRB, kCoarseNCB = kCoarseMax / kCoarseCB;
static_assert(kCoarseNRB * kCoarseNCB <= kCoarseThreads, "one tile per thread");
constexpr int kMaxCoarseComp = kCoarseMax / 4;
static_assert(kMaxAggBlocks * kCoarseMax >= 4 * kMaxNbPcg, "aggregates of up to kMaxAggBlocks blocks");

// One workgroup: the regularised matrix is formed in registers (a tile per thread),
// inverted there (gj_inverse_tiles) and written over G, each entry pair (i, j), (j, i)
// from the upper triangle, so the result is exactly symmetric.
__device__ __forceinline__ void coarse_inverse(int nc, const int32_t* __restrict__ acomp,
                                               const double* __restrict__ esum, double* __restrict__ G)
{
    __shared__ double prow[2 * kCoarseMax], fcol[2 * kCoarseMax];
    __shared__ double diag[kCoarseMax], es[kCoarseMax];
    __shared__ int32_t comp[kCoarseMax];
    __shared__ double enorm[kMaxCoarseComp];   // e^T e per component
    __shared__ double dmean_sh;
    const int t = threadIdx.x;
    if (t < nc) {
        diag[t] = G[(int64_t)t * nc + t];
        es[t] = esum[t];
        comp[t] = acomp[t / 4];   // components are numbered densely over the aggregates
    }
    __syncthreads();
    if (t == 0) {
        double sd = 0.0;
        int cnt = 0;
        for (int i = 0; i < nc; ++i)
            if (diag[i] > 0.0) {
                sd += diag[i];
                ++cnt;
            }
        dmean_sh = cnt > 0 ? sd / cnt : 1.0;
    }
    if (t < kMaxCoarseComp) {
        double en = 0.0;
        for (int i = 0; i < nc; ++i)
            if (comp[i] == t) en += es[i] * es[i];
        enorm[t] = en;
    }
    __syncthreads();
    const double dmean = dmean_sh;
    constexpr int RB = kCoarseRB, CB = kCoarseCB, NRB = kCoarseNRB, NCB = kCoarseNCB;
    const bool on = t < NRB * NCB;
    const int rb = t % NRB, cb = t / NRB;
    double a[RB][CB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int i = rb * RB + r, j = cb * CB + c;
            double v = 0.0;
            if (on && i < nc && j < nc) {
                // the two triangles are assembled by different aggregates: their mean is used
                v = 0.5 * (G[(int64_t)i * nc + j] + G[(int64_t)j * nc + i]);
                const int ci = comp[i];
                if (ci == comp[j] && enorm[ci] > 0.0) v += dmean * es[i] * es[j] / enorm[ci];
                if (i == j && !(diag[i] > 0.0)) v = 1.0;   // dropped coarse function
            }
            a[r][c] = v;
        }
    // every thread has read its entries of G before the first barrier of the inversion, and
    // G is written only after the last one
    gj_inverse_tiles<RB, CB, NRB, NCB>(a, nc, prow, fcol);
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int i = rb * RB + r, j = cb * CB + c;
            if (on && i < nc && j < nc && j >= i) {
                G[(int64_t)i * nc + j] = a[r][c];
                G[(int64_t)j * nc + i] = a[r][c];
            }
        }
}

// The coarse inverse (workgroup 0) and the block inverses (workgroups 1 .. nb) in one launch: they
// are independent, so the coarse inverse's single workgroup runs beside the blocks' workgroups
// instead of after them.  It takes longest and goes first: last, it began when the blocks before it
// were done (782 blocks: 392 us, 327 now).
static_assert(kCoarseThreads == kInvThreads, "one workgroup size for both inverses");
__global__ __launch_bounds__(kInvThreads) void k_inverses(int nb, int64_t n, int w, const int32_t* __restrict__ pcol,
                                                          const double* __restrict__ pval,
                                                          const int32_t* __restrict__ bstart,
                                                          const int32_t* __restrict__ whole, float* __restrict__ Binv,
                                                          int nc, const int32_t* __restrict__ acomp,
                                                          const double* __restrict__ esum, double* __restrict__ G)
{
    if (blockIdx.x > 0) block_inverse((int)blockIdx.x - 1, n, w, pcol, pval, bstart, whole, Binv);
    else coarse_inverse(nc, acomp, esum, G);
}

// forward: dst[i][c] = src[perm[i]][c0 + c] (dst in block order, row stride k);
// backward: dst[perm[i]][c0 + c] = src[i][c].  ld is the row stride of the vertex-order side.
struct PermJobs {
    PermJob j[kMaxVecJobs];
};

__global__ void k_permute_rows(PermJobs jb, int k, int ld, int c0, int forward)
{
    const PermJob& J = jb.j[blockIdx.y];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= J.n * k) return;
    const int64_t i = t / k;
    const int c = (int)(t - i * k);
    if (forward) J.dst[i * k + c] = J.src[(int64_t)J.perm[i] * ld + c0 + c];
    else J.dst[(int64_t)J.perm[i] * ld + c0 + c] = J.src[i * k + c];
}

// Sum of n values p[0], p[stride], ... in a fixed order: four interleaved partial sums, so
// four loads are in flight at a time, added as (s0 + s1) + (s2 + s3).
__device__ __forceinline__ double sum_fixed(const double* __restrict__ p, int n, int64_t stride)
{
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int i = 0;
    for (; i + 4 <= n; i += 4) {
        const double v0 = p[(int64_t)i * stride], v1 = p[(int64_t)(i + 1) * stride];
        const double v2 = p[(int64_t)(i + 2) * stride], v3 = p[(int64_t)(i + 3) * stride];
        a0 += v0;
        a1 += v1;
        a2 += v2;
        a3 += v3;
    }
    for (; i < n; ++i) a0 += p[(int64_t)i * stride];
    return (a0 + a1) + (a2 + a3);
}

// Dot product sum_i a[i] b[i * bstride] in a fixed order: the loads of 8 terms at a time
// are issued before they are added, term i to partial sum i % 4, and the partial sums are
// added as (s0 + s1) + (s2 + s3).
__device__ __forceinline__ double dot_fixed(const double* __restrict__ a, const double* __restrict__ b, int n,
                                            int bstride)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        double x[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            x[u] = a[i + u];
            y[u] = b[(i + u) * bstride];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u & 3] += x[u] * y[u];
    }
    for (; i < n; ++i) acc[i & 3] += a[i] * b[i * bstride];
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Fixed-order workgroup reduction of M values per thread (kThreads threads): butterfly
// within each wave, then the waves added in order.  Result in out[0 .. M).
template <int M>
__device__ __forceinline__ void wg_reduce(const double (&v)[M], double* wave_sh, double* out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const double s = wave_sum(v[q]);
        if (lane == 0) wave_sh[wave * M + q] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < M) {
        double a = wave_sh[threadIdx.x];
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) a += wave_sh[w * M + threadIdx.x];
        out[threadIdx.x] = a;
    }
    __syncthreads();
}

// ---------------------------------------------------------------- solver

struct PcgArgs {
    int64_t n;
    int nb;
    int nc;                   // coarse functions (4 per aggregate)
    int ell_w;
    const int32_t* lcol;      // [ell_w][n] columns: a row of the block, then kBS + its halo slot, or ~row
                              // (padding entries: the row itself, value 0)
    const int32_t* hoff;      // [nb + 1] halo of each block: rows of other blocks that its rows
    const int32_t* hrow;      //          have entries in (sorted, at most kPcgMaxHalo)
    const double* pval;       // [ell_w][n]
    const int32_t* bstart;    // [nb + 1]
    const int32_t* astart;    // [na + 1] first block of each aggregate
    const int32_t* agg_of_block;
    const int32_t* abl_off;   // [nb + 1] aggregates touching each block (sorted, own included)
    const int32_t* abl;
    const int8_t* rslot;      // [kPcgRowSlots][n], filled in order, -1 after the last
    const double* phi;        // [n][4]
    const double* rw;         // [kPcgRowSlots][4][n]
    const float* Binv;        // [nb][kBS][kBS], FP32
    const double* C0inv;      // [nc][nc]
    const double* b;          // [n][k] (block order)
    double* x;                // [n][k]
    double* U;                // [2][n][k] exchanged rows
    double* G;                // [2][nb][pcg_share_stride(k)] block sums of phi times the preconditioned vector [4][k]
    double* X;                // [3][nb][pcg_sum_stride(k)] block partial sums of the dot products [3][k]
    int* iters;
    double* relres;
    int* flags;
    double rtol;
    int maxiter;
    int block0;               // first workgroup of this problem in its launch
    int warm;                 // 1: x holds an initial guess (the previous solution)
};

// Values exchanged between workgroups carry their own arrival: a slot holds kEmpty (a NaN
// pattern no published value has) until its owner stores the value, and a reader loads the
// slot until it differs.  One trip through memory then replaces store - wait for the
// acknowledgement - flag - poll of all flags - load.  Stores and loads are 8-byte agent-scope
// relaxed atomics; a value is complete by itself, so no order between addresses is needed to
// read it.
//
// The pointers come from a table in memory, so the compiler cannot tell that they are not LDS
// addresses: through flat instructions every wait for an LDS value would wait for the loads
// from memory as well.  global() says so.
template <class T>
__device__ __forceinline__ T __attribute__((address_space(1))) * global(T* p)
{
    return (T __attribute__((address_space(1)))*)p;
}
constexpr unsigned long long kEmpty = ~0ull;
__device__ __forceinline__ void publish(double* p, double v)
{
    unsigned long long w = (unsigned long long)__double_as_longlong(v);
    if (w == kEmpty) w = 0x7FF8000000000000ull;   // any other NaN
    __hip_atomic_store(global(reinterpret_cast<unsigned long long*>(p)), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_empty(double* p)
{
    __hip_atomic_store(global(reinterpret_cast<unsigned long long*>(p)), kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const double* p)
{
    return __hip_atomic_load(global(reinterpret_cast<const unsigned long long*>(p)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double as_value(unsigned long long w) { return __longlong_as_double((long long)w); }

// Bounded wait: counts a poll round, every 256 rounds looks at the abort flag, and after
// kSpinLimit rounds raises it; true when the wait must end.
__device__ __forceinline__ bool give_up(unsigned& spins, int* flags)
{
    ++spins;
    if (spins > (unsigned)kSpinLimit) {
        __hip_atomic_store(&flags[kFlagCgAbort], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return (spins & 255u) == 0u &&
           __hip_atomic_load(&flags[kFlagCgAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Empties the exchange buffers of every problem of a launch (problem blockIdx.y).
__global__ void k_pcg_empty(const PcgArgs* __restrict__ tab, int k)
{
    const PcgArgs A = tab[blockIdx.y];
    const int64_t nu = 2 * A.n * k, ng = (int64_t)2 * A.nb * pcg_share_stride(k), nx = (int64_t)3 * A.nb * pcg_sum_stride(k);
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nu + ng + nx; i += step) {
        double* p = i < nu ? A.U + i : i < nu + ng ? A.G + (i - nu) : A.X + (i - nu - ng);
        *reinterpret_cast<unsigned long long*>(p) = kEmpty;
    }
}

// Sums of four doubles over the 64 lanes of a wave, each added exactly as wave_sum adds it
// (quads, 8, 16 lanes, then (r0 + r1) + (r2 + r3)); from the second step on the lanes halve the
// set of values they carry.  Lane l returns the sum of v[(l / 4) % 4].
__device__ __forceinline__ double wave_sum4(const double (&v)[4])
{
    double q[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        q[m] = v[m] + dpp_move<0xB1>(v[m]);    // quad_perm [1,0,3,2]
        q[m] = q[m] + dpp_move<0x4E>(q[m]);    // quad_perm [2,3,0,1]
    }
    const bool b2 = (threadIdx.x & 4) != 0, b3 = (threadIdx.x & 8) != 0;
    const double s0 = (b2 ? q[1] : q[0]) + dpp_move<0x141>(b2 ? q[0] : q[1]);   // row_half_mirror
    const double s1 = (b2 ? q[3] : q[2]) + dpp_move<0x141>(b2 ? q[2] : q[3]);
    double t = (b3 ? s1 : s0) + dpp_move<0x128>(b3 ? s0 : s1);                  // row_ror:8
    auto swap_add = [](double a, auto sw) {
        const auto lo = sw((unsigned)__double2loint(a));
        const auto hi = sw((unsigned)__double2hiint(a));
        return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    };
    t = swap_add(t, [](unsigned w) { return __builtin_amdgcn_permlane16_swap(w, w, false, false); });
    return swap_add(t, [](unsigned w) { return __builtin_amdgcn_permlane32_swap(w, w, false, false); });
}
// (a0 + a1) + (a2 + a3) of a quad's lanes, in every lane of the quad
__device__ __forceinline__ double quad_sum(double a)
{
    a = a + dpp_move<0xB1>(a);
    return a + dpp_move<0x4E>(a);
}

// sum_fixed of n values p[0 .. n), by the four lanes of a quad (a = lane % 4)
__device__ __forceinline__ double quad_sum_fixed(const double* p, int n, int a)
{
    double acc = 0.0;
    const int n4 = n & ~3;
#pragma unroll 4
    for (int i = a; i < n4; i += 4) acc += p[i];
    if (a == 0)
        for (int i = n4; i < n; ++i) acc += p[i];
    return quad_sum(acc);
}

// the same by the two lanes of a pair (h = lane % 2), in both lanes
__device__ __forceinline__ double pair_sum_fixed(const double* p, int n, int h)
{
    double a0 = 0.0, a1 = 0.0;
    const int n4 = n & ~3;
#pragma unroll 2
    for (int i = 2 * h; i < n4; i += 4) {
        a0 += p[i];
        a1 += p[i + 1];
    }
    if (h == 0)
        for (int i = n4; i < n; ++i) a0 += p[i];
    a0 += a1;
    return a0 + dpp_move<0xB1>(a0);
}

typedef float pcg_float4 __attribute__((ext_vector_type(4)));

constexpr int kPcgThreads = 512;    // 8 waves, 2 per SIMD: up to 256 VGPRs
constexpr int kRowThreads = kPcgThreads / kBS;   // threads per row: thread q takes columns q, q + 4, ...
constexpr int kParts = 256;         // partial sums of a fixed-order sum over values or blocks
constexpr int kCrowMax = 7680;      // cached coarse-inverse entries (FP32: 30 KB)
constexpr int kCache = 8;           // entries of a matrix row kept in registers
constexpr int kRS = kBS + 16;       // LDS row stride of the vector of the block product: the 4 x 16
                                    // values a wave loads at once fall into 64 different banks

template <int K>
struct PcgShared {
    static constexpr int CQ = (K + 3) / 4;   // column quads of the matrix instruction
    alignas(16) float r[CQ * 4][kRS];        // the preconditioned vector, FP32 (padding columns zero)
    alignas(16) float half[2][K][kBS];       // block product: the two halves of the inner dimension
    alignas(16) float crow[kCrowMax];        // C0inv rows of the touching aggregates' coarse functions,
                                             // rounded to FP32 (as the block inverses are), [slot][d][4]
    double rw[kPcgRegSlots * 4][kBS];        // per touched aggregate, the coarse part of a row of C
    double rho[kCoarseMax * K];              // coarse right-hand side [nc][K]
    double c[kMaxAggNbn * 4 * K];            // coarse values [slot][4][K]
    double ws[2][K][4];                      // sums over the two 64-row halves of the block
    double part[kParts];
    double coef[2][K];                       // alpha, beta of every column
    int live[K];                             // column not yet converged
    int bad;                                 // a wait gave up
    int32_t nbl[kMaxAggNbn];
    int32_t ast[kCoarseMax / 4 + 1];         // first block of each aggregate
    int32_t hrow[kPcgMaxHalo];
    double dyn[1];                           // launch-sized: [nb][3][K] partial sums of every block,
                                             // then [rows, halo][K] block solves or x
};

// LDS of a workgroup of a problem of nb blocks whose blocks keep up to halo rows of others on chip.
constexpr size_t kLdsBytes = 160 * 1024;
template <int K>
constexpr size_t pcg_lds(int nb, int halo)
{
    return sizeof(PcgShared<K>) + sizeof(double) * K * (3 * (size_t)nb + kBS + halo);
}
// The halo that fits for every number of columns: 256 rows up to 244 blocks, 220 at 256 blocks (nine
// columns).  Compact blocks of 128 vertices have about 60, blocks of a thin tube or around a pole
// of high degree more than any bound; rows beyond it are read from memory one by one.
template <int... K>
constexpr int pcg_halo_room(int nb, std::integer_sequence<int, K...>)
{
    return std::min({kPcgMaxHalo, (int)((kLdsBytes - pcg_lds<K + 1>(nb, 0)) / (sizeof(double) * (K + 1)))...});
}
int pcg_max_halo(int nb) { return pcg_halo_room(nb, std::make_integer_sequence<int, kMaxGroupCols>{}); }
static_assert(pcg_lds<kMaxGroupCols>(kMaxNbPcg, 200) <= kLdsBytes, "room for the halo of compact blocks");

// One launch solves the systems of ntab independent problems: problem m owns workgroups
// [tab[m].block0, tab[m + 1].block0) and exchanges values only among them, so its iterates
// are those of a launch of its own.
//
// What bounds it is latency: an iteration moves under 100 KB per workgroup and its arithmetic
// would take a microsecond, but it has two exchanges between all workgroups in series, and
// between them chains of sums whose order is part of the result.  So
//   - the exchanges poll the data themselves (publish / peek), in coalesced runs;
//   - eight waves share every phase: a thread owns one to three columns of a row, and the
//     fixed-order sums (four interleaved chains each) run one chain per lane;
//   - the block product runs on the matrix cores: v_mfma_f32_4x4x1 with the vector as its
//     broadcast operand (one register holds 16 terms of 4 columns, the instruction selects the
//     term), so C_BB^{-1} stays in registers, a lane per row, and a product reads 4 LDS words
//     per lane.  Its chain of multiply-adds rounds as a chain of v_fma_f32 does (checked bit
//     for bit), so the order of the terms is that of a loop over them.
//   - a block's remote neighbours are one list (its halo), fetched in whole rows of K values.
// Measured on the 40,000-face torus (157 workgroups, about 105 iterations), a solve of 3 columns
// 1.78 -> 0.98 ms, of 6 columns 2.67 -> 1.41 ms, of 9 columns 4.24 -> 1.99 ms against one
// workgroup of 256 threads per block, flags polled after the data were acknowledged and every
// column on the same thread; the iterates are the same bit for bit (all sums keep their order).
// In shader clocks per iteration, 3 columns (9): vector and shares 0.7 K (1.5), block product 1.4
// (3.0), shares in 1.8 (5.1), coarse values 3.5 (6.0), rows 3.0 (7.8), dot products out and in 4.9
// (6.9, plus 5 waiting for blocks that touch eight or more aggregates), their sums 2.3 (2.7),
// scalars 1.2 (1.4).  With 9 columns the 8-byte loads past the L2 (80 KB per workgroup and
// iteration) and the LDS reads of the rows and coarse values are the larger part.
// A row's entries beyond the first kCache come from memory again in each pass, four at a time: on a
// torus of 40,000 faces with random diagonals (degrees 4 to 8) nine columns take 2.40 ms, on the grid
// 2.36; two vertices of degree 40 among 16,002 make an iteration 1.5 times as long, of degree 200
// among 20,002 five times.
template <int K>
__global__ __launch_bounds__(kPcgThreads) void k_pcg(const PcgArgs* __restrict__ tab, int ntab)
{
    constexpr int T = kPcgThreads, Q = kRowThreads, KG = (K + Q - 1) / Q, CQ = PcgShared<K>::CQ;
    constexpr int GS = pcg_share_stride(K), XS = pcg_sum_stride(K);
    extern __shared__ __align__(16) char smem_raw[];
    PcgShared<K>& S = *reinterpret_cast<PcgShared<K>*>(smem_raw);
    int pm = 0;
    for (int m = 1; m < ntab; ++m)
        if ((int)blockIdx.x >= tab[m].block0) pm = m;
    const PcgArgs A = tab[pm];
    const int B = (int)blockIdx.x - A.block0;
    const int nb = A.nb, nc = A.nc;
    const int n = (int)A.n;
    const int32_t s0 = global(A.bstart)[B], cnt = global(A.bstart)[B + 1] - s0;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // row role: thread (row, q) owns columns q, q + Q, ... of row s0 + row (when row < cnt)
    const int row = t & (kBS - 1), my_q = wave / 2;
    const bool act = row < cnt;
    const int i = s0 + row;

    // block product role: wave (rh, jh, cq) takes rows 64 rh + lane, terms 64 jh .. of column quad cq
    const int rh = wave & 1, jh = (wave >> 1) & 1, cq = wave >> 2;
    float binv[kBS / 2];
    {
        const auto* src = global(A.Binv) + (int64_t)B * kBS * kBS + (int64_t)(64 * jh) * kBS + 64 * rh + lane;
#pragma unroll
        for (int j = 0; j < kBS / 2; ++j) binv[j] = src[(int64_t)j * kBS];
    }
    // aggregates touching this block (slots), and the rows of C0inv of their coarse functions
    const int nbo = global(A.abl_off)[B], nsl = global(A.abl_off)[B + 1] - nbo;
    for (int e = t; e < nsl; e += T) S.nbl[e] = global(A.abl)[nbo + e];
    for (int e = t; e <= nc / 4; e += T) S.ast[e] = global(A.astart)[e];
    for (int e = t; e < CQ * 4 * kRS; e += T) (&S.r[0][0])[e] = 0.0f;
    if (t == 0) S.bad = 0;
    __syncthreads();
    const int jobs = nsl * 4 * K;
    const bool crow_lds = nsl * 4 * nc <= kCrowMax;
    if (crow_lds)
        for (int e = t; e < nsl * 4 * nc; e += T) {
            const int slot = e / (4 * nc), d = (e / 4) % nc, f = e & 3;
            S.crow[e] = (float)global(A.C0inv)[(int64_t)(4 * S.nbl[slot] + f) * nc + d];
        }
    int own_slot = 0;
    {
        const int own = global(A.agg_of_block)[B];
        for (int e = 0; e < nsl; ++e)
            if (S.nbl[e] == own) own_slot = e;
    }

    // the matrix row: columns as slots of the rows in LDS, the first ones in registers.  The longest
    // row sets ell_w; a row's own entries are counted here (its padding names the row itself,
    // which is an entry once), so one vertex of high degree costs only the waves it is in.
    int32_t cj[kCache];
    double cv[kCache];
    int len = 0;
    bool edge = false;    // the row has a neighbour in another block, whose workgroup reads it
                          // (the pattern is symmetric)
#pragma unroll
    for (int e = 0; e < kCache; ++e) {
        const bool in = act && e < A.ell_w;
        cj[e] = in ? global(A.lcol)[(int64_t)e * n + i] : row;
        cv[e] = in ? global(A.pval)[(int64_t)e * n + i] : 0.0;
    }
    bool direct = false;  // the row of one of the first entries is not among the halo
    if (act) {
        int self = -1;
        for (int e = 0; e < A.ell_w; ++e) {
            const int32_t j = global(A.lcol)[(int64_t)e * n + i];
            edge = edge || j < 0 || j >= kBS;
            direct = direct || (j < 0 && e < kCache);
            if (j != row) len = e + 1;
            else if (self < 0) self = e;
        }
        len = max(len, self + 1);
    }
    // halo: rows of other blocks, [nh][K] values per exchange
    const int nh = global(A.hoff)[B + 1] - global(A.hoff)[B], nhk = nh * K;
    for (int e = t; e < nh; e += T) S.hrow[e] = global(A.hrow)[global(A.hoff)[B] + e];
    double* const stage = S.dyn;
    double* const rows = S.dyn + nb * 3 * K;

    // the row's coarse functions and, per touched aggregate, the coarse part of its row of C
    // (slots beyond kPcgRegSlots, rare, are read from memory when used)
    double phi[4];
    int rsl[kPcgRegSlots];
    int nq_row = 0;
    if (act)
        for (int e = 0; e < kPcgRowSlots; ++e) nq_row += global(A.rslot)[(int64_t)e * n + i] >= 0 ? 1 : 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) phi[a] = act ? global(A.phi)[(int64_t)i * 4 + a] : 0.0;
#pragma unroll
    for (int e = 0; e < kPcgRegSlots; ++e) rsl[e] = act ? (int)global(A.rslot)[(int64_t)e * n + i] : -1;
    for (int e = my_q; e < kPcgRegSlots * 4; e += Q)
        S.rw[e][row] = act && global(A.rslot)[(int64_t)(e / 4) * n + i] >= 0 ? global(A.rw)[(int64_t)e * n + i] : 0.0;

    // Row exchange number h uses copy h % 2 of U (and, in an iteration, of G), dot-product
    // exchange number g copy g % 3 of X; every row exchange is followed by a dot-product one,
    // in which all workgroups take part.  A slot is emptied by its owner once every reader is
    // known to be done with it, and before any reader can come for its next value: rows and
    // shares after the dot-product exchange that follows them, dot products g - 1 after exchange
    // g; these stores are waited for before the owner's next contribution to a dot-product
    // exchange, which every reader of the emptied slot has to receive first.
    int nrow = 0, nx = 0;
    auto ucopy = [&](int h) { return A.U + (int64_t)(h & 1) * n * K; };
    auto gcopy = [&](int h) { return A.G + (int64_t)(h & 1) * nb * GS; };
    auto xcopy = [&](int g) { return A.X + (int64_t)(g % 3) * nb * XS; };

    // the table entry again, for what is used rarely: read where it is needed instead of held in
    // scalar registers through the solve
    auto rare = [&]() {
        auto* p = (const PcgArgs __attribute__((address_space(4)))*)tab + pm;
        asm volatile("" : "+s"(p));
        return p;
    };
    // what the halo's element e of the exchange in U holds now
    auto halo = [&](const double* U, int e) {
        return peek(U + (unsigned)(S.hrow[e / K] * K + e % K));
    };
    // the value of column c in row j (a slot of the rows in LDS, or ~row), wherever it is
    auto value = [&](const double* U, int32_t j, int c) {
        if (j >= 0) return rows[j * K + c];
        unsigned spins = 0;
        unsigned long long w;
        while ((w = peek(U + (unsigned)(~j * K + c))) == kEmpty)
            if (give_up(spins, rare()->flags)) {
                S.bad = 1;
                break;
            }
        return as_value(w);
    };
    // coarse values: jobs (slot, f, c), f the coarse function, come in batches of up to kParts; a
    // job's nc terms are cut into P = kParts / (jobs of its batch) parts and a part into four
    // interleaved chains.  The slots whose jobs all lie in the first batch, with one or more
    // such slots' rows in LDS, take a lane per chain of kF functions; this thread's:
    constexpr int kF = K <= 6 ? 2 : 4;
    const int full = !crow_lds ? 0 : jobs <= kParts ? nsl : kParts / (4 * K);
    const int cP = jobs <= kParts ? kParts / jobs : 1, cchunk = (nc + cP - 1) / cP;
    const int last0 = (jobs - 1) / kParts * kParts, lastP = kParts / (jobs - last0);   // the last batch
    // the jobs of the other slots: n0 before the last batch (P = 1), then those in it
    const int tail = full * 4 * K, n0 = max(0, last0 - tail), tail1 = max(tail, last0);
    const int lchunk = (nc + lastP - 1) / lastP;
    const unsigned inv_lastP = ((1u << 20) + lastP - 1) / lastP;   // x / lastP = x inv_lastP >> 20 for x <= 1024
    int c_part = -1, c_first = 0, c_last = 0, c_row = 0, c_col = 0;   // S.part / S.c base, terms, S.crow, S.rho
    {
        const int a = t & 3, jc = (t >> 2) / cP, part = (t >> 2) - jc * cP;   // jc = (slot, f / kF, c)
        if (jc < full * (4 / kF) * K) {
            const int sf = jc / K, c = jc - sf * K, slot = sf / (4 / kF), f0 = (sf % (4 / kF)) * kF;
            c_part = ((slot * 4 + f0) * K + c) * cP + part;
            c_first = part * cchunk + a;
            c_last = min(nc, (part + 1) * cchunk);
            c_row = slot * nc * 4 + f0;
            c_col = c;
        }
    }

    // Thread c < K keeps the scalars of column c (|b|^2, last |r|^2, gamma, alpha, state,
    // iterations) and forms its alpha and beta; the others read them from LDS.
    const double rtol2 = A.rtol * A.rtol;
    double my_bb = 0.0, my_rr = 0.0, my_gam = 0.0, my_alpha = 0.0;
    bool my_done = false;
    int my_its = 0;
    double x[KG], r[KG], p[KG], s[KG];
#pragma unroll
    for (int ii = 0; ii < KG; ++ii) {
        const int c = my_q + ii * Q;
        r[ii] = (act && c < K) ? global(A.b)[(int64_t)i * K + c] : 0.0;
        x[ii] = p[ii] = s[ii] = 0.0;
    }
    int total_it = 0, cycle = 0;
    constexpr int kMaxRestarts = 6;
    bool have_bb = false, first = true;
    // Passes: kStep is an iteration; kVerify forms the true residual b - C x once the
    // iteration's own has converged, and another cycle starts from it when it has not; a warm
    // start forms |b|^2 as the residual of x = 0 (kZero), which fixes the tolerance, and starts
    // from the residual of the given x (kGuess).  One copy of the row product and of the
    // dot-product exchange serves them all.
    enum { kZero, kGuess, kStep, kVerify };
    int pass = A.warm ? kZero : kStep;
    __syncthreads();
    for (;;) {
        // index arithmetic is repeated in every pass rather than kept in registers across them
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        int q = my_q;
        asm volatile("" : "+s"(q));
#pragma unroll
        for (int e = 0; e < kCache; ++e) asm volatile("" : "+v"(cj[e]));
#pragma unroll
        for (int e = 0; e < kPcgRegSlots; ++e) asm volatile("" : "+v"(rsl[e]));
        const int t = tid, lane = t & 63, row = t & (kBS - 1);
        const bool step = pass == kStep;
        double y[KG];    // the rows to exchange: block solves, or x
        if (step) {
            // ---- block solves v = C_BB^{-1} r_B and shares Phi_B^T r of the coarse right-hand side
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) {
                const int c = q + ii * Q;
                if (c < K) {
                    S.r[c][row] = act ? (float)r[ii] : 0.0f;
                    double v[4];
#pragma unroll
                    for (int a = 0; a < 4; ++a) v[a] = act ? phi[a] * r[ii] : 0.0;
                    const double sum = wave_sum4(v);
                    if ((lane & 3) == 0 && lane < 16) S.ws[(row >> 6) & 1][c][lane >> 2] = sum;
                }
            }
            __syncthreads();
            if (t < 4 * K)
                publish(gcopy(nrow) + (unsigned)(B * GS + t), S.ws[0][t % K][t / K] + S.ws[1][t % K][t / K]);
            // The block solve is a preconditioner: C_BB^{-1} (FP32) times r rounded to FP32, with
            // FP32 sums (the solution's accuracy comes from the FP64 residuals; the CG iteration
            // counts equal those of an FP64 product).  Padding rows of the block hold r = 0 and an
            // identity block in C_BB^{-1}.  Row sums are taken in two halves of the terms.
            // (two column quads of a wave run as two chains side by side)
            constexpr int NQ = (CQ + T / 256 - 1) / (T / 256);   // quads per wave: cq, cq + T / 256
            if (cq < CQ) {
                float z[NQ][4];
                pcg_float4 acc[NQ];
#pragma unroll
                for (int u = 0; u < NQ; ++u) {
                    const int cc = min(cq + u * (T / 256), CQ - 1);
#pragma unroll
                    for (int m = 0; m < 4; ++m) z[u][m] = S.r[cc * 4 + (lane & 3)][64 * jh + 16 * m + (lane >> 2)];
                    acc[u] = pcg_float4{0.f, 0.f, 0.f, 0.f};
                }
#define TP_MM(M, J)                                                                                          \
    _Pragma("unroll") for (int u = 0; u < NQ; ++u)                                                           \
        acc[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(z[u][M], binv[16 * (M) + (J)], acc[u], 4, J, 0);
#define TP_MM16(M)                                                                                           \
    TP_MM(M, 0) TP_MM(M, 1) TP_MM(M, 2) TP_MM(M, 3) TP_MM(M, 4) TP_MM(M, 5) TP_MM(M, 6) TP_MM(M, 7)            \
    TP_MM(M, 8) TP_MM(M, 9) TP_MM(M, 10) TP_MM(M, 11) TP_MM(M, 12) TP_MM(M, 13) TP_MM(M, 14) TP_MM(M, 15)
                TP_MM16(0) TP_MM16(1) TP_MM16(2) TP_MM16(3)
#undef TP_MM16
#undef TP_MM
                // lane l now holds row 64 rh + l of the quads' four columns
#pragma unroll
                for (int u = 0; u < NQ; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int col = (cq + u * (T / 256)) * 4 + c;
                        if (col < K) S.half[jh][col][64 * rh + lane] = acc[u][c];
                    }
            }
            __syncthreads();
        }
        const double* U = ucopy(nrow);
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            y[ii] = x[ii];
            if (c < K) {
                if (step) y[ii] = (double)S.half[0][c][row] + (double)S.half[1][c][row];
                if (edge) publish(ucopy(nrow) + (unsigned)(i * K + c), y[ii]);
                rows[row * K + c] = y[ii];
            }
        }
        if (step) {
            // ---- coarse right-hand side [nc][K]: function 4g + a adds aggregate g's blocks in order
            // (an aggregate holds at most kMaxAggBlocks blocks)
            const double* G = gcopy(nrow);
            for (int e = t; e < nc * K; e += T) {
                const int d = e / K, c = e - d * K, b0 = S.ast[d >> 2], cb = S.ast[(d >> 2) + 1] - b0;
                const unsigned o = (unsigned)(b0 * GS + (d & 3) * K + c);
                unsigned long long raw[kMaxAggBlocks];
                unsigned spins = 0;
                for (;;) {
                    bool all = true;
#pragma unroll
                    for (int u = 0; u < kMaxAggBlocks; ++u) raw[u] = u < cb ? peek(G + o + u * GS) : 0ull;
#pragma unroll
                    for (int u = 0; u < kMaxAggBlocks; ++u) all = all && raw[u] != kEmpty;
                    if (all) break;
                    if (give_up(spins, rare()->flags)) {
                        S.bad = 1;
                        break;
                    }
                }
                double acc = 0.0;
#pragma unroll
                for (int u = 0; u < kMaxAggBlocks; ++u) acc += as_value(raw[u]);
                S.rho[e] = acc;
            }
        }
        ++nrow;
        // a first look at the halo, in flight beside the coarse values
        constexpr int NH = 2;
        unsigned long long raw[NH];
#pragma unroll
        for (int u = 0; u < NH; ++u) raw[u] = t + u * T < nhk ? halo(U, t + u * T) : 0ull;
        __syncthreads();
        if (step) {
            // ---- coarse values c[slot][f][c] = sum_d C0inv[4 nbl[slot] + f][d] rho[d][c]
            if (c_part >= 0) {
                double acc[kF];
#pragma unroll
                for (int f = 0; f < kF; ++f) acc[f] = 0.0;
                for (int d0 = c_first; d0 < c_last; d0 += 32) {
                    float w[8][kF];
                    double z[8];
#pragma unroll
                    for (int m = 0; m < 8; ++m) {
                        const int d = min(d0 + 4 * m, c_last - 1);
                        z[m] = d0 + 4 * m < c_last ? S.rho[d * K + c_col] : 0.0;
#pragma unroll
                        for (int f = 0; f < kF; ++f) w[m][f] = S.crow[c_row + 4 * d + f];
                    }
#pragma unroll
                    for (int m = 0; m < 8; ++m)
#pragma unroll
                        for (int f = 0; f < kF; ++f) acc[f] = __builtin_fma((double)w[m][f], z[m], acc[f]);
                }
                double* out = cP == 1 ? S.c : S.part;
#pragma unroll
                for (int f = 0; f < kF; ++f) {
                    const double sum = quad_sum(acc[f]);
                    if ((lane & 3) == f) out[c_part + f * K * cP] = sum;
                }
            }
            if (full < nsl) {   // the other slots' jobs, a lane per chain of one function
                const int tasks = (n0 + (jobs - tail1) * lastP) * 4;
                for (int e = T - 4 - (t & ~3) + (t & 3); e < tasks; e += T) {   // (idle waves first)
                    const bool early = e < 4 * n0;
                    const int x = (e >> 2) - n0, P = early ? 1 : lastP, chunk = early ? nc : lchunk;
                    const int xl = early ? 0 : (int)((unsigned)x * inv_lastP >> 20);
                    const int part = early ? 0 : x - xl * lastP, job = early ? tail + (e >> 2) : tail1 + xl;
                    const int fr = job / K, c = job - fr * K;   // fr = slot * 4 + f
                    const int d1 = min(nc, (part + 1) * chunk);
                    const auto* C0 = global(rare()->C0inv) + (int64_t)(4 * S.nbl[fr >> 2] + (fr & 3)) * nc;
                    const float* cr = S.crow + (fr >> 2) * 4 * nc + (fr & 3);
                    double acc = 0.0;
#pragma unroll 4
                    for (int d = part * chunk + (e & 3); d < d1; d += 4)
                        acc = __builtin_fma((double)(crow_lds ? cr[4 * d] : (float)C0[d]), S.rho[d * K + c], acc);
                    acc = quad_sum(acc);
                    if ((e & 3) == 0) (P == 1 ? S.c[job] : S.part[(job - last0) * P + part]) = acc;
                }
            }
            if (lastP > 1) {   // at most kParts / 2 jobs in the last batch: a quad per job
                __syncthreads();
                if (t < 4 * (jobs - last0)) {
                    const double sum = quad_sum_fixed(S.part + (t >> 2) * lastP, lastP, t & 3);
                    if ((t & 3) == 0) S.c[last0 + (t >> 2)] = sum;
                }
            }
        }
        // the halo's values, waited for where they were not there yet
        {
            unsigned spins = 0;
#pragma unroll
            for (int u = 0; u < NH; ++u) {
                const int e = t + u * T;
                while (raw[u] == kEmpty) {
                    if (give_up(spins, rare()->flags)) {
                        S.bad = 1;
                        break;
                    }
                    raw[u] = halo(U, e);
                }
                if (e < nhk) rows[kBS * K + e] = as_value(raw[u]);
            }
            for (int e = t + NH * T; e < nhk; e += T) {
                unsigned long long w;
                while ((w = halo(U, e)) == kEmpty)
                    if (give_up(spins, rare()->flags)) {
                        S.bad = 1;
                        break;
                    }
                rows[kBS * K + e] = as_value(w);
            }
        }
        __syncthreads();
        // ---- rows: an iteration's m = M^{-1} r = v + Phi c and an = C m = C v + (C Phi) c, or the
        // true residual; the terms of (r,m), (an,m), (r,r), or of (r,r) alone
        double m[KG], an[KG];
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) m[ii] = an[ii] = 0.0;
        // entries ea .. eb from memory, the loads of kSpan of them in flight together
        auto span = [&](int ea, int eb) {
            constexpr int kSpan = 4;
            for (int e0 = ea; e0 < eb; e0 += kSpan) {
                int32_t j[kSpan];
                double a[kSpan];
#pragma unroll
                for (int u = 0; u < kSpan; ++u) {
                    const int64_t at = (int64_t)min(e0 + u, eb - 1) * n + i;
                    j[u] = global(rare()->lcol)[at];
                    a[u] = global(rare()->pval)[at];
                }
#pragma unroll
                for (int u = 0; u < kSpan; ++u)
                    if (e0 + u < eb)
#pragma unroll
                        for (int ii = 0; ii < KG; ++ii)
                            if (q + ii * Q < K) an[ii] = __builtin_fma(a[u], value(U, j[u], q + ii * Q), an[ii]);
            }
        };
        if (!direct) {
#pragma unroll
            for (int e = 0; e < kCache; ++e)
#pragma unroll
                for (int ii = 0; ii < KG; ++ii)
                    if (q + ii * Q < K) an[ii] = __builtin_fma(cv[e], rows[cj[e] * K + q + ii * Q], an[ii]);
        } else {
            span(0, min(kCache, len));
        }
        if (step) {
#pragma unroll
            for (int ii = 0; ii < KG; ++ii)
                if (q + ii * Q < K) {
                    double cm = 0.0;
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        cm = __builtin_fma(phi[a], S.c[(own_slot * 4 + a) * K + q + ii * Q], cm);
                    m[ii] = y[ii] + cm;
                }
#pragma unroll
            for (int e = 0; e < kPcgRegSlots; ++e)
                if (rsl[e] >= 0)
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const double w = S.rw[e * 4 + a][row];
#pragma unroll
                        for (int ii = 0; ii < KG; ++ii)
                            if (q + ii * Q < K) an[ii] = __builtin_fma(w, S.c[(rsl[e] * 4 + a) * K + q + ii * Q], an[ii]);
                    }
            for (int e = kPcgRegSlots; e < nq_row; ++e) {   // slots are filled in order
                const int sl = global(rare()->rslot)[(int64_t)e * n + i];
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const double w = global(rare()->rw)[((int64_t)e * 4 + a) * n + i];
#pragma unroll
                    for (int ii = 0; ii < KG; ++ii)
                        if (q + ii * Q < K) an[ii] = __builtin_fma(w, S.c[(sl * 4 + a) * K + q + ii * Q], an[ii]);
                }
            }
        }
        span(kCache, len);   // (their coarse part is in rw)
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            if (c < K) {
                if (!step) r[ii] = act ? global(rare()->b)[(int64_t)i * K + c] - an[ii] : 0.0;
                double d[4] = {r[ii] * m[ii], an[ii] * m[ii], r[ii] * r[ii], 0.0};
                if (!step) d[0] = d[2];
#pragma unroll
                for (int g = 0; g < 3; ++g) d[g] = act ? d[g] : 0.0;
                const double sum = wave_sum4(d);
                if ((lane & 3) == 0 && lane < 16) S.ws[(row >> 6) & 1][c][lane >> 2] = sum;
            }
        }
        // ---- dot-product exchange of M values per block (3 K, or K for a residual)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the emptied slots are stored before the sums below
        __syncthreads();
        double* X = xcopy(nx);
        ++nx;
        if (t < (step ? 3 * K : K)) publish(X + (unsigned)(B * XS + t), S.ws[0][t % K][t / K] + S.ws[1][t % K][t / K]);
        constexpr int NL = K <= 3 ? 3 : K <= 6 ? 6 : 9;
        for (int e0 = t; e0 < nb * 3 * K; e0 += NL * T) {
            unsigned long long w[NL];
            unsigned spins = 0;
            for (;;) {
                bool all = true;
#pragma unroll
                for (int u = 0; u < NL; ++u) {
                    const int e = e0 + u * T, b = e / (3 * K), v = e - b * 3 * K;
                    w[u] = b < nb && (step || v < K) ? peek(X + (unsigned)(b * XS + v)) : 0ull;
                }
#pragma unroll
                for (int u = 0; u < NL; ++u) all = all && w[u] != kEmpty;
                if (all) break;
                if (give_up(spins, rare()->flags)) {
                    S.bad = 1;
                    break;
                }
            }
#pragma unroll
            for (int u = 0; u < NL; ++u)
                if (e0 + u * T < nb * 3 * K) stage[e0 + u * T] = as_value(w[u]);
        }
        __syncthreads();
        if (S.bad) return;
        // Each value's nb partial sums are cut into P parts of consecutive blocks and a part into
        // four interleaved chains, one per lane; chains are added as (a0 + a1) + (a2 + a3).
        auto block_sums = [&](auto mtag) {
            constexpr int M = decltype(mtag)::value, P = kParts / M, NB = ((kMaxNbPcg + P - 1) / P + 3) / 4;
            const int chunk = (nb + P - 1) / P;
#pragma unroll
            for (int h = 0; h < (M * P * 4 + T - 1) / T; ++h) {
                const int e = t + h * T;
                const int v = (e >> 2) / P, part = (e >> 2) - v * P, b0 = part * chunk + (e & 3);
                const int b1 = e < M * P * 4 ? min(nb, (part + 1) * chunk) : 0;
                double z[NB], acc = 0.0;
#pragma unroll
                for (int u = 0; u < NB; ++u) z[u] = b0 + 4 * u < b1 ? stage[(b0 + 4 * u) * 3 * K + v] : 0.0;
#pragma unroll
                for (int u = 0; u < NB; ++u) acc += z[u];
                acc = quad_sum(acc);
                if (e < M * P * 4 && (e & 3) == 0) S.part[v * P + part] = acc;
            }
        };
        if (step) block_sums(std::integral_constant<int, 3 * K>{});
        else block_sums(std::integral_constant<int, K>{});
        __syncthreads();
        const bool can = total_it < A.maxiter;
        if (t < 64) {
            // the parts of a value, added by a quad or (to stay within one wave) a pair of lanes
            constexpr int W = K <= 5 ? 4 : 2;
            const int P = step ? kParts / (3 * K) : kParts / K, v = lane / W;
            double sum = 0.0;
            if (v < (step ? 3 * K : K))
                sum = W == 4 ? quad_sum_fixed(S.part + v * P, P, lane & 3) : pair_sum_fixed(S.part + v * P, P, lane & 1);
            const int c = t % K;
            const double g = __shfl(sum, W * c), dd = __shfl(sum, W * (K + c)), rr = __shfl(sum, W * (2 * K + c));
            if (t < K && !step) {
                if (pass != kVerify || !my_done) my_rr = g;
                if (pass == kZero) {
                    my_bb = my_rr;
                    my_done = !(my_bb > 0.0);
                }
                if (pass == kVerify && !my_done && my_rr <= rtol2 * my_bb) my_done = true;
                S.live[t] = my_done ? 0 : 1;
            }
            if (t < K && step) {
                my_rr = rr;
                if (!have_bb) {
                    my_bb = my_rr;
                    my_done = !(my_bb > 0.0);
                }
                double al = 0.0, be = 0.0;
                const bool live = !my_done && my_rr > rtol2 * my_bb;
                if (live) {
                    if (can) {
                        if (first) {
                            al = g / dd;
                        } else {
                            be = g / my_gam;
                            al = g / (dd - be * g / my_alpha);
                        }
                        my_its = total_it + 1;
                    }
                    my_gam = g;
                    my_alpha = al;
                }
                S.coef[0][t] = al;
                S.coef[1][t] = be;
                S.live[t] = live ? 1 : 0;
            }
        }
        have_bb = true;
        // everyone has published this exchange, so no one still reads the rows and shares before
        // it, or the dot products of the exchange before it
        if (edge)
#pragma unroll
            for (int ii = 0; ii < KG; ++ii)
                if (q + ii * Q < K) publish_empty(ucopy(nrow - 1) + (unsigned)(i * K + q + ii * Q));
        if (t < 4 * K) publish_empty(gcopy(nrow - 1) + (unsigned)(B * GS + t));
        if (t < 3 * K) publish_empty(xcopy(nx + 1) + (unsigned)(B * XS + t));
        __syncthreads();
        bool conv = true;
#pragma unroll
        for (int c = 0; c < K; ++c) conv = conv && S.live[c] == 0;
        if (step) {
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) {
                const int c = q + ii * Q;
                if (c < K) {
                    // columns that converged (or are done) have alpha = 0: x and r stay
                    const double al = S.coef[0][c], be = S.coef[1][c];
                    p[ii] = __builtin_fma(be, p[ii], m[ii]);
                    s[ii] = __builtin_fma(be, s[ii], an[ii]);
                    x[ii] = __builtin_fma(al, p[ii], x[ii]);
                    r[ii] = __builtin_fma(-al, s[ii], r[ii]);
                }
            }
            if (conv || !can) {
                pass = kVerify;
            } else {
                ++total_it;
                first = false;
            }
        } else if (pass == kZero) {
            pass = kGuess;
#pragma unroll
            for (int ii = 0; ii < KG; ++ii)
                if (act && q + ii * Q < K) x[ii] = global(rare()->x)[(int64_t)i * K + q + ii * Q];
        } else {
            if (pass == kVerify) {
                if (conv || total_it >= A.maxiter || cycle == kMaxRestarts) break;
                ++cycle;
            }
            // a cycle starts from the current (true) residual r
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) p[ii] = s[ii] = 0.0;
            pass = kStep;
            first = true;
        }
    }
    if (act)
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = my_q + ii * Q;
            if (c < K) global(rare()->x)[(int64_t)i * K + c] = x[ii];
        }
    if (B == 0 && t < K) {
        global(rare()->iters)[t] = my_its;
        global(rare()->relres)[t] = my_bb > 0.0 ? sqrt(my_rr / my_bb) : 0.0;
    }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_pcg_setup(const PcgSetup& ps, const double* V, const int32_t* lap_off, const double* lap_val,
                            hipStream_t s)
{
    hipLaunchKernelGGL(k_perm_ell_vals, dim3((unsigned)((ps.n + 255) / 256)), dim3(256), 0, s,
                       ps.n, ps.ell_w, ps.perm, lap_off, lap_val, ps.pval);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // coarse functions, their rows of C and the Galerkin matrix; then both inverses
    hipLaunchKernelGGL(k_agg_basis, dim3(ps.na), dim3(kAggThreads), 0, s, ps.perm, V, ps.astart, ps.bstart, ps.phi,
                       ps.esum);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_row_coarse, dim3((unsigned)((ps.n + 255) / 256)), dim3(256), 0, s, ps.n, ps.ell_w, ps.pcol,
                       ps.pval, ps.eslot, ps.phi, ps.rw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t asm_smem = sizeof(double) * kAsmGroups * (size_t)ps.na * 16;
    e = hipFuncSetAttribute((const void*)k_coarse_assemble, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(sizeof(double) * kAsmGroups * (kCoarseMax / 4) * 16));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_coarse_assemble, dim3(ps.na), dim3(kAggThreads), asm_smem, s, ps.n, ps.na, ps.nc,
                       ps.astart, ps.bstart, ps.blk, ps.abl_off, ps.abl, ps.rslot, ps.phi, ps.rw, ps.C0inv);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t binv_smem = sizeof(double) * kBS * kBS;
    e = hipFuncSetAttribute((const void*)k_inverses, hipFuncAttributeMaxDynamicSharedMemorySize, (int)binv_smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_inverses, dim3(ps.nb + 1), dim3(kInvThreads), binv_smem, s, ps.nb, ps.n, ps.ell_w, ps.pcol,
                       ps.pval, ps.bstart, ps.whole, ps.Binv, ps.nc, ps.acomp, ps.esum, ps.C0inv);
    return hipGetLastError();
}

hipError_t launch_permute_rows(const PermJob* jobs, int njobs, int k, int ld, int c0, bool forward, hipStream_t s)
{
    for (int m0 = 0; m0 < njobs; m0 += kMaxVecJobs) {
        PermJobs jb;
        const int n = std::min(kMaxVecJobs, njobs - m0);
        int64_t most = 1;
        for (int q = 0; q < n; ++q) {
            jb.j[q] = jobs[m0 + q];
            most = std::max(most, jb.j[q].n);
        }
        hipLaunchKernelGGL(k_permute_rows, dim3((unsigned)((most * k + 255) / 256), n), dim3(256), 0, s, jb, k, ld, c0,
                           forward ? 1 : 0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {

struct PcgKernel {
    const void* fn;
    size_t smem;         // without the rows and halo
};

PcgKernel pcg_kernel(int k)
{
    switch (k) {
    case 1: return {(const void*)k_pcg<1>, sizeof(PcgShared<1>)};
    case 2: return {(const void*)k_pcg<2>, sizeof(PcgShared<2>)};
    case 3: return {(const void*)k_pcg<3>, sizeof(PcgShared<3>)};
    case 4: return {(const void*)k_pcg<4>, sizeof(PcgShared<4>)};
    case 5: return {(const void*)k_pcg<5>, sizeof(PcgShared<5>)};
    case 6: return {(const void*)k_pcg<6>, sizeof(PcgShared<6>)};
    case 7: return {(const void*)k_pcg<7>, sizeof(PcgShared<7>)};
    case 8: return {(const void*)k_pcg<8>, sizeof(PcgShared<8>)};
    case 9: return {(const void*)k_pcg<9>, sizeof(PcgShared<9>)};
    default: return {nullptr, 0};
    }
}

}  // namespace

int pcg_block_size() { return kBS; }
int pcg_max_blocks() { return kMaxNbPcg; }
int pcg_max_coarse() { return kCoarseMax; }
int pcg_max_block_aggregates() { return kMaxAggNbn; }
size_t pcg_table_bytes(int n) { return sizeof(PcgArgs) * (size_t)std::max(n, 1); }

hipError_t launch_pcg_batch(const PcgItem* items, int n, int k, void* tab_dev, void* tab_host,
                            hipStream_t s)
{
    if (n < 1) return hipSuccess;
    const PcgKernel kern = pcg_kernel(k);
    const void* fn = kern.fn;
    if (!fn) return hipErrorInvalidValue;
    // (each problem's own blocks and halo: the largest of each, taken apart, may not fit together)
    size_t rows = 0;
    for (int m = 0; m < n; ++m) rows = std::max(rows, 3 * (size_t)items[m].ps->nb + kBS + items[m].ps->max_halo);
    const size_t smem = kern.smem + sizeof(double) * rows * (size_t)k;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kPcgThreads, smem);
    if (e != hipSuccess) return e;
    const int64_t cap = (int64_t)per_cu * device_info().num_cu;
    PcgArgs* H = static_cast<PcgArgs*>(tab_host);
    for (int m = 0; m < n; ++m) {
        const PcgItem& it = items[m];
        const PcgSetup& ps = *it.ps;
        PcgArgs& a = H[m];
        a.n = ps.n; a.nb = ps.nb; a.nc = ps.nc; a.ell_w = ps.ell_w; a.pval = ps.pval;
        a.lcol = ps.lcol; a.hoff = ps.hoff; a.hrow = ps.hrow;
        a.bstart = ps.bstart; a.astart = ps.astart; a.agg_of_block = ps.agg_of_block; a.abl_off = ps.abl_off;
        a.abl = ps.abl; a.rslot = ps.rslot; a.phi = ps.phi; a.rw = ps.rw; a.Binv = ps.Binv; a.C0inv = ps.C0inv;
        a.b = it.b; a.x = it.x; a.U = it.w.U; a.G = it.w.G; a.X = it.w.X;
        a.iters = it.w.iters; a.relres = it.w.relres; a.flags = it.w.flags;
        a.rtol = it.rtol; a.maxiter = it.maxiter; a.block0 = 0;
        a.warm = it.warm ? 1 : 0;
        if ((int64_t)ps.nb > cap) return hipErrorCooperativeLaunchTooLarge;
    }
    // launches of consecutive problems whose workgroups are resident together
    std::vector<std::pair<int, int>> groups;
    for (int i0 = 0; i0 < n;) {
        int64_t sum = 0;
        int i1 = i0;
        while (i1 < n && sum + H[i1].nb <= cap) {
            H[i1].block0 = (int)sum;
            sum += H[i1].nb;
            ++i1;
        }
        groups.emplace_back(i0, i1);
        i0 = i1;
    }
    e = hipMemcpyAsync(tab_dev, tab_host, sizeof(PcgArgs) * n, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pcg_empty, dim3(64, (unsigned)n), dim3(256), 0, s, static_cast<const PcgArgs*>(tab_dev), k);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (const auto& g : groups) {
        const PcgArgs* t = static_cast<const PcgArgs*>(tab_dev) + g.first;
        int nt = g.second - g.first;
        int blocks = 0;
        for (int m = g.first; m < g.second; ++m) blocks += H[m].nb;
        void* params[] = {(void*)&t, (void*)&nt};
        e = hipLaunchCooperativeKernel(fn, dim3(blocks), dim3(kPcgThreads), params, (unsigned)smem, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}


// ---------------------------------------------------------------- wide solve
//
// Problems of more blocks than workgroups that can be resident at once, but no more than a few
// per workgroup: a persistent kernel with NBK blocks in each.

namespace {

struct WideArgs {
    int64_t n;
    int nb, nc, ell_w;
    const int32_t* pcol;      // [ell_w][n] (padding entries: the row itself, value 0)
    const double* pval;       // [ell_w][n]
    const int32_t* toff;      // [n + 1] the rows' entries beyond the first kWideCache (when some row has any)
    int32_t* tslot;           // [toff[n]] their columns as slots
    const int32_t* bstart;    // [nb + 1]
    const int32_t* blk;       // [n] block of each row
    const int32_t* agg_of_block;
    const double* phi;        // [n][4]
    const float* Binv;        // [nb][kBS][kBS], FP32
    const double* C0inv;      // [nc][nc]
    const double* b;          // [n][ld] (block order)
    double* x;                // [n][ld]
    int ld;
    double* U0;               // [n][k] row values of the neighbour exchanges, two copies
    double* U1;
    double* X;                // [3][entries][k][kWideSum] sums of the all-to-all exchanges
    int* iters;
    double* relres;
    int* flags;
    double rtol;
    int maxiter;
};

typedef float wide_float4 __attribute__((ext_vector_type(4)));
constexpr int kWideCols = 3;          // columns at most: what the registers of a workgroup hold
constexpr int kWideThreads = 512;     // per workgroup: 256 registers each, 64 NBK / 2 of them for the inverses
constexpr double kFresh = 1e-4;       // fall of |r| after which the coarse values are formed anew
constexpr int kWideSum = 8;           // doubles of a record of the all-to-all exchange (seven used)
constexpr int kWideCache = kPcgWideCache;   // entries of a matrix row kept in LDS
constexpr int kWideTail = 32;         // entries beyond them that a thread takes by itself
constexpr int kWideEntries = kMaxBarrierW + kCoarseMax / 4;   // records: one per workgroup and one more per aggregate

template <int K, int NBK>
struct WideDims {
    static constexpr int T = kWideThreads;
    static constexpr int R = kBS * NBK;              // rows per workgroup
    static constexpr int Q = T / R;                  // threads per row: thread q takes columns q, q + Q, ...
    static constexpr int KG = (K + Q - 1) / Q;       // columns per thread
    static constexpr int NW = T / 64;                // waves
    static constexpr int UN = R / 64;                // 64-row units of the block product
    static constexpr int SEG = NW / UN;              // parts of its inner dimension
    static constexpr int JS = kBS / SEG;             // terms per part
    static constexpr int P = NW / K;                 // waves per column in the all-to-all exchange
    static constexpr int RS = R + 4;                 // LDS row stride (floats): quads of columns miss each other's banks
    static constexpr int XE = 144 * NBK;             // entries in rows of other workgroups, kept in LDS
    static constexpr int MB = NBK == 2 ? 8 : 4;   // records per lane with their loads in flight together
    static_assert(K <= 4 && NW >= K && SEG >= 1, "one quad of columns, a wave per column, a wave per unit");
};

template <int K, int NBK>
struct WideShared {
    using D = WideDims<K, NBK>;
    union {
        struct {
            alignas(16) float r[4][D::RS];            // residual rounded to FP32 (columns from K on are not used)
            alignas(16) float part[D::SEG][K][D::RS]; // block product by parts of its inner dimension
        };
        double ext[K][D::XE];                         // u (or x) of the rows of other workgroups
    };
    int32_t xrow[D::XE];                              // which rows
    int nx;
    double u[K][D::R];                                // M^{-1} r (or x) of the own rows
    double x[K][D::R], p[K][D::R], s[K][D::R];
    double ws[NBK][2][K][8];                          // sums of the two 64-row halves of a block
    double xp[K][D::P][NBK][8];                       // all-to-all sums by wave (0-2: products, 3-6: coarse)
    double coef[2][K];                                // alpha, beta of every column
    double cval[NBK][4][K];                           // coarse values of the own aggregates
    double crow[NBK][kCoarseMax / 4][16];             // their rows of C0^{-1}, by aggregate
    int live[K];                                      // column not yet converged; 2: with its coarse values
                                                      // to be formed anew
    int bad;                                          // a wait gave up
    int wcount[D::NW], e0, ne;                        // records: this workgroup's first, all
    int la[NBK];                                      // own aggregate of each own block
    uint8_t eagg[kWideEntries];                       // aggregate of each record
    double cv[kWideCache][D::R];                      // matrix rows and coarse functions
    int32_t cj[kWideCache][D::R];
    double phi[4][D::R];
};

__global__ void k_wide_empty(WideArgs A, int k)
{
    const int64_t nu = A.n * k, nx = (int64_t)3 * kWideEntries * k * kWideSum;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2 * nu + nx; i += step) {
        double* p = i < nu ? A.U0 + i : i < 2 * nu ? A.U1 + (i - nu) : A.X + (i - 2 * nu);
        *reinterpret_cast<unsigned long long*>(p) = kEmpty;
    }
}

// What bounds it: two exchanges between workgroups in series per iteration, and the block product
// and rows of NBK blocks between them.  The five launches per iteration of the multi-launch solve
// read 51 MB of inverses and 40 MB of vectors again each time (782 blocks); here everything that
// an iteration reads stays on chip: the inverses in registers (a lane's register is its row of the
// 4 x 4 x 1 matrix tiles), matrix rows, coarse functions and the own rows of C0^{-1} in LDS, the
// iteration's vectors in registers.  The coarse solve costs no exchange of its own: the shares
// Phi^T (C u) ride with the dot products, every workgroup multiplies them by the rows of C0^{-1}
// of its own aggregates while it adds the dot products, and the coarse values of the new residual
// follow by the recurrence of the residual itself (c -= alpha C0^{-1} Phi^T s), restarted from the
// true residual with it; then u = M^{-1} r is known before the first exchange, which passes
// boundary values to neighbouring blocks only.  The recurrence's rounding stays as large as it was
// where c was, while r shrinks: by itself it held three columns of 100,002 vertices at a relative
// residual of 2e-12, whatever the tolerance.  So c is formed from r anew, by one more all-to-all
// exchange, whenever |r| has fallen to kFresh of what it was (two of 187 iterations' exchanges at
// 1e-10).  A workgroup's blocks in one aggregate are one
// record of the all-to-all exchange, so what it polls does not grow with NBK.
// Three columns of 100,002 vertices (782 blocks, 185 iterations): 7.8 ms in five launches per
// iteration (42 us), 2.8 ms here (15 us); one column 6.9 and 1.5 ms.  1,024 threads with two columns
// each spill (133 registers).  A record read by one lane in seven loads instead of by eight lanes
// in one: 3.5 ms, because each load of a lane is a request of its own to the coherence point.
//
// A row's entries beyond the first kWideCache (TAIL: some row has any) come from memory in each
// product, four at a time in a thread, a row of more than kWideTail of them by the wave.  Nine
// columns on a globe of 36,102 vertices with two poles of degree 190: 36.8 us an iteration; 993
// when every row walked as many entries as the longest has and formed their slots again, 158 in five
// launches; 32.8 on a torus grid of as many vertices.
template <int K, int NBK, bool TAIL>
__global__ __launch_bounds__((WideDims<K, NBK>::T)) void k_pcg_wide(WideArgs A)
{
    using D = WideDims<K, NBK>;
    constexpr int R = D::R, Q = D::Q, KG = D::KG, P = D::P, MB = D::MB;
    extern __shared__ __align__(16) char smem_raw[];
    WideShared<K, NBK>& S = *reinterpret_cast<WideShared<K, NBK>*>(smem_raw);
    const int B0 = (int)blockIdx.x * NBK;                   // first block of the workgroup
    const int nb = A.nb, nc = A.nc;
    const int nown = min(NBK, nb - B0);                     // its blocks
    const int64_t n = A.n;
    int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // row role: thread (row, q) owns columns q, q + Q, ... of a row; waves share q and block
    int row = t & (R - 1);
    const int q = wave / (R / 64), lb = wave % (R / 64) / 2;
    const bool has = lb < nown;
    const int32_t s0 = has ? A.bstart[B0 + lb] : 0;
    const int32_t cnt = has ? A.bstart[B0 + lb + 1] - s0 : 0;
    const bool act = (row & (kBS - 1)) < cnt;
    int i = s0 + (row & (kBS - 1));

    // block product role: wave (unit, seg) takes rows 64 unit + lane and terms seg JS ..
    const int unit = wave % D::UN, seg = wave / D::UN;
    float binv[D::JS];
    {
        const int ub = unit / 2;
        const float* src = A.Binv + (int64_t)(B0 + (ub < nown ? ub : 0)) * kBS * kBS + (unit & 1) * 64 + lane;
#pragma unroll
        for (int j = 0; j < D::JS; ++j) binv[j] = src[(int64_t)(seg * D::JS + j) * kBS];
    }
    // matrix rows: columns of the workgroup's own rows as LDS slots (>= 0), others as ~row
    auto slot_of = [&](int32_t j) -> int32_t {
        const int jb = A.blk[j] - B0;
        return jb >= 0 && jb < nown ? jb * kBS + (j - A.bstart[B0 + jb]) : ~j;
    };
    bool edge = false;    // the row is read by another workgroup (the pattern is symmetric)
    if (t == 0) S.nx = 0;
    __syncthreads();
    auto place = [&](int32_t sl) -> int32_t {               // R + the value's place in ext, when there is room
        if (sl >= 0) return sl;
        const int at = atomicAdd(&S.nx, 1);
        if (at >= D::XE) return sl;
        S.xrow[at] = ~sl;
        return R + at;
    };
#pragma unroll
    for (int e = 0; e < kWideCache; ++e) {
        const bool in = act && e < A.ell_w;
        const int32_t sl = in ? slot_of(A.pcol[(int64_t)e * n + i]) : row;
        const double v = in ? A.pval[(int64_t)e * n + i] : 0.0;
        edge = edge || sl < 0;
        if (q == 0) {
            S.cj[e][row] = place(sl);
            S.cv[e][row] = v;
        }
    }
    // the row's own entries beyond them (the longest row sets ell_w): slots formed here, once
    const int t0 = TAIL && act ? A.toff[i] : 0, tn = TAIL && act ? A.toff[i + 1] - t0 : 0;
    for (int e = 0; e < tn; ++e) {
        const int32_t sl = slot_of(A.pcol[(int64_t)(kWideCache + e) * n + i]);
        edge = edge || sl < 0;
        if (q == 0) A.tslot[t0 + e] = place(sl);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const double v = act ? A.phi[i * 4 + a] : 0.0;
        if (q == 0) S.phi[a][row] = v;
    }
    // coarse data: the own blocks' aggregates are consecutive numbers from A0
    const int A0 = A.agg_of_block[B0];
    const int nloc = A.agg_of_block[B0 + nown - 1] - A0 + 1;
    const int my_la = has ? A.agg_of_block[B0 + lb] - A0 : 0;
    if (t < NBK) S.la[t] = t < nown ? A.agg_of_block[B0 + t] - A0 : -1;
    for (int e = t; e < nloc * (nc / 4) * 16; e += D::T) {
        const int la = e / (nc * 4), g = (e / 16) % (nc / 4), a = (e / 4) & 3, a2 = e & 3;
        S.crow[la][g][a * 4 + a2] = A.C0inv[(int64_t)(4 * (A0 + la) + a) * nc + 4 * g + a2];
    }
    // entries of the all-to-all exchange: the blocks of one workgroup in one aggregate, in block order
    for (int b0 = 0, before = 0; b0 < nb; b0 += D::T) {
        const int b = b0 + t;
        const bool starts = b < nb && (b % NBK == 0 || A.agg_of_block[b] != A.agg_of_block[b - 1]);
        const unsigned long long m = __ballot(starts);
        if (lane == 0) S.wcount[wave] = __builtin_popcountll(m);
        __syncthreads();
        int id = before + __builtin_popcountll(m & ((1ull << lane) - 1ull));
        for (int v = 0; v < D::NW; ++v) {
            if (v < wave) id += S.wcount[v];
            before += S.wcount[v];
        }
        if (starts) S.eagg[id] = (uint8_t)A.agg_of_block[b];
        if (b == B0) S.e0 = id;
        if (t == 0) S.ne = before;
        __syncthreads();
    }
    if (t == 0) S.bad = 0;
    __syncthreads();
    const int e0 = S.e0, ne = S.ne;

    // Neighbour exchange number h uses copy h % 2 of U, all-to-all exchange number g copy g % 3
    // of X; every neighbour exchange is followed by an all-to-all one.  A slot is emptied by its
    // owner after every reader is known to be done with it and before any reader can come for
    // its next value: rows after the all-to-all exchange that follows them (every workgroup
    // took part in it after reading), sums of exchange g - 2 after exchange g - 1, and both
    // stores are waited for before the owner's next contribution to an all-to-all exchange.
    int nhalo = 0, nx = 0;
    auto ucopy = [&](int h) { return h & 1 ? A.U1 : A.U0; };
    auto xcopy = [&](int g) { return A.X + (int64_t)(g % 3) * ne * K * kWideSum; };
    auto empty_rows = [&]() {    // of the neighbour exchange before
        if (nhalo > 0 && edge) {
            double* U = ucopy(nhalo - 1);
#pragma unroll
            for (int ii = 0; ii < KG; ++ii)
                if (q + ii * Q < K) publish_empty(U + i * K + q + ii * Q);
        }
    };

    // w = C u for the vector u of the own rows in registers: shares it, polls the neighbours'
    auto product = [&](const double (&u)[KG], double (&w)[KG]) {
        double* U = ucopy(nhalo);
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            if (c < K) {
                if (edge) publish(U + i * K + c, u[ii]);
                S.u[c][row] = act ? u[ii] : 0.0;
            }
        }
        __syncthreads();
        ++nhalo;
        bool fail = false;
        auto wait_for = [&](int32_t j, int c) -> double {
            unsigned spins = 0;
            unsigned long long v = peek(U + (unsigned)(j * K + c));
            while (v == kEmpty && !fail) {
                v = peek(U + (unsigned)(j * K + c));
                fail = give_up(spins, A.flags);
            }
            return as_value(v);
        };
        auto value = [&](int32_t j, int c) -> double {
            return j < 0 ? wait_for(~j, c) : *(j < R ? &S.u[c][j] : &S.ext[c][j - R]);
        };
        const int nx = min(S.nx, D::XE) * K;
        constexpr int PX = 4;             // values per thread with their loads in flight together
        for (int f0 = t; f0 < nx && !fail; f0 += PX * D::T) {
            unsigned long long raw[PX];
            unsigned spins = 0;
            for (;;) {
                bool wait = false;
#pragma unroll
                for (int m = 0; m < PX; ++m) {
                    const int f = f0 + m * D::T;
                    raw[m] = f < nx ? peek(U + (unsigned)(S.xrow[f / K] * K + f % K)) : 0ull;
                }
#pragma unroll
                for (int m = 0; m < PX; ++m) wait = wait || raw[m] == kEmpty;
                if (!wait) break;
                if (give_up(spins, A.flags)) {
                    fail = true;
                    break;
                }
            }
#pragma unroll
            for (int m = 0; m < PX; ++m) {
                const int f = f0 + m * D::T;
                if (f < nx) S.ext[f % K][f / K] = as_value(raw[m]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            double acc = 0.0;
            if (c < K) {
#pragma unroll
                for (int e = 0; e < kWideCache; ++e) {
                    acc += S.cv[e][row] * value(S.cj[e][row], c);
                }
            }
            w[ii] = acc;
        }
        if (TAIL && tn > 0 && tn <= kWideTail) {
            constexpr int UT = 4;             // entries with their loads in flight together
            for (int e0 = 0; e0 < tn; e0 += UT) {
                int32_t j[UT];
                double a[UT];
#pragma unroll
                for (int m = 0; m < UT; ++m) {
                    const int e = min(e0 + m, tn - 1);
                    j[m] = A.tslot[t0 + e];
                    a[m] = A.pval[(int64_t)(kWideCache + e) * n + i];
                }
#pragma unroll
                for (int m = 0; m < UT; ++m)
                    if (e0 + m < tn)
#pragma unroll
                        for (int ii = 0; ii < KG; ++ii)
                            if (q + ii * Q < K) w[ii] += a[m] * value(j[m], q + ii * Q);
            }
        }
        for (unsigned long long ml = TAIL ? __ballot(tn > kWideTail) : 0; ml; ml &= ml - 1) {   // the wave together
            const int l = __builtin_ctzll(ml);
            const int lt0 = __builtin_amdgcn_readlane(t0, l), ltn = __builtin_amdgcn_readlane(tn, l);
            const int li = __builtin_amdgcn_readlane(i, l);
            double sum[KG];
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) sum[ii] = 0.0;
            for (int e = lane; e < ltn; e += 64) {
                const int32_t j = A.tslot[lt0 + e];
                const double a = A.pval[(int64_t)(kWideCache + e) * n + li];
#pragma unroll
                for (int ii = 0; ii < KG; ++ii)
                    if (q + ii * Q < K) sum[ii] += a * value(j, q + ii * Q);
            }
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) {
                const double all = wave_sum(sum[ii]);
                if (lane == l) w[ii] += all;
            }
        }
        if (fail) S.bad = 1;
    };

    // All-to-all exchange of the sums of r u, w u, r r and phi[a] w over every block's rows:
    // afterwards S.xp holds, by wave, the sums of the three products and of the rows of
    // C0^{-1} of the own aggregates times the shares Phi^T w.  False when a wait gave up.
    auto exchange = [&](const double (&r)[KG], const double (&u)[KG], const double (&w)[KG]) -> bool {
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            if (c < K) {
                double v[8] = {r[ii] * u[ii], w[ii] * u[ii], r[ii] * r[ii], 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int a = 0; a < 4; ++a) v[3 + a] = S.phi[a][row] * w[ii];
                if (!act)
#pragma unroll
                    for (int m = 0; m < 7; ++m) v[m] = 0.0;
                const double sum = wave_sum8(v);
                if ((lane & 7) == 0) S.ws[lb][(row >> 6) & 1][c][lane >> 3] = sum;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the emptied slots are stored before the sums below
        __syncthreads();
        double* X = xcopy(nx);
        if (t < nloc * K * 7) {
            const int la = t / (K * 7), c = (t / 7) % K, m = t % 7;
            double sum = 0.0;
            for (int l = 0; l < nown; ++l)
                if (S.la[l] == la) sum += S.ws[l][0][c][m] + S.ws[l][1][c][m];
            publish(X + ((int64_t)(e0 + la) * K + c) * kWideSum + m, sum);
        }
        ++nx;
        bool fail = false;
        const int c = wave % K, part = wave / K;
        if (part < P) {
            // eight lanes read a record together (one request each; a lane that reads a record alone
            // makes seven): lane v of them value v
            const int v = lane & 7;
            double d = 0.0, cw[NBK][4];
#pragma unroll
            for (int l = 0; l < NBK; ++l)
#pragma unroll
                for (int a = 0; a < 4; ++a) cw[l][a] = 0.0;
            for (int b0 = (lane >> 3) + 8 * part; b0 < ne && !fail; b0 += 8 * P * MB) {
                unsigned long long raw[MB];
                unsigned spins = 0;
                for (;;) {
                    bool wait = false;
#pragma unroll
                    for (int m = 0; m < MB; ++m) {
                        const int b = b0 + 8 * P * m;
                        raw[m] = b < ne && v < 7 ? peek(X + (unsigned)((b * K + c) * kWideSum + v)) : 0ull;
                    }
#pragma unroll
                    for (int m = 0; m < MB; ++m) wait = wait || raw[m] == kEmpty;
                    if (!wait) break;
                    if (give_up(spins, A.flags)) {
                        fail = true;
                        break;
                    }
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int b = b0 + 8 * P * m;
                    const double val = as_value(raw[m]);
                    if (v < 3) {
                        d += val;
                    } else if (b < ne && v < 7) {
                        const int g = S.eagg[b];
#pragma unroll
                        for (int l = 0; l < NBK; ++l)
                            if (l < nloc) {
                                const double* cr = &S.crow[l][g][v - 3];
#pragma unroll
                                for (int a = 0; a < 4; ++a) cw[l][a] += cr[a * 4] * val;
                            }
                    }
                }
            }
#pragma unroll
            for (int l = 0; l < NBK; ++l)
                if (l < nloc) {
                    double u8[8] = {v == 0 ? d : 0.0, v == 1 ? d : 0.0, v == 2 ? d : 0.0,
                                    cw[l][0], cw[l][1], cw[l][2], cw[l][3], 0.0};
                    const double sum = wave_sum8(u8);
                    if ((lane & 7) == 0) S.xp[c][part][l][lane >> 3] = sum;
                }
        }
        if (fail) S.bad = 1;
        __syncthreads();
        if (S.bad) return false;
        // everyone has the sums of this exchange, so the rows read before it and the sums of
        // the exchange before it are no longer needed by anyone
        empty_rows();
        double* Xe = xcopy(nx + 1);
        if (t < nloc * K * 7) publish_empty(Xe + ((int64_t)(e0 + t / (K * 7)) * K + (t / 7) % K) * kWideSum + t % 7);
        return true;
    };
    // scalar role: thread t < 4 K nloc keeps column sc_c's scalars (all threads of a column
    // alike) and the coarse value sc_a of an own aggregate
    const bool scalar = t < 4 * K * nloc;
    const int sc_c = t % K, sc_a = t / K;
    auto total = [&](int v) {
        double s = S.xp[sc_c][0][sc_a >> 2][v];
#pragma unroll
        for (int m = 1; m < P; ++m) s += S.xp[sc_c][m][sc_a >> 2][v];
        return s;
    };
    double my_bb = 0.0, my_rr = 0.0, my_gam = 0.0, my_alpha = 0.0, my_c = 0.0, my_cs = 0.0;
    double my_ref = 0.0;   // |r|^2 where my_c was last formed from r
    bool my_done = false;
    int my_its = 0;
    double r[KG];
#pragma unroll
    for (int ii = 0; ii < KG; ++ii) {
        r[ii] = 0.0;
        if (q + ii * Q < K) S.x[q + ii * Q][row] = S.p[q + ii * Q][row] = S.s[q + ii * Q][row] = 0.0;
    }
    const double rtol2 = A.rtol * A.rtol;
    constexpr int kMaxRestarts = 6;
    int total_it = 0, cycle = 0;
    bool first = true;
    // Passes: kZero forms the residual of x = 0 (which gives |b|^2 and so fixes the tolerance),
    // kStep is an iteration, kCoarse forms the coarse values from the iteration's residual, kVerify
    // forms the true residual once the iteration's own has converged, and starts another cycle
    // from it when it has not.  One copy of the product and of the exchange serves them all.
    // (kCoarse has no neighbour exchange: the rows that its exchange empties are empty already,
    // and its owner fills them again only after the next one.)
    enum { kZero, kStep, kCoarse, kVerify };
    int pass = kZero;
    __syncthreads();
    for (;;) {
        // addresses are formed anew in each pass: kept across it they would not fit the registers
        asm volatile("" : "+v"(t), "+v"(lane), "+v"(row), "+v"(i));
        double u[KG], w[KG];
        if (pass == kStep) {
            // u = M^{-1} r.  The block solve is a preconditioner: C_BB^{-1} (FP32) times r
            // rounded to FP32, with FP32 sums (the solution's accuracy comes from the FP64
            // residuals).  Padding rows hold r = 0 and an identity block in C_BB^{-1}.
#pragma unroll
            for (int ii = 0; ii < KG; ++ii)
                if (q + ii * Q < K) S.r[q + ii * Q][row] = act ? (float)r[ii] : 0.0f;
            __syncthreads();
            {
                const float* y = &S.r[lane & 3][(unit / 2) * kBS + seg * D::JS];
                wide_float4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < D::JS; j += 4) {
                    const float4 yj = *reinterpret_cast<const float4*>(y + j);
                    a0 = __builtin_amdgcn_mfma_f32_4x4x1f32(binv[j], yj.x, a0, 0, 0, 0);
                    a1 = __builtin_amdgcn_mfma_f32_4x4x1f32(binv[j + 1], yj.y, a1, 0, 0, 0);
                    a0 = __builtin_amdgcn_mfma_f32_4x4x1f32(binv[j + 2], yj.z, a0, 0, 0, 0);
                    a1 = __builtin_amdgcn_mfma_f32_4x4x1f32(binv[j + 3], yj.w, a1, 0, 0, 0);
                }
                // lane l now holds rows 4 (l / 4) .. + 3 of column l % 4
                const int c = lane & 3;
                if (c < K) {
                    const wide_float4 v = a0 + a1;
                    *reinterpret_cast<float4*>(&S.part[seg][c][unit * 64 + (lane & ~3)]) =
                        make_float4(v.x, v.y, v.z, v.w);
                }
            }
            __syncthreads();
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) {
                const int c = q + ii * Q;
                u[ii] = 0.0;
                if (c < K) {
                    float v = S.part[0][c][row];
#pragma unroll
                    for (int m = 1; m < D::SEG; ++m) v += S.part[m][c][row];
                    double cm = 0.0;
#pragma unroll
                    for (int a = 0; a < 4; ++a) cm += S.phi[a][row] * S.cval[my_la][a][c];
                    u[ii] = (double)v + cm;
                }
            }
        } else {
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) u[ii] = q + ii * Q < K ? S.x[q + ii * Q][row] : 0.0;
        }
        if (pass != kCoarse) product(u, w);
        if (pass != kStep)
#pragma unroll
            for (int ii = 0; ii < KG; ++ii) {
                const int c = q + ii * Q;
                if (pass != kCoarse) {
                    r[ii] = act && c < K ? A.b[(int64_t)i * A.ld + c] - w[ii] : 0.0;
                    if (c < K) S.p[c][row] = S.s[c][row] = 0.0;
                }
                u[ii] = 0.0;
                w[ii] = r[ii];
            }
        // sums of r u, w u, r r and the shares of w (of a residual: u = 0, w = r)
        if (!exchange(r, u, w)) return;
        if (pass != kStep) {
            if (scalar) {
                my_rr = my_ref = total(2);
                my_c = total(3 + (sc_a & 3));
                if (pass != kCoarse) my_cs = 0.0;
                S.cval[sc_a >> 2][sc_a & 3][sc_c] = my_c;
                if (pass == kZero) {
                    my_bb = my_rr;
                    my_done = !(my_bb > 0.0);
                }
                if (pass == kVerify && !my_done && my_rr <= rtol2 * my_bb) my_done = true;
                if (sc_a == 0) S.live[sc_c] = my_done ? 0 : 1;
            }
            if (pass == kVerify) {
                __syncthreads();
                bool all = true;
#pragma unroll
                for (int c = 0; c < K; ++c) all = all && S.live[c] == 0;
                if (all || total_it >= A.maxiter || cycle == kMaxRestarts) break;
                ++cycle;
            }
            if (pass != kCoarse) first = true;
            pass = kStep;
            continue;
        }
        const bool can = total_it < A.maxiter;
        if (scalar) {
            const double g = total(0), d = total(1);
            my_rr = total(2);
            double al = 0.0, be = 0.0;
            const bool live = !my_done && my_rr > rtol2 * my_bb;
            if (live) {
                if (can) {
                    if (first) {
                        al = g / d;
                    } else {
                        be = g / my_gam;
                        al = g / (d - be * g / my_alpha);
                    }
                    my_its = total_it + 1;
                }
                my_gam = g;
                my_alpha = al;
            }
            my_cs = total(3 + (sc_a & 3)) + be * my_cs;
            my_c -= al * my_cs;
            S.cval[sc_a >> 2][sc_a & 3][sc_c] = my_c;
            if (sc_a == 0) {
                S.coef[0][sc_c] = al;
                S.coef[1][sc_c] = be;
                S.live[sc_c] = live ? my_rr < kFresh * kFresh * my_ref ? 2 : 1 : 0;
            }
        }
        __syncthreads();
        bool conv = true, stale = false;
#pragma unroll
        for (int c = 0; c < K; ++c) {
            conv = conv && S.live[c] == 0;
            stale = stale || S.live[c] == 2;
        }
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            if (c < K) {
                // columns that converged (or are done) have alpha = 0: x and r stay
                const double al = S.coef[0][c], be = S.coef[1][c];
                const double pn = u[ii] + be * S.p[c][row], sn = w[ii] + be * S.s[c][row];
                S.p[c][row] = pn;
                S.s[c][row] = sn;
                S.x[c][row] += al * pn;
                r[ii] -= al * sn;
            }
        }
        if (conv || !can) {
            pass = kVerify;
        } else {
            ++total_it;
            first = false;
            if (stale) pass = kCoarse;
        }
    }
    if (act)
#pragma unroll
        for (int ii = 0; ii < KG; ++ii) {
            const int c = q + ii * Q;
            if (c < K) A.x[(int64_t)i * A.ld + c] = S.x[c][row];
        }
    if (B0 == 0 && t < K) {
        A.iters[t] = my_its;
        A.relres[t] = my_bb > 0.0 ? sqrt(my_rr / my_bb) : 0.0;
    }
}

// Solves in groups of up to kWideCols columns when every workgroup can be resident; *done says so.
// Two blocks per workgroup up to 512 blocks, four up to 1,024: at 392 blocks three columns take
// 1.61 ms with two and 1.97 ms with four (145 iterations).  Nine columns are three groups, one after
// the other: 8.5 ms at 782 blocks, where the multi-launch solve of all nine takes 13.2 ms.
hipError_t launch_pcg_wide(const PcgSetup& ps, const double* b, double* x, int k, double rtol, int maxiter,
                           const PcgMlWork& w, int* iters, double* relres, hipStream_t s, bool* done)
{
    *done = false;
    static_assert(sizeof(WideShared<kWideCols, 4>) <= 160 * 1024, "LDS of a workgroup");
    if (ps.nb > 4 * kMaxBarrierW || 3 * kWideEntries * kWideSum > ps.n) return hipSuccess;
    const int nbk = ps.nb <= 2 * kMaxBarrierW ? 2 : 4;
    const int wgs = (ps.nb + nbk - 1) / nbk;
    struct Kernel {
        const void* fn;
        size_t smem;
    };
#define TP_WIDE(K, NBK, TAIL) {(const void*)k_pcg_wide<K, NBK, TAIL>, sizeof(WideShared<K, NBK>)}
    static const Kernel kernels[2][2][kWideCols] = {
        {{TP_WIDE(1, 2, false), TP_WIDE(2, 2, false), TP_WIDE(3, 2, false)},
         {TP_WIDE(1, 4, false), TP_WIDE(2, 4, false), TP_WIDE(3, 4, false)}},
        {{TP_WIDE(1, 2, true), TP_WIDE(2, 2, true), TP_WIDE(3, 2, true)},
         {TP_WIDE(1, 4, true), TP_WIDE(2, 4, true), TP_WIDE(3, 4, true)}}};
#undef TP_WIDE
    WideArgs A;
    A.n = ps.n; A.nb = ps.nb; A.nc = ps.nc; A.ell_w = ps.ell_w; A.pcol = ps.pcol; A.pval = ps.pval;
    A.toff = ps.toff; A.tslot = ps.tslot;
    A.bstart = ps.bstart; A.blk = ps.blk; A.agg_of_block = ps.agg_of_block; A.phi = ps.phi; A.Binv = ps.Binv;
    A.C0inv = ps.C0inv; A.ld = k; A.U0 = w.m; A.U1 = w.an; A.X = w.v; A.flags = w.flags; A.rtol = rtol;
    A.maxiter = maxiter;
    for (int c0 = 0; c0 < k; c0 += kWideCols) {
        const int kc = std::min(kWideCols, k - c0);
        const Kernel& kern = kernels[ps.ell_w > kWideCache ? 1 : 0][nbk == 2 ? 0 : 1][kc - 1];
        hipError_t e = hipFuncSetAttribute(kern.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kern.smem);
        if (e != hipSuccess) return e;
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern.fn, kWideThreads, kern.smem);
        if (e != hipSuccess) return e;
        if (c0 == 0 && (int64_t)wgs > (int64_t)per_cu * device_info().num_cu) return hipSuccess;
        A.b = b + c0; A.x = x + c0; A.iters = iters + c0; A.relres = relres + c0;
        hipLaunchKernelGGL(k_wide_empty, dim3(256), dim3(256), 0, s, A, kc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        void* params[] = {(void*)&A};
        e = hipLaunchCooperativeKernel(kern.fn, dim3(wgs), dim3(kWideThreads), params, (unsigned)kern.smem, s);
        if (e != hipSuccess) return e;
    }
    *done = true;
    return hipSuccess;
}

}  // namespace

// ---------------------------------------------------------------- multi-launch solve
//
// For problems with more than four blocks per workgroup that can be resident at once, the same
// preconditioned Chronopoulos-Gear iteration runs as one kernel per phase; the kernel
// boundaries are the grid-wide synchronisation.  Per iteration:
//   k_ml_block       the previous iteration's update of the block's rows (p = m + beta p,
//                    s = an + beta s, x += alpha p, r -= alpha s), then v = C_BB^{-1} r_B
//                    (FP32, as in k_pcg) and the block's shares Phi_B^T r
//   k_ml_coarse_rhs  coarse right-hand side g: per aggregate, its blocks' shares in order
//   k_ml_apply       coarse values of the aggregates of the workgroup's rows (rows of
//                    C0^{-1} times g), m = v + Phi c
//   k_ml_spmv        an = C m, partial sums of (r, m), (an, m), (r, r) per workgroup
//   k_ml_scalars     the sums in fixed order, alpha and beta per column, the stop flag
// Every kernel returns at once when the stop flag is set, so a batch of iterations
// enqueued past convergence costs only its launches; the host reads the flag after each
// batch, then verifies with the true residual b - C x and restarts from it when needed.
// The update of an iteration that raised the stop flag is never applied: it has alpha = 0
// in every column, so it would leave x and r as they are.

constexpr int kMlRows = kThreads;     // rows per workgroup of the row-parallel kernels
constexpr int kMlBatch = 16;          // iterations enqueued between two reads of the flag
constexpr int kMlScalarThreads = 1024;

struct MlState {
    int stop, total_it, first, have_bb;
    int upd;                                       // an update is pending (ca, cb)
    int done[kMaxGroupCols], its[kMaxGroupCols];
    double bb[kMaxGroupCols], rr[kMaxGroupCols], gam[kMaxGroupCols], alpha[kMaxGroupCols];
    double ca[kMaxGroupCols], cb[kMaxGroupCols];   // this iteration's alpha, beta (0 when frozen)
};

__global__ void k_ml_init(MlState* st)
{
    if (threadIdx.x == 0) {
        st->stop = 0;
        st->total_it = 0;
        st->first = 1;
        st->have_bb = 0;
        st->upd = 0;
        for (int c = 0; c < kMaxGroupCols; ++c) {
            st->done[c] = 0;
            st->its[c] = 0;
            st->bb[c] = st->rr[c] = st->gam[c] = st->alpha[c] = st->ca[c] = st->cb[c] = 0.0;
        }
    }
}

// r = b - C x (x = 0 when zero_x: then r = b and x is cleared), p = s = 0, and per
// workgroup the partial sums of r^2 (part[wg][0][c]).
template <int KG>
__global__ __launch_bounds__(kMlRows) void k_ml_residual(int64_t n, int k, int w, const int32_t* __restrict__ pcol,
                                                         const double* __restrict__ pval, const double* __restrict__ b,
                                                         double* __restrict__ x, double* __restrict__ r,
                                                         double* __restrict__ p, double* __restrict__ s,
                                                         double* __restrict__ part, int zero_x)
{
    __shared__ double wave_sh[(kMlRows / 64) * KG];
    __shared__ double sums[KG];
    const int64_t i = (int64_t)blockIdx.x * kMlRows + threadIdx.x;
    double rr[KG];
#pragma unroll
    for (int c = 0; c < KG; ++c) rr[c] = 0.0;
    if (i < n) {
        double cx[KG];
#pragma unroll
        for (int c = 0; c < KG; ++c) cx[c] = 0.0;
        if (!zero_x)
            for (int e = 0; e < w; ++e) {
                const int32_t j = pcol[(int64_t)e * n + i];
                const double a = pval[(int64_t)e * n + i];
#pragma unroll
                for (int c = 0; c < KG; ++c)
                    if (c < k) cx[c] += a * x[(int64_t)j * k + c];
            }
#pragma unroll
        for (int c = 0; c < KG; ++c)
            if (c < k) {
                const int64_t id = i * k + c;
                const double rv = b[id] - cx[c];
                if (zero_x) x[id] = 0.0;   // (x is not read when zero_x)
                r[id] = rv;
                p[id] = 0.0;
                s[id] = 0.0;
                rr[c] = rv * rv;
            }
    }
    wg_reduce<KG>(rr, wave_sh, sums);
    if ((int)threadIdx.x < KG) part[(int64_t)blockIdx.x * 3 * KG + threadIdx.x] = sums[threadIdx.x];
}

// The block's rows of r are read and its rows of v written as one contiguous range (the
// row stride is KG), staged through LDS.
template <int KG>
__global__ __launch_bounds__(kThreads) void k_ml_block(const MlState* __restrict__ st,
                                                       const int32_t* __restrict__ bstart,
                                                       const float* __restrict__ Binv, const double* __restrict__ phi,
                                                       const double* __restrict__ m, const double* __restrict__ an,
                                                       double* __restrict__ p, double* __restrict__ s,
                                                       double* __restrict__ x, double* __restrict__ r,
                                                       double* __restrict__ v, double* __restrict__ shares)
{
    __shared__ float r32[kBS * KG];
    __shared__ double y64[kBS * KG];
    __shared__ double half[kBS * KG];
    __shared__ double wave_sh[(kThreads / 64) * 4 * KG];
    __shared__ double sums[4 * KG];
    __shared__ double coef[2 * KG];
    if (st->stop) return;
    const int B = blockIdx.x, t = threadIdx.x;
    const int32_t s0 = bstart[B], cnt = bstart[B + 1] - s0;
    const bool upd = st->upd != 0;
    if (t < KG) {
        coef[t] = st->ca[t];
        coef[KG + t] = st->cb[t];
    }
    __syncthreads();
    const int64_t e0 = (int64_t)s0 * KG;
    for (int e = t; e < kBS * KG; e += kThreads) {
        double yv = 0.0;
        if (e < cnt * KG) {
            const int64_t id = e0 + e;
            yv = r[id];
            if (upd) {
                const int c = e % KG;
                const double al = coef[c], be = coef[KG + c];
                const double pn = m[id] + be * p[id];
                const double sn = an[id] + be * s[id];
                p[id] = pn;
                s[id] = sn;
                x[id] += al * pn;
                yv -= al * sn;
                r[id] = yv;
            }
        }
        y64[e] = yv;
        r32[e] = (float)yv;
    }
    __syncthreads();
    // the block product as in k_pcg: FP32, row tt's sum in two halves of j
    const int tt = t & (kBS - 1), jbeg = (t / kBS) * (kBS / 2);
    const float* Bi = Binv + (int64_t)B * kBS * kBS;
    float v32[KG];
#pragma unroll
    for (int c = 0; c < KG; ++c) v32[c] = 0.0f;
    constexpr int CH = 8;
#pragma unroll 1
    for (int j0 = jbeg; j0 < jbeg + kBS / 2; j0 += CH) {
        float bj[CH], yj[CH * KG];
#pragma unroll
        for (int q = 0; q < CH; ++q) bj[q] = Bi[(j0 + q) * kBS + tt];
#pragma unroll
        for (int q = 0; q < CH * KG; ++q) yj[q] = r32[j0 * KG + q];
#pragma unroll
        for (int q = 0; q < CH; ++q)
#pragma unroll
            for (int c = 0; c < KG; ++c) v32[c] = __builtin_fmaf(bj[q], yj[q * KG + c], v32[c]);
    }
    if (t >= kBS) {
#pragma unroll
        for (int c = 0; c < KG; ++c) half[tt * KG + c] = (double)v32[c];
    }
    __syncthreads();
    if (t < kBS) {
#pragma unroll
        for (int c = 0; c < KG; ++c) half[t * KG + c] += (double)v32[c];   // own half + helper half
    }
    // the block's shares of the coarse right-hand side: sum over its rows of phi[a] y
    double tmp[4 * KG];
    {
        const bool act = t < cnt;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double ph = act ? phi[(int64_t)(s0 + t) * 4 + a] : 0.0;
#pragma unroll
            for (int c = 0; c < KG; ++c) tmp[a * KG + c] = act ? ph * y64[t * KG + c] : 0.0;
        }
    }
    wg_reduce<4 * KG>(tmp, wave_sh, sums);   // (its barriers also order the writes to half)
    if (t < 4 * KG) shares[(int64_t)B * 4 * KG + t] = sums[t];
    double* vb = v + (int64_t)s0 * KG;
    for (int e = t; e < cnt * KG; e += kThreads) vb[e] = half[e];
}

// g[4 ag + a][c] = sum over the blocks of aggregate ag, in order, of their shares.
template <int KG>
__global__ __launch_bounds__(64) void k_ml_coarse_rhs(const MlState* __restrict__ st, const int32_t* __restrict__ astart,
                                                      const double* __restrict__ shares, double* __restrict__ g)
{
    if (st->stop) return;
    const int ag = blockIdx.x, t = threadIdx.x;
    if (t >= 4 * KG) return;
    const int b0 = astart[ag], b1 = astart[ag + 1];
    double acc = 0.0;
    for (int bb = b0; bb < b1; bb += 8) {
        double u[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) u[q] = bb + q < b1 ? shares[(int64_t)(bb + q) * 4 * KG + t] : 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += u[q];
    }
    g[(int64_t)ag * 4 * KG + t] = acc;
}

// Coarse values of the aggregates of rows [r0, r0 + kMlRows) (consecutive in block order),
// then m = v + Phi c for those rows.
template <int KG>
__global__ __launch_bounds__(kMlRows) void k_ml_apply(const MlState* __restrict__ st, int64_t n, int nc,
                                                      const int32_t* __restrict__ blk,
                                                      const int32_t* __restrict__ agg_of_block,
                                                      const double* __restrict__ C0inv, const double* __restrict__ g,
                                                      const double* __restrict__ phi, const double* __restrict__ v,
                                                      double* __restrict__ m)
{
    __shared__ double gs[kCoarseMax * KG];
    __shared__ double cw[kCoarseMax * KG];
    __shared__ double psum[kMlRows];
    if (st->stop) return;
    const int t = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kMlRows;
    const int64_t r1 = min(n, r0 + kMlRows);
    const int ag_lo = agg_of_block[blk[r0]], ag_hi = agg_of_block[blk[r1 - 1]];
    for (int q = t; q < nc * KG; q += kMlRows) gs[q] = g[q];
    __syncthreads();
    const int jobs = (ag_hi - ag_lo + 1) * 4 * KG;
    for (int j0 = 0; j0 < jobs; j0 += kMlRows) {
        const int nj = min(kMlRows, jobs - j0);
        const int P = max(1, kMlRows / nj);
        const int chunk = (nc + P - 1) / P;
        const int jl = t / P, pt = t - jl * P;
        if (jl < nj) {
            const int job = j0 + jl, row = job / KG, c = job - row * KG;
            const int d = 4 * ag_lo + row;
            const int d0 = pt * chunk, d1 = min(nc, d0 + chunk);
            psum[jl * P + pt] = d1 > d0 ? dot_fixed(C0inv + (int64_t)d * nc + d0, gs + d0 * KG + c, d1 - d0, KG) : 0.0;
        }
        __syncthreads();
        if (t < nj) cw[j0 + t] = sum_fixed(psum + t * P, P, 1);
        __syncthreads();
    }
    // element-wise over the rows' KG columns (contiguous loads and stores)
    for (int64_t e = r0 * KG + t; e < r1 * KG; e += kMlRows) {
        const int64_t i = e / KG;
        const int c = (int)(e - i * KG);
        const int ag = agg_of_block[blk[i]] - ag_lo;
        double cm = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) cm += phi[i * 4 + a] * cw[(ag * 4 + a) * KG + c];
        m[e] = v[e] + cm;
    }
}

// an = C m and the partial sums of (r, m), (an, m), (r, r): one thread per element (row,
// column) of R = kMlSpThreads / KG rows at a time, `rounds` times (chosen at launch so
// that there are about kMlSpTargetWg workgroups: enough to fill the device, few enough
// partial sums for the scalars kernel), the gathers of a row's KG values contiguous across
// lanes; the partial sums go through LDS and are added per column over the rows in order.
constexpr int kMlSpThreads = 1024;
constexpr int kMlSpTargetWg = 384;
constexpr int kMlSpMaxRounds = 4;
template <int KG>
__global__ __launch_bounds__(kMlSpThreads) void k_ml_spmv(const MlState* __restrict__ st, int64_t n, int rounds, int w,
                                                          const int32_t* __restrict__ pcol,
                                                          const double* __restrict__ pval,
                                                          const double* __restrict__ m, const double* __restrict__ r,
                                                          double* __restrict__ an, double* __restrict__ part)
{
    constexpr int R = kMlSpThreads / KG;
    __shared__ double val[3][R * KG];
    if (st->stop) return;
    const int t = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * R * rounds;
    const int rl = t / KG, c = t - rl * KG;
    double v0 = 0.0, v1 = 0.0, v2 = 0.0;   // this thread's column, its rows added in order
    for (int rd = 0; rd < rounds; ++rd) {
        const int64_t i = r0 + (int64_t)rd * R + rl;
        if (rl < R && i < n) {
            double acc = 0.0;
            for (int e = 0; e < w; ++e) {
                const int32_t j = pcol[(int64_t)e * n + i];
                acc += pval[(int64_t)e * n + i] * m[(int64_t)j * KG + c];
            }
            const int64_t id = i * KG + c;
            const double mi = m[id], ri = r[id];
            an[id] = acc;
            v0 += ri * mi;
            v1 += acc * mi;
            v2 += ri * ri;
        }
    }
    if (rl < R) {
        val[0][t] = v0;
        val[1][t] = v1;
        val[2][t] = v2;
    }
    __syncthreads();
    // each of the 3 KG sums over the R rows in P parts of consecutive rows, then the parts
    // in order
    constexpr int M = 3 * KG, P = kMlSpThreads / M, CH = (R + P - 1) / P;
    __shared__ double ps[kMlSpThreads];
    {
        const int q = t / P, pt = t - q * P;
        if (q < M) {
            const int g = q / KG, cc = q - g * KG;
            const int ro0 = pt * CH, ro1 = min(R, ro0 + CH);
            double acc = 0.0;
            for (int ro = ro0; ro < ro1; ++ro) acc += val[g][ro * KG + cc];
            ps[q * P + pt] = acc;
        }
    }
    __syncthreads();
    if (t < M) {
        double a = 0.0;
        for (int z = 0; z < P; ++z) a += ps[t * P + z];
        part[(int64_t)blockIdx.x * 3 * KG + t] = a;
    }
}

// Sums over the nwg workgroups of the first M values of part ([nwg][3KG]) in a fixed
// order (each value cut into P parts of consecutive workgroups, the parts added in order)
// into tot[0 .. M), by kMlScalarThreads threads.
template <int M, int KG>
__device__ __forceinline__ void ml_grid_sum(const double* __restrict__ part, int nwg, double* ps, double* tot)
{
    constexpr int P = kMlScalarThreads / M;
    const int t = threadIdx.x;
    const int chunk = (nwg + P - 1) / P;
    const int q = t / P, pt = t - q * P;
    if (q < M) {
        const int w0 = pt * chunk, w1 = min(nwg, w0 + chunk);
        double acc = 0.0;
        for (int ww = w0; ww < w1; ww += 8) {
            double u[8];
#pragma unroll
            for (int z = 0; z < 8; ++z) u[z] = ww + z < w1 ? part[(int64_t)(ww + z) * 3 * KG + q] : 0.0;
#pragma unroll
            for (int z = 0; z < 8; ++z) acc += u[z];
        }
        ps[q * P + pt] = acc;
    }
    __syncthreads();
    if (t < M) {
        double a = 0.0;
        for (int z = 0; z < P; ++z) a += ps[t * P + z];
        tot[t] = a;
    }
    __syncthreads();
}

// The column scalars of one iteration (the rules of k_pcg): gamma = (r, m), delta =
// (an, m), |r|^2; the first iteration of a solve takes |b|^2 from it; columns whose |r|^2
// is at or below rtol^2 |b|^2 are frozen (alpha = beta = 0); the stop flag is raised when
// no column is open or the iteration budget is spent.
template <int KG>
__global__ __launch_bounds__(kMlScalarThreads) void k_ml_scalars(MlState* __restrict__ st, const double* __restrict__ part,
                                                                  int nwg, int k, double rtol2, int maxiter)
{
    __shared__ double ps[kMlScalarThreads];
    __shared__ double tot[3 * KG];
    __shared__ int live_sh[KG];
    if (st->stop) return;
    ml_grid_sum<3 * KG, KG>(part, nwg, ps, tot);
    const int t = threadIdx.x;
    const bool can = st->total_it < maxiter;
    if (t < KG) {
        const int c = t;
        const double gm = tot[c], de = tot[KG + c], rrv = tot[2 * KG + c];
        if (!st->have_bb) {
            st->bb[c] = rrv;
            st->done[c] = (c >= k || !(rrv > 0.0)) ? 1 : 0;
        }
        st->rr[c] = rrv;
        const bool live = !st->done[c] && rrv > rtol2 * st->bb[c];
        double al = 0.0, be = 0.0;
        if (live) {
            if (can) {
                if (st->first) {
                    al = gm / de;
                } else {
                    be = gm / st->gam[c];
                    al = gm / (de - be * gm / st->alpha[c]);
                }
                st->its[c] = st->total_it + 1;
            }
            st->gam[c] = gm;
            st->alpha[c] = al;
        }
        st->ca[c] = al;
        st->cb[c] = be;
        live_sh[c] = live ? 1 : 0;
    }
    __syncthreads();
    if (t == 0) {
        bool any = false;
        for (int c = 0; c < KG; ++c) any = any || live_sh[c] != 0;
        st->have_bb = 1;
        if (!any || !can) {
            st->stop = 1;
        } else {
            st->total_it += 1;
            st->first = 0;
            st->upd = 1;
        }
    }
}

// After a true residual (k_ml_residual): columns at or below rtol^2 |b|^2 are done; the
// solve ends when all are done or the budget is spent, else it restarts from r (the stop
// flag is lowered and the next iteration is a first one).
template <int KG>
__global__ __launch_bounds__(kMlScalarThreads) void k_ml_verify(MlState* __restrict__ st, const double* __restrict__ part,
                                                                 int nwg, double rtol2, int maxiter)
{
    __shared__ double ps[kMlScalarThreads];
    __shared__ double tot[KG];
    ml_grid_sum<KG, KG>(part, nwg, ps, tot);
    const int t = threadIdx.x;
    if (t < KG && !st->done[t]) {
        st->rr[t] = tot[t];
        if (tot[t] <= rtol2 * st->bb[t]) st->done[t] = 1;
    }
    __syncthreads();
    if (t == 0) {
        bool all = true;
        for (int c = 0; c < KG; ++c) all = all && st->done[c] != 0;
        st->upd = 0;
        if (all || st->total_it >= maxiter) {
            st->stop = 1;
        } else {
            st->stop = 0;
            st->first = 1;
        }
    }
}

__global__ void k_ml_finish(const MlState* __restrict__ st, int k, int* __restrict__ iters, double* __restrict__ relres)
{
    const int c = threadIdx.x;
    if (c < k) {
        iters[c] = st->its[c];
        relres[c] = st->bb[c] > 0.0 ? sqrt(st->rr[c] / st->bb[c]) : 0.0;
    }
}

namespace {

template <int KG>
hipError_t launch_pcg_ml_k(const PcgSetup& ps, const double* b, double* x, int k, double rtol, int maxiter,
                           const PcgMlWork& w, int* iters, double* relres, hipStream_t s)
{
    const int64_t n = ps.n;
    const int nwg = (int)((n + kMlRows - 1) / kMlRows);
    constexpr int kSpR = kMlSpThreads / KG;
    const int sp_rounds = (int)std::max<int64_t>(1, std::min<int64_t>(kMlSpMaxRounds, (n + kSpR - 1) / kSpR / kMlSpTargetWg));
    const int64_t sp_rows = (int64_t)kSpR * sp_rounds;
    const int nws = (int)((n + sp_rows - 1) / sp_rows);
    if (k != KG) return hipErrorInvalidValue;
    MlState* st = static_cast<MlState*>(w.state);
    MlState* hs = static_cast<MlState*>(w.state_host);
    const double rtol2 = rtol * rtol;
    hipError_t e;
#define TP_ML_CHECK() do { if ((e = hipGetLastError()) != hipSuccess) return e; } while (0)
    hipLaunchKernelGGL(k_ml_init, dim3(1), dim3(64), 0, s, st);
    TP_ML_CHECK();
    hipLaunchKernelGGL((k_ml_residual<KG>), dim3(nwg), dim3(kMlRows), 0, s, n, k, ps.ell_w, ps.pcol, ps.pval, b, x,
                       w.r, w.p, w.s, w.part, 1);
    TP_ML_CHECK();
    constexpr int kMaxRestarts = 6;
    for (int cycle = 0;; ++cycle) {
        for (;;) {
            for (int q = 0; q < kMlBatch; ++q) {
                hipLaunchKernelGGL((k_ml_block<KG>), dim3(ps.nb), dim3(kThreads), 0, s, st, ps.bstart, ps.Binv,
                                   ps.phi, w.m, w.an, w.p, w.s, x, w.r, w.v, w.shares);
                hipLaunchKernelGGL((k_ml_coarse_rhs<KG>), dim3(ps.na), dim3(64), 0, s, st, ps.astart, w.shares, w.g);
                hipLaunchKernelGGL((k_ml_apply<KG>), dim3(nwg), dim3(kMlRows), 0, s, st, n, ps.nc, ps.blk,
                                   ps.agg_of_block, ps.C0inv, w.g, ps.phi, w.v, w.m);
                hipLaunchKernelGGL((k_ml_spmv<KG>), dim3(nws), dim3(kMlSpThreads), 0, s, st, n, sp_rounds, ps.ell_w, ps.pcol,
                                   ps.pval, w.m, w.r, w.an, w.part);
                hipLaunchKernelGGL((k_ml_scalars<KG>), dim3(1), dim3(kMlScalarThreads), 0, s, st, w.part, nws, k,
                                   rtol2, maxiter);
            }
            TP_ML_CHECK();
            if ((e = hipMemcpyAsync(hs, st, sizeof(MlState), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
            if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
            if (hs->stop) break;
        }
        // true residual, then verification (and a restart from it when needed)
        hipLaunchKernelGGL((k_ml_residual<KG>), dim3(nwg), dim3(kMlRows), 0, s, n, k, ps.ell_w, ps.pcol, ps.pval, b,
                           x, w.r, w.p, w.s, w.part, 0);
        hipLaunchKernelGGL((k_ml_verify<KG>), dim3(1), dim3(kMlScalarThreads), 0, s, st, w.part, nwg, rtol2, maxiter);
        TP_ML_CHECK();
        if ((e = hipMemcpyAsync(hs, st, sizeof(MlState), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (hs->stop || cycle >= kMaxRestarts) break;
    }
    hipLaunchKernelGGL(k_ml_finish, dim3(1), dim3(64), 0, s, st, k, iters, relres);
    TP_ML_CHECK();
#undef TP_ML_CHECK
    return hipSuccess;
}

}  // namespace

int pcg_max_blocks_multi() { return kMaxNbMulti; }
size_t pcg_ml_state_bytes() { return sizeof(MlState); }
// per-workgroup partial sums: the residual kernel's kMlRows rows per workgroup or the
// sparse product's one round of kMlSpThreads / KG rows, whichever gives more workgroups
size_t pcg_ml_part_doubles(int64_t n)
{
    const int64_t rows = std::min<int64_t>(kMlRows, kMlSpThreads / kMaxGroupCols);
    return (size_t)((n + rows - 1) / rows) * 3 * kMaxGroupCols;
}

hipError_t launch_pcg_ml(const PcgSetup& ps, const double* b, double* x, int k, double rtol, int maxiter,
                         const PcgMlWork& w, int* iters, double* relres, hipStream_t s)
{
    bool done = false;
    const hipError_t e = launch_pcg_wide(ps, b, x, k, rtol, maxiter, w, iters, relres, s, &done);
    if (done || e != hipSuccess) return e;
    switch (k) {
    case 1: return launch_pcg_ml_k<1>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 2: return launch_pcg_ml_k<2>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 3: return launch_pcg_ml_k<3>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 4: return launch_pcg_ml_k<4>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 5: return launch_pcg_ml_k<5>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 6: return launch_pcg_ml_k<6>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 7: return launch_pcg_ml_k<7>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 8: return launch_pcg_ml_k<8>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    case 9: return launch_pcg_ml_k<9>(ps, b, x, k, rtol, maxiter, w, iters, relres, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tp
