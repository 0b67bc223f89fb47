// Barnes-Hut approximation of the energy and its differential (Sec. 4) on gfx950.
//
// Tree.  Faces are sorted by the 30-bit Morton code of their barycenters (10 bits per
// coordinate, quantized on the bounding box of all barycenters), ties by the caller's face
// number (faces are stored internally in the Morton order of the first mesh).  Leaves hold `leaf` consecutive sorted
// faces and the internal nodes form a perfect binary tree over the leaves in heap order
// (node 1 is the root, node i has children 2i and 2i + 1, the leaves are nodes
// P .. 2P - 1).  The tree is therefore fixed by the sort alone: no pointer chasing, and
// the traversal needs no stack (the next node after a subtree follows from the heap
// index).  Node quantities are built level by level: a_I, sum a_T X_T, the bounding box of
// the faces' vertices, X_I and r_I^2 (largest squared distance from X_I to a box corner).
// The geometric quantities that decide admissibility are formed in FP64 without fused
// multiply-adds, in a fixed order, so the interaction lists are a function of the mesh.
//
// Admissibility: node I is admissible for face S when max(r_S^2, r_I^2) < theta^2 dist^2
// (r_S: largest distance from X_S to a corner of S; dist: distance between the box of S's
// vertices and the box of I).
//
// Traversal.  One thread per face, threads in Morton order, and the 64 lanes of a wave walk
// the tree together: the wave visits the union of its lanes' lists, each lane taking the
// terms of its own, and every lane reads the same node at the same time (k_bh_traverse
// here, wave_walk for the other walks).  An admissible node adds K(X_S, N_S; X_I)
// a_S a_I, a leaf that is not admissible adds the exact terms of its faces T != S, other
// nodes are opened.  The
// differential is that of E_BH with the lists held fixed: the face S side is summed per
// thread; the target side (dX, da of a face T or a node I) is summed across the wave and
// added with device-scope atomics, one set per wave and target; node derivatives then
// reach their member faces through X_I = sum a_T X_T / a_I and a_I = sum a_T, walking up
// each face's ancestors.  The atomic sums make the last bits
// of dE depend on scheduling; E itself is summed per face in a fixed order.
#include "tp_internal.h"
#include "tp_tree.h"

#include <hipcub/hipcub.hpp>

#include <algorithm>

namespace tp {

namespace {

#pragma clang fp contract(off)

__device__ __forceinline__ uint32_t spread10(uint32_t v)
{
    uint32_t out = 0;
    for (int b = 0; b < 10; ++b) out |= ((v >> b) & 1u) << (3 * b);
    return out;
}

__device__ __forceinline__ uint32_t quant10(double x, double lo, double hi)
{
    if (!(hi > lo)) return 0u;
    double t = floor(1024.0 * ((x - lo) / (hi - lo)));
    t = t < 0.0 ? 0.0 : (t > 1023.0 ? 1023.0 : t);
    return (uint32_t)t;
}

// Face boxes (of the three vertices) and r_S^2.
__global__ void k_bh_faceprep(const double* __restrict__ V, const int32_t* __restrict__ F, int64_t nF,
                              const double4* __restrict__ dx, double* __restrict__ flo,
                              double* __restrict__ fhi, double* __restrict__ fr2)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nF) return;
    const double4 X = dx[s];
    const double xs[3] = {X.x, X.y, X.z};
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    double best = 0.0;
    for (int c = 0; c < 3; ++c) {
        const double* v = V + 3 * (int64_t)F[3 * s + c];
        double d2 = 0.0;
        for (int m = 0; m < 3; ++m) {
            lo[m] = v[m] < lo[m] ? v[m] : lo[m];
            hi[m] = v[m] > hi[m] ? v[m] : hi[m];
            const double dm = v[m] - xs[m];
            d2 = d2 + dm * dm;
        }
        best = d2 > best ? d2 : best;
    }
    for (int m = 0; m < 3; ++m) {
        flo[3 * s + m] = lo[m];
        fhi[3 * s + m] = hi[m];
    }
    fr2[s] = best;
}

// Bounding boxes of the barycenters, one per workgroup (min and max do not depend on order);
// k_bh_keys takes them together.  One workgroup for all faces took 117 us at 327,680 faces, this
// 6 us.
constexpr int kBoxBlocks = 128;

__device__ __forceinline__ double pick(double a, double b, bool mx) { return mx ? (a > b ? a : b) : (a < b ? a : b); }

__global__ __launch_bounds__(256) void k_bh_bbox(const double4* __restrict__ dx, int64_t nF,
                                                 double* __restrict__ box)
{
    __shared__ double sh[6][256];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < nF; s += (int64_t)gridDim.x * 256) {
        const double4 X = dx[s];
        const double x[3] = {X.x, X.y, X.z};
        for (int m = 0; m < 3; ++m) {
            lo[m] = pick(x[m], lo[m], false);
            hi[m] = pick(x[m], hi[m], true);
        }
    }
    for (int m = 0; m < 3; ++m) {
        sh[m][threadIdx.x] = lo[m];
        sh[3 + m][threadIdx.x] = hi[m];
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int m = 0; m < 6; ++m) sh[m][threadIdx.x] = pick(sh[m][threadIdx.x + w], sh[m][threadIdx.x], m >= 3);
        __syncthreads();
    }
    if (threadIdx.x < 6) box[6 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

// Keys (Morton code << 32 | caller's face number) and the internal face index as value;
// the caller's numbers make the order independent of how faces are stored.
__global__ __launch_bounds__(256) void k_bh_keys(const double4* __restrict__ dx, int64_t nF,
                                                 const double* __restrict__ boxes, int nbox,
                                                 const int32_t* __restrict__ orig, uint64_t* __restrict__ keys,
                                                 int32_t* __restrict__ idx)
{
    __shared__ double sh[6][kBoxBlocks];
    __shared__ double box[6];
    for (int i = threadIdx.x; i < 6 * nbox; i += 256) sh[i % 6][i / 6] = boxes[i];
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int m = wave; m < 6; m += 4) {
        double v = m < 3 ? INFINITY : -INFINITY;
        for (int i = lane; i < nbox; i += 64) v = pick(sh[m][i], v, m >= 3);
        for (int o = 32; o > 0; o >>= 1) v = pick(__shfl_xor(v, o), v, m >= 3);
        if (lane == 0) box[m] = v;
    }
    __syncthreads();
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nF) return;
    const double4 X = dx[s];
    const uint32_t code = (spread10(quant10(X.x, box[0], box[3])) << 2) |
                          (spread10(quant10(X.y, box[1], box[4])) << 1) | spread10(quant10(X.z, box[2], box[5]));
    keys[s] = ((uint64_t)code << 32) | (uint64_t)(uint32_t)(orig ? orig[s] : (int32_t)s);
    idx[s] = (int32_t)s;
}

// Sorted positions, and the face data (X, a) in sorted order.
__global__ void k_bh_pos(const int32_t* __restrict__ order, int64_t nF, const double4* __restrict__ dx,
                         int32_t* __restrict__ pos, double4* __restrict__ srt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nF) return;
    const int32_t t = order[p];
    pos[t] = (int32_t)p;
    srt[p] = dx[t];
}

// Sums and box of a node while the tree is built: a, sum a X, lo, hi.
struct NodeSums {
    double v[10];
};

__device__ __forceinline__ NodeSums node_join(const NodeSums& L, const NodeSums& R)
{
    NodeSums o;
    for (int m = 0; m < 4; ++m) o.v[m] = L.v[m] + R.v[m];
    for (int m = 4; m < 10; ++m) o.v[m] = pick(L.v[m], R.v[m], m >= 7);
    return o;
}

// Every array of a node: a, sum a X, box, X = sum a X / a, r^2, and its record (lo, hi, r^2, a: one
// 64-byte line, what a test of admissibility reads).
__device__ __forceinline__ void node_store(const BhBuffers& b, int64_t node, const NodeSums& n)
{
    const double a = n.v[0];
    double r2 = 0.0, X[3] = {0.0, 0.0, 0.0};
    if (a > 0.0)
        for (int m = 0; m < 3; ++m) {
            X[m] = n.v[1 + m] / a;
            const double u = X[m] - n.v[4 + m], v = n.v[7 + m] - X[m];
            const double w = u > v ? u : v;
            r2 = r2 + w * w;
        }
    b.na[node] = a;
    b.nr2[node] = r2;
    for (int m = 0; m < 3; ++m) {
        b.nsx[3 * node + m] = n.v[1 + m];
        b.nlo[3 * node + m] = n.v[4 + m];
        b.nhi[3 * node + m] = n.v[7 + m];
        b.nX[3 * node + m] = X[m];
        b.rec[8 * node + m] = n.v[4 + m];
        b.rec[8 * node + 3 + m] = n.v[7 + m];
    }
    b.nxa[node] = double4{X[0], X[1], X[2], a};
    b.rec[8 * node + 6] = r2;
    b.rec[8 * node + 7] = a;
}

// Leaves P + l (sums over the member faces in sorted order) and the levels above them up to one
// node per workgroup, in LDS.  All levels in one workgroup took 557 us at 65,536 leaves (a barrier
// and a pass over global memory per level, 1,024 threads for 131,072 nodes); subtrees of kSubLeaves
// leaves in parallel take 22 us with the leaves (15 us alone), the small launch for what is above 8 us.
constexpr int kSubLeaves = 256;

__global__ __launch_bounds__(kSubLeaves) void k_bh_subtrees(int64_t nF, int leaf, int64_t P, BhBuffers b)
{
    __shared__ double sh[10][kSubLeaves];
    const int t = threadIdx.x;
    const int64_t l = (int64_t)blockIdx.x * kSubLeaves + t;
    if (l == 0) b.nxa[0] = double4{0.0, 0.0, 0.0, 0.0};   // (no node: what k_bct_far reads past a list's end)
    if (l < P) {
        NodeSums n = {{0.0, 0.0, 0.0, 0.0, INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY}};
        for (int64_t p = l * leaf; p < (l + 1) * leaf && p < nF; ++p) {
            const int32_t s = b.order[p];
            const double4 X = b.srt[p];
            const double x[3] = {X.x, X.y, X.z};
            n.v[0] = n.v[0] + X.w;
            for (int m = 0; m < 3; ++m) {
                n.v[1 + m] = n.v[1 + m] + X.w * x[m];
                n.v[4 + m] = pick(b.flo[3 * s + m], n.v[4 + m], false);
                n.v[7 + m] = pick(b.fhi[3 * s + m], n.v[7 + m], true);
            }
        }
        node_store(b, P + l, n);
        for (int m = 0; m < 10; ++m) sh[m][t] = n.v[m];
    }
    int64_t base = P + (int64_t)blockIdx.x * kSubLeaves;
    for (int w = (int)min((int64_t)kSubLeaves, P) >> 1; w >= 1; w >>= 1) {
        base >>= 1;
        __syncthreads();
        NodeSums n;
        if (t < w) {
            NodeSums L, R;
            for (int m = 0; m < 10; ++m) {
                L.v[m] = sh[m][2 * t];
                R.v[m] = sh[m][2 * t + 1];
            }
            n = node_join(L, R);
            node_store(b, base + t, n);
        }
        __syncthreads();
        if (t < w)
            for (int m = 0; m < 10; ++m) sh[m][t] = n.v[m];
    }
}

// The levels above the subtrees (children before parents), one workgroup.
__global__ __launch_bounds__(1024) void k_bh_top(int64_t P, BhBuffers b)
{
    for (int64_t n0 = P / kSubLeaves / 2; n0 >= 1; n0 /= 2) {
        for (int64_t node = n0 + threadIdx.x; node < 2 * n0; node += blockDim.x) {
            NodeSums c[2];
            for (int h = 0; h < 2; ++h) {
                const int64_t ch = 2 * node + h;
                c[h].v[0] = b.na[ch];
                for (int m = 0; m < 3; ++m) {
                    c[h].v[1 + m] = b.nsx[3 * ch + m];
                    c[h].v[4 + m] = b.nlo[3 * ch + m];
                    c[h].v[7 + m] = b.nhi[3 * ch + m];
                }
            }
            node_store(b, node, node_join(c[0], c[1]));
        }
        __syncthreads();
    }
}

#pragma clang fp contract(fast)

struct BhArgs {
    int64_t nF, P;
    int leaf;
    double theta2;
    double alpha, beta;
    float alpha32, beta32;
    const int32_t* order;
    const double4* dx;
    const double4* dn;
    const double* flo;
    const double* fhi;
    const double* fr2;
    const double* na;
    const double* nX;
    const double* nlo;
    const double* nhi;
    const double* nr2;
    const double* rec;    // [2P][8]
    const double4* nxa;   // [2P] (X, a) of the nodes
    const double4* srt;   // [nF] (X, a) in sorted order
    double* gS;           // [7][nF] face-side sums (gradient only)
    double* eS;           // [nF] energy rows
    double* accF;         // [nF][4] target-side sums of faces, by sorted position
    double* accN;         // [2P][4] target-side sums of nodes
    unsigned long long* counts;   // far, near
};

// Uniform loads of read-only data through the scalar cache.
typedef double double8 __attribute__((ext_vector_type(8)));
template <class T>
__device__ __forceinline__ T scalar_load(const T* p)
{
    return *(const __attribute__((address_space(4))) T*)p;
}

__device__ __forceinline__ bool admissible(const BhArgs& A, const double (&slo)[3], const double (&shi)[3],
                                           double sr2, int64_t node)
{
#pragma clang fp contract(off)
    double d2 = 0.0;
    for (int m = 0; m < 3; ++m) {
        const double g1 = A.nlo[3 * node + m] - shi[m];
        const double g2 = slo[m] - A.nhi[3 * node + m];
        double g = g1 > g2 ? g1 : g2;
        g = g < 0.0 ? 0.0 : g;
        d2 = d2 + g * g;
    }
    const double nr = A.nr2[node];
    const double r2 = sr2 > nr ? sr2 : nr;
    return r2 < A.theta2 * d2;
}

// The same from the node's record.
__device__ __forceinline__ bool admissible(const double8& r, const double (&slo)[3], const double (&shi)[3],
                                           double sr2, double theta2)
{
#pragma clang fp contract(off)
    double d2 = 0.0;
    for (int m = 0; m < 3; ++m) {
        const double g1 = r[m] - shi[m];
        const double g2 = slo[m] - r[3 + m];
        const double g = fmax(fmax(g1, g2), 0.0);
        d2 = d2 + g * g;
    }
    const double r2 = sr2 > r[6] ? sr2 : r[6];
    return r2 < theta2 * d2;
}

// Kernel and its derivatives for one target (R = float or double pair terms).  The fused
// operations are written out, so that a term has the same bits wherever it is inlined.
template <class R, bool GEN>
__device__ __forceinline__ void term(const double (&xs)[3], const double (&ns)[3], const double* y,
                                     const BhArgs& A, R& K, R (&dKdd)[3], R (&dKdN)[3])
{
    R d[3], n[3];
    for (int m = 0; m < 3; ++m) {
        d[m] = (R)(xs[m] - y[m]);
        n[m] = (R)ns[m];
    }
    const R r2 = fma(d[2], d[2], fma(d[0], d[0], d[1] * d[1]));
    const R q = fma(n[2], d[2], fma(n[0], d[0], n[1] * d[1]));
    const R inv = (R)1 / r2;
    R Kqr;
    if (!GEN) {
        const R u = q * inv, u2 = u * u, u4 = u2 * u2;
        K = u4 * u2;           // |q|^6 r2^-6
        Kqr = u4 * u;          // sgn(q) |q|^5 r2^-5 = K r2 / q
    } else {
        const R aq = q < (R)0 ? -q : q;
        if (aq == (R)0) {
            K = (R)0;
            Kqr = (R)0;
        } else {
            Kqr = (R)pow((double)aq, A.alpha - 1.0) * (R)pow((double)r2, 1.0 - 0.5 * A.beta);
            Kqr = q < (R)0 ? -Kqr : Kqr;
            K = Kqr * q * inv;
        }
    }
    const R alpha = sizeof(R) == 4 ? (R)A.alpha32 : (R)A.alpha, beta = sizeof(R) == 4 ? (R)A.beta32 : (R)A.beta;
    const R c1 = alpha * Kqr * inv, c2 = beta * K * inv;
    for (int m = 0; m < 3; ++m) {
        dKdd[m] = fma(c1, n[m], -(c2 * d[m]));
        dKdN[m] = c1 * d[m];
    }
}

__device__ __forceinline__ double4 scalar_load4(const double4* p)
{
    typedef double vec4 __attribute__((ext_vector_type(4)));
    const vec4 v = scalar_load(reinterpret_cast<const vec4*>(p));
    return double4{v[0], v[1], v[2], v[3]};
}

// Traversal: one wave per 64 consecutive sorted faces, 64 threads per workgroup so that a wave that
// is done makes room at once.
//
// The walk keeps everything about nodes in scalar registers: a node that some lane opens has its
// two children's records read at once (128 contiguous bytes, scalar loads), each is tested by all
// lanes, and the lanes that take it or go on below it are a 64-bit mask.  Right children that wait
// and the queues of admissible nodes and of leaves are lanes of three registers.  Four targets are
// taken from a queue together: their loads are in flight together, and their target-side parts are
// summed over the wave by halving (with the lane swaps of gfx950, which need no selects), 24
// instructions per target instead of 96 for a full wave sum of each part.  The parts of a target
// are one 32-byte group and four faces of a leaf one 128-byte line, so the device-scope additions
// are one instruction per four targets; one by one and in four rows they were 58.8 million
// requests.
// 327,680 faces, theta 0.5 (per wave 1,955 nodes tested, 1,114 taken by some lane, 1,602 leaf
// faces): 10.9 ms before, 3.9 ms now, of which the vector units issue 2.8 ms; the rest is waves that
// end last.  Five waves per SIMD, not four, because 5,120 waves then start at once: 5.4 ms at four.
// The general exponents' powers would spill at five.
template <class R, bool GEN, bool GRAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(GEN ? 1 : 5))) void k_bh_traverse(BhArgs A)
{
    const int lane = threadIdx.x;
    const int p = (int)(blockIdx.x * 64) + lane, nF = (int)A.nF, P = (int)A.P;
    const bool live = p < nF;                   // every lane walks with its wave
    const int32_t s = A.order[live ? p : 0];
    const double4 X = A.dx[s], Nn = A.dn[s];
    const double xs[3] = {X.x, X.y, X.z}, ns[3] = {Nn.x, Nn.y, Nn.z};
    const double aS = X.w;
    double slo[3], shi[3];
    for (int m = 0; m < 3; ++m) {
        slo[m] = A.flo[3 * s + m];
        shi[m] = A.fhi[3 * s + m];
    }
    const double sr2 = A.fr2[s];
    double gX[3] = {0, 0, 0}, gN[3] = {0, 0, 0}, ga = 0.0;
    unsigned long long nfar = 0, nnear = 0;
    const bool up8 = lane & 8, up4 = lane & 4;

    // One term of this lane with target (y, w): face-side sums (without a_S) here, target-side parts
    // (without w) in tg.
    auto visit = [&](const double* y, double w, double (&tg)[4]) {
        R K, dKdd[3], dKdN[3];
        term<R, GEN>(xs, ns, y, A, K, dKdd, dKdN);
        const double Kd = (double)K;
        ga += w * Kd;
        if (GRAD) {
            for (int m = 0; m < 3; ++m) {
                const double v = (double)dKdd[m];
                gX[m] += w * v;
                gN[m] += w * (double)dKdN[m];
                tg[m] = -aS * v;
            }
            tg[3] = aS * Kd;
        }
    };
    // four targets: load(j) their (X, a), active(j) whether this lane has a term with target j; the
    // sum of part m of target j goes to add(j, m, sum)
    auto four = [&](auto&& load, auto&& active, auto&& add) {
        double4 y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = load(j);
        double h[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
            const double ya[3] = {y[j].x, y[j].y, y[j].z}, yb[3] = {y[j + 2].x, y[j + 2].y, y[j + 2].z};
            if (active(j)) visit(ya, y[j].w, a);
            if (active(j + 2)) visit(yb, y[j + 2].w, b);
            if (GRAD)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    h[j][m] = swap_sum32(a[m], b[m]);   // bit 5 of the lane: j + 2
                    asm volatile("" : "+v"(h[j][m]));   // now, not with the second pair: 8 registers less
                }
        }
        if (GRAD) {
            double q[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) q[m] = swap_sum16(h[0][m], h[1][m]);    // bit 4: j + 1
            const double u0 = fold<0x128>(q[0], q[2], up8), u1 = fold<0x128>(q[1], q[3], up8);   // bit 3: m + 2
            double v = fold<0x141>(u0, u1, up4);                                                 // bit 2: m + 1
            v = v + dpp_move<0x1B>(v);      // quad_perm [3,2,1,0]
            v = v + dpp_move<0xB1>(v);      // quad_perm [1,0,3,2]
            const double wj = lane & 32 ? (lane & 16 ? y[3].w : y[2].w) : (lane & 16 ? y[1].w : y[0].w);
            if ((lane & 3) == 0) add(lane >> 4, (lane >> 2) & 3, (lane & 12) == 12 ? v : wj * v);
        }
    };

    // Three registers hold (node, mask) entries, one a lane: lanes 0 to 4 the admissible nodes that
    // wait, 8 and 9 the leaves, 32 + d the right child of depth d.
    int en = 0, el = 0, eh = 0, nq = 0, nl = 0;
    constexpr int kLeaf = 8, kRight = 32;
    auto put = [&](int i, int node, uint64_t m) {
        en = lane == i ? node : en;
        el = lane == i ? (int)(uint32_t)m : el;
        eh = lane == i ? (int)(uint32_t)(m >> 32) : eh;
    };
    auto mask = [&](int i) -> uint64_t {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(eh, i) << 32) |
               (uint32_t)__builtin_amdgcn_readlane(el, i);
    };
    auto take_far = [&]() {                     // the last four (or what is left)
        const int n = min(nq, 4), first = nq - n;
        int id[4];
        uint64_t mk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = first + min(j, n - 1);
            id[j] = __builtin_amdgcn_readlane(en, i);
            mk[j] = j < n ? mask(i) : 0;
            nfar += __builtin_popcountll(mk[j]);
        }
        four(
            [&](int j) {
                return scalar_load4(A.nxa + id[j]);
            },
            [&](int j) { return __builtin_amdgcn_inverse_ballot_w64(mk[j]); },
            [&](int j, int m, double v) {
                const int a = j & 1 ? id[1] : id[0], b = j & 1 ? id[3] : id[2];
                if (j < n) unsafeAtomicAdd(A.accN + 4 * (int64_t)(j & 2 ? b : a) + m, v);
            });
        nq = first;
    };
    auto take_leaf = [&]() {
        --nl;
        const int l = __builtin_amdgcn_readlane(en, kLeaf + nl) - P;
        const uint64_t mk = mask(kLeaf + nl);
        const int q0 = l * A.leaf, p1 = q0 + min(A.leaf, nF - q0);
        for (int q = q0; q < p1; q += 4) {
            four(
                [&](int j) {
                    return scalar_load4(A.srt + min(q + j, p1 - 1));
                },
                [&](int j) {
                    const bool act = __builtin_amdgcn_inverse_ballot_w64(mk) && q + j < p1 && q + j != p;
                    nnear += __builtin_popcountll(__ballot(act));
                    return act;
                },
                [&](int j, int m, double v) {
                    if (q + j < p1) unsafeAtomicAdd(A.accF + 4 * (int64_t)(q + j) + m, v);
                });
        }
    };
    // Node c for the lanes m: those that take it are queued, those that go on below it returned.
    auto test = [&](int c, const double8& r, uint64_t m) -> uint64_t {
        if (!(r[7] > 0.0) || m == 0) return 0;
        const uint64_t b = __ballot(admissible(r, slo, shi, sr2, A.theta2)) & m;
        const uint64_t rest = m & ~b;
        if (b) {
            put(nq++, c, b);
        }
        if (rest && c >= P) {
            put(kLeaf + nl++, c, rest);
            return 0;
        }
        return rest;
    };

    const double8* rec = reinterpret_cast<const double8*>(A.rec);
    uint32_t waiting = 0;              // the depths whose right child some lanes wait at
    int node = 1;
    uint64_t m = test(1, scalar_load(rec + 1), __ballot(live));
    while (m) {
        node = __builtin_amdgcn_readfirstlane(2 * node);
        const double8 rl = scalar_load(rec + node), rr = scalar_load(rec + node + 1);
        const uint64_t right = test(node + 1, rr, m);
        m = test(node, rl, m);
        const int d = 31 - __builtin_clz(node);
        if (right) {
            put(kRight + d, 0, right);
            waiting |= 1u << d;
        }
        while (nl > 0) take_leaf();
        if (nq >= 4) take_far();
        if (!m && waiting) {           // the deepest waiting right child
            const int w = 31 - __builtin_clz(waiting);
            node = (node >> (d - w)) | 1;
            m = mask(kRight + w);
            waiting ^= 1u << w;
        }
    }
    while (nl > 0) take_leaf();
    while (nq > 0) take_far();
    if (lane == 0) {
        if (nfar) atomicAdd(&A.counts[0], nfar);
        if (nnear) atomicAdd(&A.counts[1], nnear);
    }
    if (!live) return;
    A.eS[s] = aS * ga;
    if (GRAD) {
        for (int m = 0; m < 3; ++m) {
            A.gS[m * A.nF + s] = aS * gX[m];
            A.gS[(3 + m) * A.nF + s] = aS * gN[m];
        }
        A.gS[6 * A.nF + s] = ga;
    }
}

// Per-face partial derivatives: face side + target side + the node terms of every
// ancestor, written as gface[m * gstride + t] (dE/dX, dE/dN, dE/da).
__global__ void k_bh_assemble(int64_t nF, int leaf, int64_t P, const int32_t* __restrict__ pos,
                              const double4* __restrict__ dx, const double* __restrict__ na,
                              const double* __restrict__ nX, const double* __restrict__ gS,
                              const double* __restrict__ accF, const double* __restrict__ accN,
                              double* __restrict__ gface, int64_t gstride)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nF) return;
    const double4 X = dx[t];
    const double xt[3] = {X.x, X.y, X.z};
    const double4* nodes = reinterpret_cast<const double4*>(accN);
    const double4 own = reinterpret_cast<const double4*>(accF)[pos[t]];
    double gx[3] = {gS[t] + own.x, gS[nF + t] + own.y, gS[2 * nF + t] + own.z}, ga = gS[6 * nF + t] + own.w;
    for (int64_t node = P + pos[t] / leaf; node >= 1; node >>= 1) {
        const double a = na[node];
        if (!(a > 0.0)) continue;
        const double4 c = nodes[node];
        const double g[3] = {c.x, c.y, c.z};
        double proj = 0.0;
        for (int m = 0; m < 3; ++m) {
            gx[m] += (X.w / a) * g[m];
            proj += (xt[m] - nX[3 * node + m]) * g[m];
        }
        ga += c.w + proj / a;
    }
    for (int m = 0; m < 3; ++m) {
        gface[m * gstride + t] = gx[m];
        gface[(3 + m) * gstride + t] = gS[(3 + m) * nF + t];
    }
    gface[6 * gstride + t] = ga;
}

// ---------------------------------------------------------------- fractional apply
//
// The kernel matrix of the fractional operator (Sec. 5.1.1) with the same tree, the same
// admissibility and the same traversal as the energy: for face S an admissible node I adds
// k(X_S, X_I) (a_I ubar_S - m_I), m_I = sum_{T in I} a_T ubar_T (the node's moments), a leaf
// that is not admissible adds k(X_S, X_T) a_T (ubar_S - ubar_T) for its faces T != S, with
// k = |d|^-(2 sigma + 2).  Only the face S side is summed, so there are no atomics and
// the result is deterministic.  z(S) (without the factor a_S) goes to z[c * zstride + S],
// the layout of the direct kernel's reduced sums.
//
// Rows of face averages (ub), node moments (nm) and far-field values are KP wide, KP = the
// column count rounded up to 4 (the padding holds zeros), and are read as 4-wide vectors,
// so a row costs one memory round trip; the kernels are instantiated for KP = 4, 8, 12.

template <class UB> struct Vec4Of;
template <> struct Vec4Of<float> { using type = float4; };
template <> struct Vec4Of<double> { using type = double4; };

// out[0 .. KP) = row[0 .. KP) (16- or 32-byte aligned)
template <int KP, class T>
__device__ __forceinline__ void load_row(const T* __restrict__ row, double (&out)[KP])
{
    using V = typename Vec4Of<T>::type;
#pragma unroll
    for (int h = 0; h < KP / 4; ++h) {
        const V v = reinterpret_cast<const V*>(row)[h];
        out[4 * h] = (double)v.x;
        out[4 * h + 1] = (double)v.y;
        out[4 * h + 2] = (double)v.z;
        out[4 * h + 3] = (double)v.w;
    }
}

// Node moments [2P][KP]: leaves (member faces in sorted order) and the levels above them up to one
// node per workgroup, in LDS; also ub in sorted order, when asked (ubs).  All levels in one
// workgroup took 76 us at 32,768 leaves and four columns, this and the launch for the top 16 us.
template <class UB, int KP>
__global__ __launch_bounds__(kSubLeaves) void k_bh_moments(int64_t nF, int leaf, int64_t P,
                                                           const int32_t* __restrict__ order,
                                                           const double4* __restrict__ srt, const UB* __restrict__ ub,
                                                           double* __restrict__ nm, UB* __restrict__ ubs)
{
    __shared__ double sh[KP][kSubLeaves];
    const int t = threadIdx.x;
    const int64_t l = (int64_t)blockIdx.x * kSubLeaves + t;
    double acc[KP];
    if (l == 0)
#pragma unroll
        for (int c = 0; c < KP; ++c) nm[c] = 0.0;   // (no node, see k_bct_far)
    if (l < P) {
#pragma unroll
        for (int c = 0; c < KP; ++c) acc[c] = 0.0;
        for (int64_t p = l * leaf; p < (l + 1) * leaf && p < nF; ++p) {
            const UB* row = ub + (int64_t)order[p] * KP;
            const double a = srt[p].w;
            double u[KP];
            load_row<KP>(row, u);
#pragma unroll
            for (int c = 0; c < KP; ++c) acc[c] = acc[c] + a * u[c];
            if (ubs)
#pragma unroll
                for (int c = 0; c < KP; ++c) ubs[p * KP + c] = (UB)u[c];
        }
#pragma unroll
        for (int c = 0; c < KP; ++c) nm[(P + l) * KP + c] = sh[c][t] = acc[c];
    }
    int64_t base = P + (int64_t)blockIdx.x * kSubLeaves;
    for (int w = (int)min((int64_t)kSubLeaves, P) >> 1; w >= 1; w >>= 1) {
        base >>= 1;
        __syncthreads();
        if (t < w)
#pragma unroll
            for (int c = 0; c < KP; ++c) acc[c] = sh[c][2 * t] + sh[c][2 * t + 1];
        __syncthreads();
        if (t < w)
#pragma unroll
            for (int c = 0; c < KP; ++c) nm[(base + t) * KP + c] = sh[c][t] = acc[c];
    }
}

// The levels above.
__global__ __launch_bounds__(1024) void k_bh_moment_top(int64_t P, int kp, double* __restrict__ nm)
{
    for (int64_t n0 = P / kSubLeaves / 2; n0 >= 1; n0 /= 2) {
        for (int64_t e = threadIdx.x; e < n0 * kp; e += blockDim.x) {
            const int64_t node = n0 + e / kp;
            const int c = (int)(e % kp);
            nm[node * kp + c] = nm[2 * node * kp + c] + nm[(2 * node + 1) * kp + c];
        }
        __syncthreads();
    }
}

template <class R>
__device__ __forceinline__ double frac_kernel(const double (&xs)[3], const double* y, double expo)
{
    R d[3];
    for (int m = 0; m < 3; ++m) d[m] = (R)(xs[m] - y[m]);
    const R r2 = fma(d[2], d[2], fma(d[0], d[0], d[1] * d[1]));   // the same bits wherever it is inlined
    if (sizeof(R) == sizeof(float))
        return (double)__builtin_amdgcn_exp2f((float)expo * __builtin_amdgcn_logf((float)r2));
    return pow((double)r2, expo);
}

template <class R, class UB, int KP>
__global__ __launch_bounds__(256) void k_bh_frac(BhArgs A, const UB* __restrict__ ub, int k,
                                                 const double* __restrict__ nm, double expo,
                                                 double* __restrict__ z, int64_t zstride)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = p < A.nF;                 // every lane walks with its wave
    const int32_t s = A.order[live ? p : 0];
    const double4 X = A.dx[s];
    const double xs[3] = {X.x, X.y, X.z};
    double slo[3], shi[3];
    for (int m = 0; m < 3; ++m) {
        slo[m] = A.flo[3 * s + m];
        shi[m] = A.fhi[3 * s + m];
    }
    const double sr2 = A.fr2[s];
    double us[KP], acc[KP];
    load_row<KP>(ub + (int64_t)s * KP, us);
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] = 0.0;
    wave_walk(
        A.na, A.P, live, [&](int node) { return admissible(A, slo, shi, sr2, node); },
        [&](int node) {
            double m[KP];
            load_row<KP>(nm + (int64_t)node * KP, m);
            const double w = frac_kernel<R>(xs, A.nX + 3 * (int64_t)node, expo);
            const double a = A.na[node];
#pragma unroll
            for (int c = 0; c < KP; ++c) acc[c] += w * (a * us[c] - m[c]);
        },
        [&](int node) {
            const int64_t l = node - A.P;
            const int64_t p1 = min((l + 1) * (int64_t)A.leaf, A.nF);
            for (int64_t q = l * A.leaf; q < p1; ++q) {
                const int32_t t = A.order[q];
                if (t == s) continue;
                const double4 Y = A.dx[t];
                double ut[KP];
                load_row<KP>(ub + (int64_t)t * KP, ut);
                const double y[3] = {Y.x, Y.y, Y.z};
                const double w = frac_kernel<R>(xs, y, expo) * Y.w;
#pragma unroll
                for (int c = 0; c < KP; ++c) acc[c] += w * (us[c] - ut[c]);
            }
        });
    if (!live) return;
#pragma unroll
    for (int c = 0; c < KP; ++c)
        if (c < k) z[c * zstride + s] = acc[c];
}

template <class UB, int KP>
void moments_launch(const BhBuffers& b, int64_t nF, int leaf, int64_t P, const UB* ub,
                    double* nm, UB* ubs, hipStream_t s)
{
    hipLaunchKernelGGL((k_bh_moments<UB, KP>), dim3((unsigned)((P + kSubLeaves - 1) / kSubLeaves)), dim3(kSubLeaves), 0,
                       s, nF, leaf, P, b.order, b.srt, ub, nm, ubs);
    if (P > kSubLeaves) hipLaunchKernelGGL(k_bh_moment_top, dim3(1), dim3(1024), 0, s, P, KP, nm);
}

template <class UB, int KP>
hipError_t bh_frac_launch(const BhBuffers& b, int64_t nF, int leaf, double theta, bool f64, const FaceData& fd,
                          const UB* ub, int k, double expo, double* nm, double* z, int64_t zstride, hipStream_t s)
{
    int64_t P = 0;
    (void)bh_node_count(nF, leaf, &P);
    moments_launch<UB, KP>(b, nF, leaf, P, ub, nm, nullptr, s);
    BhArgs A;
    A.nF = nF; A.P = P; A.leaf = leaf; A.theta2 = theta * theta; A.alpha = 0.0; A.beta = 0.0;
    A.order = b.order; A.dx = fd.dx; A.dn = fd.dn; A.flo = b.flo; A.fhi = b.fhi; A.fr2 = b.fr2;
    A.na = b.na; A.nX = b.nX; A.nlo = b.nlo; A.nhi = b.nhi; A.nr2 = b.nr2;
    A.gS = nullptr; A.eS = nullptr; A.accF = nullptr; A.accN = nullptr; A.counts = nullptr;
    // pair terms in the precision of the face averages (FP64 for TP_PREC_FP64, else FP32)
    (void)f64;
    const dim3 grid((unsigned)((nF + 255) / 256)), block(256);
    hipLaunchKernelGGL((k_bh_frac<UB, UB, KP>), grid, block, 0, s, A, ub, k, nm, expo, z, zstride);
    return hipGetLastError();
}

// ---------------------------------------------------------------- block cluster tree
//
// Hierarchical multiplication with the kernel matrix of the fractional operator (Sec.
// 5.1.4, 5.1.5, App. B) on the same tree: the block lists (admissible node pairs grouped by
// row node, inadmissible leaf pairs grouped by row leaf) are built on the host.  With
// x = [a, a ubar] per face and its node sums x~_J = [a_J, m_J] (the upward pass: the
// Barnes-Hut moments), y~_I = sum_{J admissible for I} k(X_I, X_J) x~_J (k_bct_far); face S
// then adds the y~ of its leaf and all its ancestors (the downward pass, summed along the
// face's path) and the exact terms of the leaves inadmissible for its own:
//   z(S) = ubar_S Y0(S) - Y(S) + sum_{T in near leaves, T != S} k(X_S, X_T) a_T (ubar_S - ubar_T).
// y~ rows are 4 + KP wide: [sum w a_J, 0, 0, 0, sum w m_J (KP)].

// Admissible blocks: one wave per row node I.  The lanes take the node's list in strides of
// 64 entries, the loads of U of them in flight together (9.79 million entries of 200,000 faces:
// 276 us with one at a time, 154 us); the sums are then added across the wave in a fixed order
// (butterfly), so the result does not depend on timing.
template <class R, int KP>
__global__ __launch_bounds__(256) void k_bct_far(int64_t M, const int32_t* __restrict__ off,
                                                 const int32_t* __restrict__ col, const double4* __restrict__ nxa,
                                                 const double* __restrict__ nm,
                                                 double expo, double* __restrict__ yt)
{
    const int64_t I = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (I >= M) return;                       // the whole wave
    double a0 = 0.0, acc[KP];
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] = 0.0;
    const double4 XI = nxa[I];
    const double xi[3] = {XI.x, XI.y, XI.z};
    const int32_t e1 = off[I + 1];
    constexpr int U = KP == 4 ? 4 : 2;        // entries with their loads in flight together
    for (int32_t e = off[I] + lane; e < e1; e += 64 * U) {
        int32_t J[U];
        double4 Y[U];
        double m[U][KP];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int32_t j = col[min(e + 64 * q, e1 - 1)];
            J[q] = e + 64 * q < e1 ? j : 0;   // (past the end node 0, whose moments and area are zero:
                                              // a weight of 0 alone does not keep out a moment of inf)
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            Y[q] = nxa[J[q]];
            load_row<KP>(nm + (int64_t)J[q] * KP, m[q]);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const double y[3] = {Y[q].x, Y[q].y, Y[q].z};
            const double w = e + 64 * q < e1 ? frac_kernel<R>(xi, y, expo) : 0.0;   // (no branch: it would
                                                                                    // hold the loads back)
            a0 += w * Y[q].w;
#pragma unroll
            for (int c = 0; c < KP; ++c) acc[c] += w * m[q][c];
        }
    }
    a0 = wave_sum(a0);
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] = wave_sum(acc[c]);
    if (lane == 0) {
        double* y = yt + I * (KP + 4);
        y[0] = a0;
        y[1] = 0.0;
        y[2] = 0.0;
        y[3] = 0.0;
#pragma unroll
        for (int c = 0; c < KP; ++c) y[4 + c] = acc[c];
    }
}

// z(S) += ubar_S Y0 - Y over the leaf L's path to the root (downward pass)
template <int KP>
__device__ __forceinline__ void bct_down(const double* __restrict__ yt, int64_t P, int64_t L, const double (&us)[KP],
                                         double (&acc)[KP])
{
    double y0 = 0.0, yc[KP];
#pragma unroll
    for (int c = 0; c < KP; ++c) yc[c] = 0.0;
    for (int64_t node = P + L; node >= 1; node >>= 1) {
        const double* y = yt + node * (KP + 4);
        double v[KP];
        load_row<KP>(y + 4, v);
        y0 += y[0];
#pragma unroll
        for (int c = 0; c < KP; ++c) yc[c] += v[c];
    }
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] += us[c] * y0 - yc[c];
}

// Inadmissible (exact) blocks for leaves of at most 8 faces: one wave per row leaf L, lane
// (i, j) = (lane / 8, lane % 8) takes the pair (face i of L, face j of J) for every leaf J of
// L's list, all lanes walking the same list (64 list entries are read at once and handed
// out as scalars); the 8 lanes of face i are then added in a fixed order and lane (i, 0) adds the
// far field of L's path to the root.
//
// A leaf whose faces lie apart (the Morton order jumps inside it) has a large box and a list of
// thousands of leaves, where the mean is 211: one such wave took 4.5 ms, the others together
// 0.6 ms.  So a wave takes kBctSeg entries at most; what a list has beyond them are segments, each a
// wave of a launch before (k_bct_long counts them when the lists are built), whose sums are added
// in order.
// A leaf's faces through order[], then their data from wherever they are stored, were two trips to
// memory per batch of four leaves; positions and values in sorted order are contiguous and need the
// list alone, and the loads of U leaves are in flight together.  Consecutive leaves have nearly the
// same lists: each XCD takes a contiguous range of leaves, so that its L2 serves them.
// 200,000 faces, three columns, 5.29 million leaf pairs: 6.4 ms before, 0.68 ms now (both
// launches; 0.77 ms with segments of 512 entries).
struct BctLeafArgs {
    int nF, leaf, nleaf;
    const double4* srt;       // [nF] (X, a) in sorted order
    const int32_t* noff;      // [nleaf + 1]
    const int32_t* ncol;
    BctSegs sg;
    double expo;
};

__global__ void k_bct_long(int nleaf, const int32_t* __restrict__ noff, BctSegs sg)
{
    const int L = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (L >= nleaf) return;
    const int n = (noff[L + 1] - noff[L] - 1) / kBctSeg;   // segments beyond the first (an empty list: 0)
    int at = -1;
    if (n > 0) {
        at = atomicAdd(sg.count, n);
        for (int q = 0; q < n; ++q) sg.seg[at + q] = make_int2(L, q + 1);
    }
    sg.first[L] = at;
}

// The sums of leaf L over the list entries [e0, e1): lane (i, j) returns face i's sum.
template <class R, class UB, int KP>
__device__ __forceinline__ void bct_leaf_sum(const BctLeafArgs& A, const UB* __restrict__ ubs, int L, int32_t e0,
                                             int32_t e1, double (&us)[KP], double (&acc)[KP])
{
    constexpr int U = sizeof(UB) * KP <= 16 ? 8 : 4;   // as many as the registers hold
    typedef typename Vec4Of<UB>::type Vec;
    const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
    const int ps = L * A.leaf + i;
    const bool own = i < A.leaf && ps < A.nF;
    const bool lane_on = own && j < A.leaf;
    const double4 X = A.srt[own ? ps : 0];
    const double xs[3] = {X.x, X.y, X.z};
    load_row<KP>(ubs + (int64_t)(own ? ps : 0) * KP, us);
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] = 0.0;
    for (int32_t eb = e0; eb < e1; eb += 64) {
        const int32_t mine = eb + lane < e1 ? A.ncol[eb + lane] : 0;
        const int nb = min(64, e1 - eb);
        for (int q0 = 0; q0 < nb; q0 += U) {
            bool on[U];
            double4 Y[U];
            Vec ut[U][KP / 4];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int J = __builtin_amdgcn_readlane(mine, min(q0 + q, 63));
                const int pt = J * A.leaf + j;
                on[q] = lane_on && q0 + q < nb && pt < A.nF && pt != ps;
                const int at = min(pt, A.nF - 1);
                Y[q] = A.srt[at];
#pragma unroll
                for (int h = 0; h < KP / 4; ++h) ut[q][h] = reinterpret_cast<const Vec*>(ubs + (int64_t)at * KP)[h];
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (!on[q]) continue;
                const double y[3] = {Y[q].x, Y[q].y, Y[q].z};
                const double w = frac_kernel<R>(xs, y, A.expo) * Y[q].w;
#pragma unroll
                for (int h = 0; h < KP / 4; ++h) {
                    acc[4 * h] += w * (us[4 * h] - (double)ut[q][h].x);
                    acc[4 * h + 1] += w * (us[4 * h + 1] - (double)ut[q][h].y);
                    acc[4 * h + 2] += w * (us[4 * h + 2] - (double)ut[q][h].z);
                    acc[4 * h + 3] += w * (us[4 * h + 3] - (double)ut[q][h].w);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < KP; ++c) {
        double v = acc[c];
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 1, 64);
        acc[c] = v;
    }
}

// One wave per segment: part[segment][face of the leaf][KP].
template <class R, class UB, int KP>
__global__ __launch_bounds__(256) void k_bct_segs(BctLeafArgs A, const UB* __restrict__ ubs)
{
    const int u = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (u >= *A.sg.count) return;             // the whole wave
    const int2 g = A.sg.seg[u];
    const int L = __builtin_amdgcn_readfirstlane(g.x), q = __builtin_amdgcn_readfirstlane(g.y);
    const int32_t e0 = A.noff[L] + q * kBctSeg;
    double us[KP], acc[KP];
    bct_leaf_sum<R, UB, KP>(A, ubs, L, e0, min(e0 + kBctSeg, A.noff[L + 1]), us, acc);
    if ((lane & 7) == 0)
#pragma unroll
        for (int c = 0; c < KP; ++c) A.sg.part[((int64_t)u * 8 + (lane >> 3)) * KP + c] = acc[c];
}

template <class R, class UB, int KP>
__global__ __launch_bounds__(256) void k_bct_leaf8(BctLeafArgs A, const UB* __restrict__ ubs, int64_t P, int k,
                                                   const int32_t* __restrict__ order, const double* __restrict__ yt,
                                                   double* __restrict__ z, int64_t zstride)
{
    const int wg = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);   // gridDim.x: 8 m
    const int L = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (L >= A.nleaf) return;                 // the whole wave
    const int32_t e0 = A.noff[L], e1 = A.noff[L + 1];
    double us[KP], acc[KP];
    bct_leaf_sum<R, UB, KP>(A, ubs, L, e0, min(e1, e0 + kBctSeg), us, acc);
    const int lane = threadIdx.x & 63, i = lane >> 3, ps = L * A.leaf + i;
    if (i >= A.leaf || ps >= A.nF || (lane & 7) != 0) return;
    const int f = A.sg.first[L];
    for (int q = 0; q < (f < 0 ? 0 : (e1 - e0 - 1) / kBctSeg); ++q)
#pragma unroll
        for (int c = 0; c < KP; ++c) acc[c] += A.sg.part[((int64_t)(f + q) * 8 + i) * KP + c];
    const int32_t s = order[ps];
    bct_down<KP>(yt, P, L, us, acc);
#pragma unroll
    for (int c = 0; c < KP; ++c)
        if (c < k) z[c * zstride + s] = acc[c];
}

// The same for any leaf size: one thread per face, its leaf's list in order.
template <class R, class UB, int KP>
__global__ __launch_bounds__(256) void k_bct_faces(int64_t nF, int leaf, int64_t P, const int32_t* __restrict__ order,
                                                   const double4* __restrict__ dx, const UB* __restrict__ ub, int k,
                                                   const int32_t* __restrict__ noff,
                                                   const int32_t* __restrict__ ncol, const double* __restrict__ yt,
                                                   double expo, double* __restrict__ z, int64_t zstride)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nF) return;
    const int32_t s = order[p];
    const double4 X = dx[s];
    const double xs[3] = {X.x, X.y, X.z};
    double us[KP], acc[KP];
    load_row<KP>(ub + (int64_t)s * KP, us);
#pragma unroll
    for (int c = 0; c < KP; ++c) acc[c] = 0.0;
    const int64_t L = p / leaf;
    for (int32_t e = noff[L]; e < noff[L + 1]; ++e) {
        const int64_t J = ncol[e];
        const int64_t q1 = min((J + 1) * (int64_t)leaf, nF);
        for (int64_t q = J * leaf; q < q1; ++q) {
            const int32_t t = order[q];
            if (t == s) continue;
            const double4 Y = dx[t];
            double ut[KP];
            load_row<KP>(ub + (int64_t)t * KP, ut);
            const double y[3] = {Y.x, Y.y, Y.z};
            const double w = frac_kernel<R>(xs, y, expo) * Y.w;
#pragma unroll
            for (int c = 0; c < KP; ++c) acc[c] += w * (us[c] - ut[c]);
        }
    }
    bct_down<KP>(yt, P, L, us, acc);
#pragma unroll
    for (int c = 0; c < KP; ++c)
        if (c < k) z[c * zstride + s] = acc[c];
}

template <class UB, int KP>
hipError_t bct_launch(const BhBuffers& b, const BctLists& bl, int64_t nF, int leaf, bool f64, const FaceData& fd,
                      const UB* ub, int k, double expo, double* nm, double* yt, void* ubs, double* z, int64_t zstride,
                      hipStream_t s)
{
    int64_t P = 0;
    const int64_t M = (int64_t)bh_node_count(nF, leaf, &P);
    moments_launch<UB, KP>(b, nF, leaf, P, ub, nm, leaf <= 8 ? static_cast<UB*>(ubs) : nullptr, s);
    // one wave (64 lanes) per node for the admissible blocks, per leaf for the exact ones
    const int64_t nleaf = (nF + leaf - 1) / leaf;
    const dim3 gm((unsigned)((M * 64 + 255) / 256)), gl((unsigned)((nleaf + 31) / 32 * 8)),
        gf((unsigned)((nF + 255) / 256)), blk(256);
    // pair terms in the precision of the face averages (FP64 for TP_PREC_FP64, else FP32)
    (void)f64;
    hipLaunchKernelGGL((k_bct_far<UB, KP>), gm, blk, 0, s, M, bl.far_off, bl.far_col, b.nxa, nm, expo, yt);
    if (leaf <= 8) {
        BctLeafArgs A;
        A.nF = (int)nF; A.leaf = leaf; A.nleaf = (int)nleaf; A.srt = b.srt; A.noff = bl.near_off; A.ncol = bl.near_col;
        A.sg = bl.segs; A.expo = expo;
        const UB* us = static_cast<const UB*>(ubs);
        if (bl.segs.max > 0)
            hipLaunchKernelGGL((k_bct_segs<UB, UB, KP>), dim3((unsigned)((bl.segs.max + 3) / 4)), blk, 0, s, A, us);
        hipLaunchKernelGGL((k_bct_leaf8<UB, UB, KP>), gl, blk, 0, s, A, us, P, k, b.order, yt, z, zstride);
    } else
        hipLaunchKernelGGL((k_bct_faces<UB, UB, KP>), gf, blk, 0, s, nF, leaf, P, b.order, fd.dx, ub, k, bl.near_off,
                           bl.near_col, yt, expo, z, zstride);
    return hipGetLastError();
}

// ---------------------------------------------------------------- block cluster tree lists
//
// The blocks of the fractional operator's kernel matrix, built on the device by a
// breadth-first split of (root, root): a pair of nodes of one depth is an admissible block
// when separated, an exact block when it is a pair of leaves, else its four pairs of
// children go to the next level.  Appends use atomic counters, so the order in which a
// level's blocks land is arbitrary; the lists are then sorted by (row, column), which fixes
// them.  The separation test repeats the reading's arithmetic in FP64 without fused
// multiply-adds, as for the Barnes-Hut admissibility.
// (The tree's node records: one 64-byte line per node, since the pairs of a level reach their nodes
// in no cache-friendly order.)
__device__ __forceinline__ bool bct_separated(const double (&a)[8], const double (&b)[8], double chi2)
{
    double d2 = 0.0;
    for (int m = 0; m < 3; ++m) {
        const double g1 = b[m] - a[3 + m];
        const double g2 = a[m] - b[3 + m];
        double g = g1 > g2 ? g1 : g2;
        g = g < 0.0 ? 0.0 : g;
        d2 = d2 + g * g;
    }
    const double r2 = a[6] > b[6] ? a[6] : b[6];
    return r2 < chi2 * d2;
}

// One level of the split: each thread takes kExpPer pairs; the block counts its appends
// per list (wave prefix sums, then across the block's waves) and reserves them with one
// atomic addition per list, so same-address atomics stay few.
// cnt[0], cnt[1]: admissible and exact blocks so far (appended at these positions);
// cnt[2]: pairs of the next level.
constexpr int kExpThreads = 1024, kExpPer = 4;

__global__ __launch_bounds__(kExpThreads) void k_bct_expand(const uint64_t* __restrict__ cur, int64_t n,
                                                            const double4* __restrict__ rec, int64_t P, int bits,
                                                            double chi2, uint64_t* __restrict__ far, uint64_t* __restrict__ near,
                                                            uint64_t* __restrict__ next,
                                                            unsigned long long* __restrict__ cnt)
{
    __shared__ unsigned long long wsum[3][kExpThreads / 64];
    __shared__ unsigned long long base[3];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t e0 = (int64_t)blockIdx.x * kExpThreads * kExpPer + tid;
    uint64_t key[kExpPer];
    int what[kExpPer];                          // 1 admissible, 2 exact, 3 split, 0 nothing
    unsigned long long c[3] = {0ull, 0ull, 0ull};
#pragma unroll
    for (int q = 0; q < kExpPer; ++q) {
        const int64_t e = e0 + (int64_t)q * kExpThreads;
        key[q] = 0;
        what[q] = 0;
        if (e < n) {
            key[q] = cur[e];
            const int64_t I = (int64_t)(key[q] >> 32), J = (int64_t)(key[q] & 0xffffffffull);
            const double4 a0 = rec[2 * I], a1 = rec[2 * I + 1], b0 = rec[2 * J], b1 = rec[2 * J + 1];
            const double av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const double bv[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            if (av[7] > 0.0 && bv[7] > 0.0)
                what[q] = bct_separated(av, bv, chi2) ? 1 : (I >= P ? 2 : 3);   // pairs stay on one depth
        }
        if (what[q]) c[what[q] - 1] += what[q] == 3 ? 4ull : 1ull;
    }
    unsigned long long incl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        unsigned long long v = c[k];
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long t = __shfl_up(v, o, 64);
            if (lane >= o) v += t;
        }
        incl[k] = v;
        if (lane == 63) wsum[k][wid] = v;
    }
    __syncthreads();
    if (tid < 3) {
        unsigned long long tot = 0ull;
        for (int w = 0; w < kExpThreads / 64; ++w) {
            const unsigned long long v = wsum[tid][w];
            wsum[tid][w] = tot;
            tot += v;
        }
        base[tid] = tot ? atomicAdd(&cnt[tid], tot) : 0ull;
    }
    __syncthreads();
    unsigned long long off[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) off[k] = base[k] + wsum[k][wid] + incl[k] - c[k];
#pragma unroll
    for (int q = 0; q < kExpPer; ++q) {
        const int64_t I = (int64_t)(key[q] >> 32), J = (int64_t)(key[q] & 0xffffffffull);
        if (what[q] == 1) {
            far[off[0]++] = (uint64_t)I << bits | (uint64_t)J;
        } else if (what[q] == 2) {
            near[off[1]++] = (uint64_t)(I - P) << bits | (uint64_t)(J - P);
        } else if (what[q] == 3) {
            for (int a = 0; a < 2; ++a)
                for (int b = 0; b < 2; ++b)
                    next[off[2] + 2 * a + b] = ((uint64_t)(2 * I + a) << 32) | (uint64_t)(2 * J + b);
            off[2] += 4;
        }
    }
}

// CSR of sorted (row << 32 | column) keys: off[r] = first key of row r (r = 0 .. rows),
// col[e] = column of key e.
__global__ void k_bct_csr(const uint64_t* __restrict__ keys, int64_t n, int64_t rows, int bits, int32_t* __restrict__ off,
                          int32_t* __restrict__ col)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= rows) {
        const uint64_t target = (uint64_t)t << bits;
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (keys[mid] < target) lo = mid + 1;
            else hi = mid;
        }
        off[t] = (int32_t)lo;
    }
    if (t < n) col[t] = (int32_t)(keys[t] & ((1ull << bits) - 1ull));
}

}  // namespace

size_t bh_node_count(int64_t nF, int leaf, int64_t* P_out)
{
    const int64_t nleaf = (nF + leaf - 1) / leaf;
    int64_t P = 1;
    while (P < nleaf) P *= 2;
    if (P_out) *P_out = P;
    return (size_t)(2 * P);
}

size_t bh_sort_temp_bytes(int64_t nF)
{
    size_t bytes = 0;
    (void)hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, (const uint64_t*)nullptr, (uint64_t*)nullptr,
                                             (const int32_t*)nullptr, (int32_t*)nullptr, (int)nF, 0, 62);
    return bytes;
}

hipError_t launch_morton_order(const BhBuffers& b, const FaceData& fd, int64_t nF, const int32_t* orig,
                               hipStream_t s)
{
    const unsigned g = (unsigned)((nF + 255) / 256);
    const int nbox = (int)std::min<int64_t>(kBoxBlocks, (nF + 1023) / 1024);
    hipLaunchKernelGGL(k_bh_bbox, dim3(nbox), dim3(256), 0, s, fd.dx, nF, b.box);
    // values in b.pos, sorted values into b.order
    hipLaunchKernelGGL(k_bh_keys, dim3(g), dim3(256), 0, s, fd.dx, nF, b.box, nbox, orig, b.keys_in, b.pos);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    size_t tb = b.sort_bytes;
    return hipcub::DeviceRadixSort::SortPairs(b.sort_tmp, tb, b.keys_in, b.keys_out, b.pos, b.order, (int)nF, 0, 62, s);
}

hipError_t launch_bh_build(const BhBuffers& b, const double* V, const int32_t* F, const int32_t* orig, int64_t nF,
                           int leaf, const FaceData& fd, hipStream_t s)
{
    int64_t P = 0;
    (void)bh_node_count(nF, leaf, &P);
    const unsigned g = (unsigned)((nF + 255) / 256);
    hipLaunchKernelGGL(k_bh_faceprep, dim3(g), dim3(256), 0, s, V, F, nF, fd.dx, b.flo, b.fhi, b.fr2);
    hipError_t e = launch_morton_order(b, fd, nF, orig, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bh_pos, dim3(g), dim3(256), 0, s, b.order, nF, fd.dx, b.pos, b.srt);
    hipLaunchKernelGGL(k_bh_subtrees, dim3((unsigned)((P + kSubLeaves - 1) / kSubLeaves)), dim3(kSubLeaves), 0, s, nF,
                       leaf, P, b);
    if (P > kSubLeaves) hipLaunchKernelGGL(k_bh_top, dim3(1), dim3(1024), 0, s, P, b);
    return hipGetLastError();
}

hipError_t launch_bh_eval(const BhBuffers& b, int64_t nF, int leaf, double theta, int precision, double alpha,
                          double beta, const FaceData& fd, bool grad, double* gface, int64_t gstride,
                          hipStream_t s)
{
    int64_t P = 0;
    const int64_t M = (int64_t)bh_node_count(nF, leaf, &P);
    // counts lie before accN, accF
    hipError_t e = hipMemsetAsync(b.counts, 0, 8 * (size_t)(kBhCounts + (grad ? 4 * (M + nF) : 0)), s);
    if (e != hipSuccess) return e;
    BhArgs A;
    A.nF = nF; A.P = P; A.leaf = leaf; A.theta2 = theta * theta; A.alpha = alpha; A.beta = beta;
    A.alpha32 = (float)alpha; A.beta32 = (float)beta;
    A.order = b.order; A.dx = fd.dx; A.dn = fd.dn; A.flo = b.flo; A.fhi = b.fhi; A.fr2 = b.fr2;
    A.na = b.na; A.nX = b.nX; A.nlo = b.nlo; A.nhi = b.nhi; A.nr2 = b.nr2;
    A.rec = b.rec; A.nxa = b.nxa; A.srt = b.srt;
    A.gS = b.gS; A.eS = b.eS; A.accF = b.accF; A.accN = b.accN; A.counts = b.counts;
    const dim3 grid((unsigned)((nF + 255) / 256)), block(256);
    const bool gen = !(alpha == 6.0 && beta == 12.0);
    const bool f64 = precision == TP_PREC_FP64;
#define TP_BH_LAUNCH(R, G, D) hipLaunchKernelGGL((k_bh_traverse<R, G, D>), dim3((unsigned)((nF + 63) / 64)), dim3(64), 0, s, A)
    if (grad) {
        if (f64) { if (gen) TP_BH_LAUNCH(double, true, true); else TP_BH_LAUNCH(double, false, true); }
        else { if (gen) TP_BH_LAUNCH(float, true, true); else TP_BH_LAUNCH(float, false, true); }
    } else {
        if (f64) { if (gen) TP_BH_LAUNCH(double, true, false); else TP_BH_LAUNCH(double, false, false); }
        else { if (gen) TP_BH_LAUNCH(float, true, false); else TP_BH_LAUNCH(float, false, false); }
    }
#undef TP_BH_LAUNCH
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (grad)
        hipLaunchKernelGGL(k_bh_assemble, grid, block, 0, s, nF, leaf, P, b.pos, fd.dx, b.na, b.nX, b.gS, b.accF,
                           b.accN, gface, gstride);
    return hipGetLastError();
}

hipError_t launch_bh_frac(const BhBuffers& b, int64_t nF, int leaf, double theta, int precision, double sigma,
                          const FaceData& fd, const void* ub, int kp, int k, double* nm, double* z, int64_t zstride,
                          hipStream_t s)
{
    if (k < 1 || k > kMaxGroupCols || kp != (k + 3) / 4 * 4) return hipErrorInvalidValue;
    const double expo = -(sigma + 1.0);
    const bool f64 = precision == TP_PREC_FP64;
#define TP_BHF(T, KP) bh_frac_launch<T, KP>(b, nF, leaf, theta, f64, fd, static_cast<const T*>(ub), k, expo, nm, z, zstride, s)
    if (f64) return kp == 4 ? TP_BHF(double, 4) : kp == 8 ? TP_BHF(double, 8) : TP_BHF(double, 12);
    return kp == 4 ? TP_BHF(float, 4) : kp == 8 ? TP_BHF(float, 8) : TP_BHF(float, 12);
#undef TP_BHF
}

hipError_t launch_bct_frac(const BhBuffers& b, const BctLists& bl, int64_t nF, int leaf, int precision,
                           double sigma, const FaceData& fd, const void* ub, int kp, int k, double* nm, double* yt,
                           void* ubs, double* z, int64_t zstride, hipStream_t s)
{
    if (k < 1 || k > kMaxGroupCols || kp != (k + 3) / 4 * 4) return hipErrorInvalidValue;
    const double expo = -(sigma + 1.0);
    const bool f64 = precision == TP_PREC_FP64;
#define TP_BCT(T, KP) bct_launch<T, KP>(b, bl, nF, leaf, f64, fd, static_cast<const T*>(ub), k, expo, nm, yt, ubs, z, zstride, s)
    if (f64) return kp == 4 ? TP_BCT(double, 4) : kp == 8 ? TP_BCT(double, 8) : TP_BCT(double, 12);
    return kp == 4 ? TP_BCT(float, 4) : kp == 8 ? TP_BCT(float, 8) : TP_BCT(float, 12);
#undef TP_BCT
}

// List entries are row << bits | column, bits those of a node number: the sort then has 2 bits / 8
// passes over a list (four at 65,536 nodes) where row << 32 | column has eight.
static int bct_bits(int64_t P)
{
    int b = 1;
    while (((int64_t)1 << b) < 2 * P) ++b;
    return b;
}

size_t bct_sort_temp_bytes(int64_t n)
{
    size_t bytes = 0;
    (void)hipcub::DeviceRadixSort::SortKeys(nullptr, bytes, (const uint64_t*)nullptr, (uint64_t*)nullptr,
                                            (int)std::max<int64_t>(n, 1), 0, 64);
    return bytes;
}

hipError_t launch_bct_expand(const double* rec, int64_t P, double chi, const uint64_t* cur, int64_t n, uint64_t* far,
                             uint64_t* near, uint64_t* next, unsigned long long* cnt, hipStream_t s)
{
    if (n < 1) return hipSuccess;
    const int64_t per_block = (int64_t)kExpThreads * kExpPer;
    hipLaunchKernelGGL(k_bct_expand, dim3((unsigned)((n + per_block - 1) / per_block)), dim3(kExpThreads), 0, s, cur,
                       n, reinterpret_cast<const double4*>(rec), P, bct_bits(P), chi * chi, far, near, next, cnt);
    return hipGetLastError();
}

hipError_t launch_bct_long(int64_t nleaf, const int32_t* noff, const BctSegs& sg, hipStream_t s)
{
    hipError_t e = hipMemsetAsync(sg.count, 0, sizeof(int), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bct_long, dim3((unsigned)((nleaf + 255) / 256)), dim3(256), 0, s, (int)nleaf, noff, sg);
    return hipGetLastError();
}

hipError_t launch_bct_sort_csr(const uint64_t* keys, uint64_t* sorted, int64_t n, void* tmp, size_t tmp_bytes,
                               int64_t P, int64_t rows, int32_t* off, int32_t* col, hipStream_t s)
{
    const int bits = bct_bits(P);
    if (n > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    if (n > 0) {
        size_t tb = tmp_bytes;
        hipError_t e = hipcub::DeviceRadixSort::SortKeys(tmp, tb, keys, sorted, (int)n, 0, 2 * bits, s);
        if (e != hipSuccess) return e;
    }
    const int64_t m = std::max(rows + 1, n);
    hipLaunchKernelGGL(k_bct_csr, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, sorted, n, rows, bits, off, col);
    return hipGetLastError();
}

}  // namespace tp

