// Skeletal density function on a grid (eq. 10A, 11, 12a, 13, 15, 16c, 17t).
//
// The boundary samples are put in Hilbert order (a stable sort of their
// quantised positions) and cut into leaves of 64 consecutive samples, four
// leaves to a parent, four parents to a grandparent and so on, every tree node
// with the FP64 bounding box of its samples.  Runs of a Hilbert curve are
// connected, so the boxes are compact at every level.
//
// One wave owns a brick of 16 grid nodes (4 x 2 x 2, 4 x 4 in the plane): lane
// = 16 g + n handles node n and, of every four samples, the g-th.  The wave
// walks the tree depth first, the four lane groups testing four siblings at a
// time, so it sees only what can matter to its own 16 nodes.
//
// Pass 1 finds each node's nearest sample (lowest original index on exact
// ties), its membership sign and the distance floor test.  These are discrete
// decisions, taken in FP64 from FP64 sample positions in both precisions, so
// the classification of every node is the one an FP64 evaluation makes.
//
// Pass 2 sums the kernel over the eps-approximate contact ball in the
// context's precision T.  Tree nodes outside every node's ball are dropped;
// a sample whose squared distance lies within 4e-6 (relative) of the ball's
// squared radius is re-tested in FP64.
//
// With r = eta / |xi| the kernel of eq. 15 on zeta = xi + i eta reduces to
//   phi = lambda / (2 pi sigma xi^2) * G(r) * P(r) / (1 + r^2)^2,
//   G = exp(-(r - 1)^2 / (2 sigma^2)),  P = (1 - i r)^2 outside, (1 + i r)^2 inside,
// so a pair costs one reciprocal square root, one exponential and one
// reciprocal, with no trigonometric calls.
//
// Two things make the FP32 sum cheap (FP64 contexts sum every pair):
//   - Far clusters by interpolation.  Seen from a node, a cluster that lies
//     wholly inside its ball and is small against its distance and against xi
//     contributes a smooth function of the sample position, so its samples
//     are replaced by a tensor grid of Chebyshev points over its box carrying
//     sum_j L_m(q_j) w_j n_j (L_m the Lagrange polynomials): the same pair
//     term over fewer points.  The orders follow the ellipse of analyticity
//     (error rho^-p below kInterpEps per cluster), one per axis, so flat
//     clusters get flat grids.
//   - Distances and projections on the matrix cores.  With both positions
//     relative to the cluster's centre, |p - q|^2 = |p|^2 + (-2 q, |q|^2).(p, 1) and
//     (p - q).wn = (wn, -q.wn).(p, 1): two 16 x 16 x 4 FP32 MFMAs give 16 nodes x 16
//     samples of each, 9 of the 23 vector instructions of a pair.  Clusters
//     closer than their own radius cancel too much, and those with a record that
//     is not finite would reach nodes that they do not concern: these take FP64
//     differences, sample by sample.
// Bound by VALU issue (88% busy): about 60 instructions per 16 x 16 pairs beyond
// the 14 of each pair's term.  Measured, whole builds on 128^3 nodes: 242k samples
// of a union of 2000 spheres 322 -> 64 ms, 15.7k samples of a box with a bore 23.0
// -> 10.3 ms (from one 256-node brick per block with LDS tiles of 256 samples,
// every pair of the visited tiles summed); error against 64 bits of the latter
// 6.9e-7 -> 2.2e-7 (2-norm).
#include <algorithm>
#include <type_traits>

#include "block_order.hpp"
#include "common.hpp"
#include "launch.hpp"

namespace sdf {

namespace {

constexpr int kSdfBlock = 256;
constexpr int kSdfTile = 256;
constexpr int kLeaf = 64;       // samples per leaf
constexpr int kFan = 4;         // children per tree node
constexpr int kMaxLevels = 14;  // 64 * 4^13 > 2^30 samples
constexpr int kBrick = 16;      // grid nodes per wave
static_assert(kSdfTile == kLeaf * kFan, "a 256-sample tile is a first-level tree node");

// interpolation of far clusters: error target of one cluster, largest order
// per axis, largest share of a cluster's samples worth replacing, and the
// factor of xi that bounds the accepted size (at sigma = 0.5, the Gaussian's
// width in r)
constexpr double kInterpEps = 1e-6;
constexpr int kInterpMax = 12;
constexpr double kInterpShare = 0.4;
constexpr double kInterpXi = 1.2;
constexpr int kInterpSplit = 2048;  // samples per block of the weight sums

// relative half-width of the band around the ball's squared radius that is
// decided in FP64.  FP32 squared distances are nearer than that: FP64 differences
// give them to 4e-7; the matrix form sums |p|^2, -2 p.q and |q|^2, at most (|p| + |q|)^2
// <= 9 d^2 where it is used (|q| <= d), in five roundings of 6e-8.
constexpr double kBallBand = 4e-6;

template <typename T>
struct __align__(4 * sizeof(T)) v4 {
    T x, y, z, w;
};
using f32x4 = float __attribute__((ext_vector_type(4)));

// FP32 uses the hardware approximations directly (about 1 ulp each):
// v_rsq_f32 (live pairs have d^2 >= xi_floor^2, far from denormals),
// v_exp_f32 on a base-2 argument of magnitude below about 7, and v_rcp_f32.
// FP64 uses the correctly rounded library functions.
template <typename T>
__device__ __forceinline__ T fast_rsqrt(T x);
template <>
__device__ __forceinline__ float fast_rsqrt<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <>
__device__ __forceinline__ double fast_rsqrt<double>(double x) { return rsqrt(x); }

template <typename T>
__device__ __forceinline__ T dev_exp2(T x);
template <>
__device__ __forceinline__ float dev_exp2<float>(float x) { return __builtin_amdgcn_exp2f(x); }
template <>
__device__ __forceinline__ double dev_exp2<double>(double x) { return exp2(x); }

template <typename T>
__device__ __forceinline__ T dev_rcp(T x);
template <>
__device__ __forceinline__ float dev_rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <>
__device__ __forceinline__ double dev_rcp<double>(double x) { return 1.0 / x; }

// ---- sample tree
struct TreeNode {
    double lo[3], hi[3];  // box of the node's samples (infinite if one is not finite)
    double c[3];          // grid-lattice point nearest the box centre: origin of the node's FP32 records
    float reach2;         // square of the distance and xi from which its interpolation points stand in; < 0: none
    float qmax2;          // leaves: largest squared sample distance from c; infinite for a node with a sample whose
                          // position is not finite or whose record is not plain
    int px;               // first 16-point record group of the interpolation points
    int order;            // their orders per axis, 4 bits each
};
struct SampleTree {
    const TreeNode* node;
    int levels;            // level 0: leaves; the top level has at most kFan nodes
    int off[kMaxLevels];   // first node of each level
    int cnt[kMaxLevels];
};

__host__ __device__ inline int order_count(int o) { return (o & 15) * ((o >> 4) & 15) * ((o >> 8) & 15); }

// most interpolation points of a cluster of `size` samples, in whole groups of 16
__host__ __device__ inline int interp_cap(int64_t size) {
    const int64_t m = int64_t(kInterpShare * double(size));
    const int64_t top = int64_t(kInterpMax) * kInterpMax * kInterpMax;
    return int(((m < top ? m : top) + 15) / 16 * 16);
}

__device__ __forceinline__ double dist2(double dx, double dy, double dz) {
    return __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
}
// least and largest squared distance from p to a node's box
__device__ __forceinline__ double node_dmin2(const TreeNode& t, double px, double py, double pz) {
    const double dx = fmax(0.0, fmax(t.lo[0] - px, px - t.hi[0]));
    const double dy = fmax(0.0, fmax(t.lo[1] - py, py - t.hi[1]));
    const double dz = fmax(0.0, fmax(t.lo[2] - pz, pz - t.hi[2]));
    return dist2(dx, dy, dz);
}
__device__ __forceinline__ double node_dmax2(const TreeNode& t, double px, double py, double pz) {
    const double dx = fmax(t.hi[0] - px, px - t.lo[0]);
    const double dy = fmax(t.hi[1] - py, py - t.lo[1]);
    const double dz = fmax(t.hi[2] - pz, pz - t.lo[2]);
    return dist2(dx, dy, dz);
}

// Sibling groups of a depth-first walk: a level, the first of its (up to
// four) siblings, and per level the siblings still to visit, 4 bits each.
struct Walk {
    int l, base;
    uint64_t pend;
    __device__ __forceinline__ int take() {  // next sibling of the current group (there is one)
        const int m = int(pend >> (4 * l)) & 15;
        pend &= ~(uint64_t(m & -m) << (4 * l));
        return base + __builtin_ctz(unsigned(m));
    }
    __device__ __forceinline__ void down(int i) {
        --l;
        base = kFan * i;
    }
    // climbs to the nearest level with siblings left; false at the end
    __device__ __forceinline__ bool climb(int levels) {
        while (((pend >> (4 * l)) & 15) == 0) {
            if (++l >= levels) return false;
            base = (base >> 2) & ~3;
        }
        return true;
    }
};
// bit g set if any lane of lane group g has its bit in m
__device__ __forceinline__ int group_any(uint64_t m) {
    return (m & 0xffffull ? 1 : 0) | (m & 0xffff0000ull ? 2 : 0) | (m & 0xffff00000000ull ? 4 : 0) |
           (m >> 48 ? 8 : 0);
}

// bricks of kBrick nodes
struct BrickGrid {
    int sx, sy, sz, nx, ny, nz;
};
__host__ __device__ inline BrickGrid wave_bricks(int gx, int gy, int gz) {
    BrickGrid b{4, gz == 1 ? 4 : 2, gz == 1 ? 1 : 2, 0, 0, 0};
    b.nx = (gx + b.sx - 1) / b.sx;
    b.ny = (gy + b.sy - 1) / b.sy;
    b.nz = (gz + b.sz - 1) / b.sz;
    return b;
}

// the nearer of two candidates (Hilbert positions): lower squared distance,
// then lower original index
__device__ __forceinline__ void nearer(double d2, int s, const int* __restrict__ js, double& best, int& sbest) {
    if (d2 < best || (d2 == best && sbest >= 0 && s >= 0 && js[s] < js[sbest])) {
        best = d2;
        sbest = s;
    }
}

// Pass 1 (FP64) for the wave's 16 nodes: squared distance to the nearest
// sample and its Hilbert position (-1: no finite sample), the lowest original
// index on exact ties, in all four lanes of a node.  With WPB = 4 the wave sees
// the sub-th quarter of every leaf.
template <int WPB>
__device__ __forceinline__ void wave_nearest(const double* __restrict__ qs, const int* __restrict__ js,
                                             const TreeNode* __restrict__ nodes, const SampleTree& tr, int64_t ns,
                                             double px, double py, double pz, bool valid, int sub, double& best,
                                             int& sbest, unsigned long long* visited) {
    const int gq = (int(threadIdx.x) & 63) >> 4;
    best = INFINITY;          // over the samples this lane has seen
    double bound = INFINITY;  // over those its node's four lanes have seen
    sbest = -1;
    int first = -1;  // the leaf of the first bound
    auto leaf_nearest = [&](int leaf) {
        const int64_t s0 = int64_t(leaf) * kLeaf;
        const int cnt = int(ns - s0 < kLeaf ? ns - s0 : kLeaf);
        if (visited && valid)
            for (int a = 4 * sub + gq; a < cnt; a += 4 * WPB) ++*visited;
#pragma unroll 4
        for (int a = 4 * sub + gq; a < cnt; a += 4 * WPB) {
            const int64_t s = s0 + a;
            nearer(dist2(px - qs[3 * s], py - qs[3 * s + 1], pz - qs[3 * s + 2]), int(s), js, best, sbest);
        }
        bound = fmin(best, __shfl_xor(best, 16));
        bound = fmin(bound, __shfl_xor(bound, 32));
    };
    {
        // a first bound from the leaf found by going down towards the brick
        // (its first node), the nearest sibling at every level
        const double ax = __shfl(px, 0), ay = __shfl(py, 0), az = __shfl(pz, 0);
        int at = 0;
        for (int l = tr.levels - 1; l >= 0; --l) {
            const int c = at + gq;
            double d = c < tr.cnt[l] ? node_dmin2(nodes[tr.off[l] + c], ax, ay, az) : INFINITY;
            int id = c;
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1) {
                const double d1 = __shfl_xor(d, off);
                const int i1 = __shfl_xor(id, off);
                if (d1 < d || (d1 == d && i1 < id)) {
                    d = d1;
                    id = i1;
                }
            }
            id = __builtin_amdgcn_readfirstlane(id);
            if (l == 0) leaf_nearest(first = id);
            else at = kFan * id;
        }
    }
    {
        Walk w{tr.levels - 1, 0, 0};
        auto test = [&]() {
            const int c = w.base + gq;
            // prune only beyond rounding of either side; NaN bounds (no finite sample yet) keep walking
            const bool hit = valid && c < tr.cnt[w.l] &&
                             !(node_dmin2(nodes[tr.off[w.l] + c], px, py, pz) > bound * (1.0 + 1e-9));
            w.pend |= uint64_t(group_any(__ballot(hit))) << (4 * w.l);
        };
        test();
        while (w.climb(tr.levels)) {
            const int c = w.take();
            if (w.l == 0) {
                if (c != first) leaf_nearest(c);  // that one is seen
            } else {
                w.down(c);
                test();
            }
        }
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const double d1 = __shfl_xor(best, off);
        const int s1 = __shfl_xor(sbest, off);
        nearer(d1, s1, js, best, sbest);
    }
}

// eq. 3a: lambda1 gb(xi / R - 1) + i lambda2 gb(xi / R + 1), FP64, defined on the
// boundary too (no floor); gb truncates at |x| > eps
template <typename T>
__device__ __forceinline__ cplx<T> dsl_value(double xi, const ParamDesc& prm) {
    const double x1 = xi / prm.radius - 1.0, x2 = xi / prm.radius + 1.0;
    const double c = 1.0 / (2.5066282746310002 * prm.sigma);
    const double h = -0.5 / (prm.sigma * prm.sigma);
    const double re = fabs(x1) <= prm.eps ? prm.lambda1 * c * exp(h * x1 * x1) : 0.0;
    const double im = fabs(x2) <= prm.eps ? prm.lambda2 * c * exp(h * x2 * x2) : 0.0;
    return mk(T(re), T(im));
}
// membership of p from its nearest sample j
__device__ __forceinline__ int side_of(const double* __restrict__ q, const double* __restrict__ nrm, int64_t j,
                                       double px, double py, double pz) {
    const double dot =
        (px - q[3 * j]) * nrm[3 * j] + (py - q[3 * j + 1]) * nrm[3 * j + 1] + (pz - q[3 * j + 2]) * nrm[3 * j + 2];
    return dot > 0.0 ? 1 : (dot < 0.0 ? -1 : 0);
}
// The kernel sum of a node at squared distance `best` from its nearest sample:
// exp(-(r - 1)^2 / (2 sigma^2)) = 2^(-u^2) with u = (r - 1) gs,
// gs = sqrt(log2(e) / 2) / sigma, and u = eta (gs / xi) - gs
template <typename T, int PHI>
struct NodeSum {
    T inv_xi2, gs, inv_xi_gs;
    T re = T(0), im = T(0);  // sums of coef (1 - r^2) and of coef eta
    __device__ __forceinline__ NodeSum(double best, double xi, double sigma) {
        const double gs64 = std::sqrt(0.5 * 1.4426950408889634) / sigma;
        inv_xi2 = T(1.0 / best);
        gs = T(gs64);
        inv_xi_gs = T(gs64 / xi);
    }
    __device__ __forceinline__ void add(T d2, T wdot) {
        const T inv_eta = fast_rsqrt(d2);
        const T eta = d2 * inv_eta;
        T coef = wdot * inv_eta;
        if constexpr (PHI == kPhiSkeletal) {
            const T u = eta * inv_xi_gs - gs;
            coef *= dev_exp2(-u * u);
        }
        const T den = T(1) + d2 * inv_xi2;
        coef *= dev_rcp(den * den);
        re += coef * (T(1) - d2 * inv_xi2);
        im += coef * eta;
    }
    __device__ __forceinline__ cplx<T> value(int side, double best, double xi, const ParamDesc& prm) const {
        const double lam = side > 0 ? prm.lambda1 : -prm.lambda2;
        const T scale = T(lam / (2.0 * 3.14159265358979323846 * prm.sigma * best));
        const T im_sign = side > 0 ? T(-2) : T(2);  // P = (1 - r^2) -+ 2 i r, applied once per node
        return mk(re * scale, im * (im_sign * (T(1.0 / xi) * scale)));
    }
};

// PHI: the kernel of eq. 13 (kPhi* in launch.hpp): skeletal (eq. 15),
// inverse-square (eq. 15 with the medial Gaussian at its peak: the pair
// term without the exponential), or the double skin layer of eq. 3a, which
// needs only the signed distance of pass 1.
// FAST (FP32): pass 2 over the FP32 records with interpolated far clusters and
// MFMA distances; otherwise over the FP64 samples, pair by pair.
// WPB: waves per brick.  4 waves share the samples of a brick (and meet in
// LDS after each pass) where a grid has too few bricks to fill the chip.
// STATS (measurement builds only): adds to stats[0..2] the node-sample pairs
// evaluated in pass 1, the pairs (and interpolation points) evaluated in pass
// 2, and the pairs inside the contact ball, represented ones included.
template <typename T, int PHI, bool FAST, int WPB, bool STATS = false>
__global__ __launch_bounds__(64 * WPB, STATS ? 3 : (FAST ? 7 : 4)) void sdf_build_kernel(const double* __restrict__ q,
                                                              const double* __restrict__ nrm,
                                                              const double* __restrict__ qs,
                                                              const double* __restrict__ wn,
                                                              const int* __restrict__ js,
                                                              const TreeNode* __restrict__ nodes, SampleTree tr,
                                                              const float* __restrict__ rec1,
                                                              const float* __restrict__ rec2, int64_t ns, GridDesc g,
                                                              ParamDesc prm, cplx<T>* __restrict__ out,
                                                              unsigned long long* __restrict__ stats, int64_t brick0) {
    static_assert(WPB == 1 || WPB == 4, "waves per brick");
    __shared__ double sh_best[WPB == 4 ? 256 : 1];
    __shared__ __align__(8) int sh_idx[WPB == 4 ? 256 : 2];
    const int lane = int(threadIdx.x) & 63, sub = WPB == 1 ? 0 : uniform(int(threadIdx.x) >> 6);
    const int n = lane & 15, gq = lane >> 4;
    const int64_t brick = brick0 + blockIdx.x;
    const BrickGrid bg = wave_bricks(g.nx, g.ny, g.nz);
    // Consecutive blocks go to the XCDs and their shader engines in turn, so a
    // row of bricks as long as a multiple of their number would give each
    // engine one column of the grid, whose work differs several times over:
    // every row starts at another column.
    const int by = int((brick / bg.nx) % bg.ny), bz = int(brick / (int64_t(bg.nx) * bg.ny));
    const int bx = int((brick + 5 * by + 11 * bz) % bg.nx);
    const int i = bx * bg.sx + (n & 3), j = by * bg.sy + ((n >> 2) & (bg.sy - 1)),
              k = bz * bg.sz + (n >> 2) / bg.sy;
    const bool valid = i < g.nx && j < g.ny && k < g.nz;
    const double px = g.ox + g.h * i, py = g.oy + g.h * j, pz = g.oz + g.h * k;
    unsigned long long vis1 = 0, vis2 = 0, inball = 0;

    // ---- pass 1 (FP64): nearest sample, lowest original index on exact ties
    double best;
    int sbest;
    wave_nearest<WPB>(qs, js, nodes, tr, ns, px, py, pz, valid, sub, best, sbest, STATS ? &vis1 : nullptr);
    if constexpr (WPB == 4) {
        sh_best[threadIdx.x] = best;
        sh_idx[threadIdx.x] = sbest;
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) nearer(sh_best[64 * wv + n], sh_idx[64 * wv + n], js, best, sbest);
        __syncthreads();
    }
    const int64_t jb = sbest >= 0 ? js[sbest] : 0;
    const int pmc = side_of(q, nrm, jb, px, py, pz);
    const double xi_abs64 = sqrt(best);
    const bool writer = valid && gq == 0 && sub == 0;
    cplx<T>* dst = out + (int64_t(k) * g.ny + j) * g.nx + i;
    if constexpr (PHI == kPhiDsl) {
        if (writer) *dst = dsl_value<T>(pmc * xi_abs64, prm);
        return;
    }
    const bool live = valid && pmc != 0 && xi_abs64 >= prm.xi_floor;

    // ---- pass 2 (T): truncated kernel sum over the contact ball
    const double r2max64 = (1.0 + prm.eps) * (1.0 + prm.eps) * best;
    const T r2lo = T(r2max64 * (1.0 - kBallBand)), r2hi = T(r2max64 * (1.0 + kBallBand));
    const float r2mid = float(r2max64), r2gap = float(r2max64 * kBallBand), r2above = r2mid * (1.f + 2.4e-7f);
    NodeSum<T, PHI> acc(best, xi_abs64, prm.sigma);
    auto edge_in = [&](int64_t s) {  // the ball test of sample s in FP64
        return dist2(px - qs[3 * s], py - qs[3 * s + 1], pz - qs[3 * s + 2]) <= r2max64;
    };
    // 16 samples (or interpolation points) per group from group `grp0` on, with
    // positions relative to c; s0: Hilbert position of the first sample.  A node
    // that the item does not concern takes d^2 = 1 and w.d = 0: no lane is masked.
    auto matrix_item = [&](auto cut_tag, const double c[3], int grp0, int ngrp, bool mine, int64_t s0) {
        constexpr bool cut = decltype(cut_tag)::value;
        const float fx = float(px - c[0]), fy = float(py - c[1]), fz = float(pz - c[2]);
        const float b = !mine ? 0.f : (gq == 0 ? fx : (gq == 1 ? fy : (gq == 2 ? fz : 1.f)));
        const float p2 = mine ? fx * fx + fy * fy + fz * fz : 1.f;
        const f32x4 cc = {p2, p2, p2, p2}, zero = {0.f, 0.f, 0.f, 0.f};
        // a group's operands through buffer descriptors: scalar offsets, no vector address arithmetic
        const int last = ngrp - 1;
        const auto d1 = buffer_rsrc(rec1 + 64 * int64_t(grp0), uint32_t(ngrp) * 256);
        const auto d2r = buffer_rsrc(rec2 + 64 * int64_t(grp0), uint32_t(ngrp) * 256);
        auto load1 = [&](int gr) {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(d1, 4 * lane, 256 * min(gr, last), 0));
        };
        auto load2 = [&](int gr) {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(d2r, 4 * lane, 256 * min(gr, last), 0));
        };
        auto terms = [&](f32x4 d2, f32x4 wd, int gr) {
            if constexpr (cut) {
                const float gap = fminf(fminf(fabsf(d2[0] - r2mid), fabsf(d2[1] - r2mid)),
                                        fminf(fabsf(d2[2] - r2mid), fabsf(d2[3] - r2mid)));
                if (gap <= r2gap) {  // near the sphere: FP64 decides, and d^2 is moved to its side
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int64_t sr = s0 + 16 * gr + 4 * gq + r;
                        if (fabsf(d2[r] - r2mid) <= r2gap && sr < ns)
                            d2[r] = edge_in(sr) ? fminf(d2[r], r2mid) : fmaxf(d2[r], r2above);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (STATS && mine && d2[r] <= r2mid && s0 + 16 * gr + 4 * gq + r < ns) ++inball;
                    wd[r] = d2[r] <= r2mid ? wd[r] : 0.f;
                }
            }
            if (STATS && mine) vis2 += 4;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc.add(T(d2[r]), T(wd[r]));
        };
        // the next group's operands load under this group's terms; seven waves per SIMD hide the rest
        float u0 = load1(sub), v0 = load2(sub);
        for (int gr = sub; gr < ngrp; gr += WPB) {
            const f32x4 da = __builtin_amdgcn_mfma_f32_16x16x4f32(u0, b, cc, 0, 0, 0);
            const f32x4 wa = __builtin_amdgcn_mfma_f32_16x16x4f32(v0, b, zero, 0, 0, 0);
            u0 = load1(gr + WPB);
            v0 = load2(gr + WPB);
            terms(da, wa, gr);
        }
    };
    // the pairs of a leaf by differences, taken in FP64: a leaf may be as wide as
    // the part (sparse samples, a window of a larger part), and rounded about its
    // centre the positions would carry 6e-8 of its radius into a short distance
    auto plain_leaf = [&](int leaf) {
        const int64_t s0 = int64_t(leaf) * kLeaf;
        const int cnt = int(ns - s0 < kLeaf ? ns - s0 : kLeaf);
        if (!live) return;
        for (int a = 4 * sub + gq; a < cnt; a += 4 * WPB) {
            const int64_t s = s0 + a;
            const T dx = T(px - qs[3 * s]), dy = T(py - qs[3 * s + 1]), dz = T(pz - qs[3 * s + 2]);
            T wx, wy, wz;
            if constexpr (FAST) {
                const int64_t o = (s >> 4) * 64 + (s & 15);
                wx = T(rec2[o]);
                wy = T(rec2[o + 16]);
                wz = T(rec2[o + 32]);
            } else {
                wx = T(wn[3 * s]);
                wy = T(wn[3 * s + 1]);
                wz = T(wn[3 * s + 2]);
            }
            const T d2 = dx * dx + dy * dy + dz * dz;
            if (STATS) ++vis2;
            if (d2 <= r2hi) {
                const bool in = d2 <= r2lo || edge_in(s);
                if (in) {
                    if (STATS) ++inball;
                    acc.add(d2, dx * wx + dy * wy + dz * wz);
                }
            }
        }
    };
    {
        // accepted sizes: within kInterpXi of xi at sigma >= 0.5, less for narrower Gaussians
        const double fs = kInterpXi * fmin(1.0, 2.0 * prm.sigma);
        const double xi2 = fs * fs * best;
        const double r2out = r2max64 * (1.0 + 1e-9), r2in = r2max64 * (1.0 - 1e-9);
        Walk w{tr.levels - 1, 0, 0};
        auto visit = [&]() {  // tests four siblings, sums those that need no descent
            const int cnt = tr.cnt[w.l], off = tr.off[w.l];
            const int c = w.base + gq;
            const TreeNode& t = nodes[off + (c < cnt ? c : w.base)];
            const double dmin2 = node_dmin2(t, px, py, pz);
            const bool reach = live && c < cnt && !(dmin2 > r2out);
            const bool cut = reach && !(node_dmax2(t, px, py, pz) <= r2in);
            bool far = false;
            if constexpr (FAST)
                far = t.reach2 >= 0.f &&
                      double(t.reach2) <= fmin(xi2, dist2(px - 0.5 * (t.lo[0] + t.hi[0]), py - 0.5 * (t.lo[1] + t.hi[1]),
                                                          pz - 0.5 * (t.lo[2] + t.hi[2])));
            const uint64_t m_reach = __ballot(reach), m_cut = __ballot(cut);
            const uint64_t m_fail = FAST ? __ballot(reach && (cut || !far)) : m_reach;
            const uint64_t m_near = __ballot(reach && (w.l > 0 || dmin2 < double(t.qmax2)));
            int open = group_any(m_reach);
            const int cuts = group_any(m_cut), fails = group_any(m_fail), nears = group_any(m_near);
            int later = 0;
            while (open) {
                const int e = __builtin_ctz(unsigned(open));
                open &= open - 1;
                const TreeNode& te = nodes[off + w.base + e];
                const bool mine = (m_reach >> (16 * e + n)) & 1;
                if (FAST && !((fails >> e) & 1)) {
                    matrix_item(std::false_type{}, te.c, uniform(te.px), uniform((order_count(te.order) + 15) >> 4), mine,
                                0);
                    if (STATS && mine && gq == 0 && sub == 0) {
                        const int64_t size = int64_t(kLeaf) << (2 * w.l), s0 = size * (w.base + e);
                        inball += ns - s0 < size ? ns - s0 : size;
                    }
                } else if (w.l > 0) {
                    later |= 1 << e;
                } else if (FAST && !((nears >> e) & 1)) {
                    const bool ce = (cuts >> e) & 1;
                    const int64_t s0 = int64_t(w.base + e) * kLeaf;
                    const int cnt_s = int(ns - s0 < kLeaf ? ns - s0 : kLeaf);
                    if (ce) matrix_item(std::true_type{}, te.c, int(s0 >> 4), (cnt_s + 15) >> 4, mine, s0);
                    else matrix_item(std::false_type{}, te.c, int(s0 >> 4), (cnt_s + 15) >> 4, mine, s0);
                    if (STATS && !ce && mine)
                        for (int a = 4 * sub + gq; a < cnt_s; a += 4 * WPB) ++inball;
                } else {
                    plain_leaf(w.base + e);
                }
            }
            w.pend |= uint64_t(later) << (4 * w.l);
        };
        if (__ballot(live)) {
            visit();
            while (w.climb(tr.levels)) {
                w.down(w.take());
                visit();
            }
        }
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        acc.re += __shfl_xor(acc.re, off);
        acc.im += __shfl_xor(acc.im, off);
    }
    if constexpr (WPB == 4) {
        double* sh_im = reinterpret_cast<double*>(sh_idx);  // 64 sums fit
        if (gq == 0) {
            sh_best[16 * sub + n] = double(acc.re);
            sh_im[16 * sub + n] = double(acc.im);
        }
        __syncthreads();
        acc.re = T(sh_best[n]);
        acc.im = T(sh_im[n]);
#pragma unroll
        for (int wv = 1; wv < 4; ++wv) {
            acc.re += T(sh_best[16 * wv + n]);
            acc.im += T(sh_im[16 * wv + n]);
        }
    }
    if constexpr (STATS) {
        unsigned long long c[3] = {vis1, vis2, inball};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            for (int off = 32; off > 0; off >>= 1) c[a] += __shfl_xor(c[a], off);
            if (lane == 0) atomicAdd(stats + a, c[a]);
        }
    }
    if (writer) *dst = live ? acc.value(pmc, best, xi_abs64, prm) : mk(T(0), T(0));
}

// brick of nodes handled by one block
struct Brick {
    int bx, by, bz;
};
__host__ __device__ inline Brick brick_shape(int nz) { return nz == 1 ? Brick{16, 16, 1} : Brick{8, 8, 4}; }

// Few samples, many nodes: a thread per node walks all samples in their given
// order, with no sort and no tree (both passes' decisions are those of the tree
// kernels: FP64, the lowest index on ties).  Sample indices are uniform, so
// positions come through the scalar cache; w n goes through LDS.  Bound by VALU
// issue, some 30 instructions a pair; on small grids a chain of one sample after
// the other.
constexpr int kFewMax = 576;
template <typename T, int PHI>
__global__ __launch_bounds__(kSdfBlock) void sdf_few_kernel(const double* __restrict__ q,
                                                            const double* __restrict__ nrm,
                                                            const double* __restrict__ w, int ns, GridDesc g,
                                                            ParamDesc prm, cplx<T>* __restrict__ out, int64_t brick0) {
    __shared__ v4<T> wn[kFewMax];
    if constexpr (PHI != kPhiDsl) {
        for (int a = int(threadIdx.x); a < ns; a += kSdfBlock)
            wn[a] = v4<T>{T(w[a] * nrm[3 * a]), T(w[a] * nrm[3 * a + 1]), T(w[a] * nrm[3 * a + 2]), T(0)};
        __syncthreads();
    }
    const Brick br = brick_shape(g.nz);
    const int64_t nbx = (g.nx + br.bx - 1) / br.bx, nby = (g.ny + br.by - 1) / br.by, blk = brick0 + blockIdx.x;
    const int t = int(threadIdx.x);
    const int i = int(blk % nbx) * br.bx + t % br.bx, j = int(blk / nbx % nby) * br.by + t / br.bx % br.by,
              k = int(blk / (nbx * nby)) * br.bz + t / (br.bx * br.by);
    if (i >= g.nx || j >= g.ny || k >= g.nz) return;
    const double px = g.ox + g.h * i, py = g.oy + g.h * j, pz = g.oz + g.h * k;
    double best = INFINITY;
    int jb = 0;
#pragma unroll 4
    for (int a = 0; a < ns; ++a) {
        const double d2 = dist2(px - q[3 * a], py - q[3 * a + 1], pz - q[3 * a + 2]);
        if (d2 < best) {
            best = d2;
            jb = a;
        }
    }
    const int side = side_of(q, nrm, jb, px, py, pz);
    const double xi = sqrt(best);
    cplx<T>* dst = out + (int64_t(k) * g.ny + j) * g.nx + i;
    if constexpr (PHI == kPhiDsl) {
        *dst = dsl_value<T>(side * xi, prm);
        return;
    }
    if (!(side != 0 && xi >= prm.xi_floor)) {
        *dst = mk(T(0), T(0));
        return;
    }
    const double r2max = (1.0 + prm.eps) * (1.0 + prm.eps) * best;
    const T r2lo = T(r2max * (1.0 - kBallBand)), r2hi = T(r2max * (1.0 + kBallBand));
    NodeSum<T, PHI> acc(best, xi, prm.sigma);
#pragma unroll 2
    for (int a = 0; a < ns; ++a) {
        const double ex = px - q[3 * a], ey = py - q[3 * a + 1], ez = pz - q[3 * a + 2];
        const T dx = T(ex), dy = T(ey), dz = T(ez);
        const T d2 = dx * dx + dy * dy + dz * dz;
        if (d2 <= r2hi && (d2 <= r2lo || dist2(ex, ey, ez) <= r2max)) {
            const v4<T> m = wn[a];
            acc.add(d2, dx * m.x + dy * m.y + dz * m.z);
        }
    }
    *dst = acc.value(side, best, xi, prm);
}

// Samples in Hilbert order with per-tile bounding boxes.
struct SampleTiles {
    const double* qs;   // positions, n x 3
    const double* wn;   // w_j n_j, n x 3
    const int* js;      // original index of each sample
    const double* box;  // per tile of kSdfTile samples: lo x, y, z, hi x, y, z
    int64_t ntile;
};

__device__ __forceinline__ double box_dmin2(const double bl[3], const double bh[3], const double* __restrict__ t) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d = fmax(0.0, fmax(t[a] - bh[a], bl[a] - t[3 + a]));
        s += d * d;
    }
    return s;
}
__device__ __forceinline__ double box_dmax2(const double bl[3], const double bh[3], const double* __restrict__ t) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d = fmax(fabs(t[3 + a] - bl[a]), fabs(bh[a] - t[a]));
        s += d * d;
    }
    return s;
}

template <bool MAX>
__device__ __forceinline__ double block_reduce(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off);
        v = MAX ? fmax(v, o) : fmin(v, o);
    }
    __syncthreads();  // red is free
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int wv = 1; wv < kSdfBlock / 64; ++wv) v = MAX ? fmax(v, red[wv]) : fmin(v, red[wv]);
    return v;
}

// least squared distance between a brick's box and a tree node's
__device__ __forceinline__ double box_gap2(const double bl[3], const double bh[3], const TreeNode& t) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d = fmax(0.0, fmax(t.lo[a] - bh[a], bl[a] - t.hi[a]));
        s += d * d;
    }
    return s;
}

// ---- radial-basis affinity (eq. 2, continuum form): Gaussian shells of
// radius R around the +R (skin) and -R (core) offsets of the boundary.
// The offset points come as samples whose "w n" slot holds their complex
// weight (lambda1 w, 0) or (0, lambda2 w); a node sums
//   c_j g_sigma(|p - s_j| / R - 1)  over |(|p - s_j| / R - 1)| <= eps,
// i.e. over the shell R max(0, 1 - eps) <= |p - s_j| <= R (1 + eps), whose
// edges are decided in FP64 (squared radii within 1e-4 are re-tested).
template <typename T>
__global__ __launch_bounds__(kSdfBlock) void sdf_radial_kernel(SampleTiles st, int64_t ns, GridDesc g,
                                                               ParamDesc prm, cplx<T>* __restrict__ out) {
    __shared__ v4<double> sq[2 * kSdfTile];
    __shared__ int sidx[kSdfTile];
    __shared__ int tflag[kSdfBlock];
    v4<T>* sq2 = reinterpret_cast<v4<T>*>(sq);             // (sx, sy, sz, -) relative to the brick
    v4<T>* sn2 = reinterpret_cast<v4<T>*>(sq) + kSdfTile;  // (c.re, c.im, -, -)

    const Brick br = brick_shape(g.nz);
    const int nbx = (g.nx + br.bx - 1) / br.bx, nby = (g.ny + br.by - 1) / br.by;
    const int blk = blockIdx.x;
    const int i0 = (blk % nbx) * br.bx, j0 = ((blk / nbx) % nby) * br.by, k0 = (blk / (nbx * nby)) * br.bz;
    const int li = threadIdx.x % br.bx, lj = (threadIdx.x / br.bx) % br.by, lk = threadIdx.x / (br.bx * br.by);
    const int i = i0 + li, j = j0 + lj, k = k0 + lk;
    const bool valid = i < g.nx && j < g.ny && k < g.nz;
    const double cx = g.ox + g.h * i0, cy = g.oy + g.h * j0, cz = g.oz + g.h * k0;
    const double rx = g.h * li, ry = g.h * lj, rz = g.h * lk;
    const double px = cx + rx, py = cy + ry, pz = cz + rz;
    const double bl[3] = {cx, cy, cz};
    const double bh[3] = {cx + g.h * (min(br.bx, g.nx - i0) - 1), cy + g.h * (min(br.by, g.ny - j0) - 1),
                          cz + g.h * (min(br.bz, g.nz - k0) - 1)};

    const double rhi = prm.radius * (1.0 + prm.eps);
    const double rlo = prm.eps < 1.0 ? prm.radius * (1.0 - prm.eps) : 0.0;
    const double hi2 = rhi * rhi, lo2 = rlo * rlo;
    const T hi2a = T(hi2 * (1.0 - 1e-4)), hi2b = T(hi2 * (1.0 + 1e-4));
    const T lo2a = T(lo2 * (1.0 - 1e-4)), lo2b = T(lo2 * (1.0 + 1e-4));
    // g_sigma(eta / R - 1) = 2^(-u^2) / (sqrt(2 pi) sigma), u = (eta / R - 1) gs
    const double gs64 = std::sqrt(0.5 * 1.4426950408889634) / prm.sigma;
    const T gs = T(gs64), inv_r_gs = T(gs64 / prm.radius);
    const T prx = T(rx), pry = T(ry), prz = T(rz);
    T acc_re = T(0), acc_im = T(0);
    for (int64_t c0 = 0; c0 < st.ntile; c0 += kSdfBlock) {
        const int64_t tc = c0 + threadIdx.x;
        __syncthreads();
        tflag[threadIdx.x] = tc < st.ntile && box_dmin2(bl, bh, st.box + 6 * tc) <= hi2 * (1.0 + 1e-9) &&
                             !(box_dmax2(bl, bh, st.box + 6 * tc) < lo2 * (1.0 - 1e-9));
        __syncthreads();
        const int nchunk = int(st.ntile - c0 < kSdfBlock ? st.ntile - c0 : kSdfBlock);
        for (int kk = 0; kk < nchunk; ++kk) {
            if (!tflag[kk]) continue;  // uniform across the block
            const int64_t t0 = (c0 + kk) * kSdfTile;
            const int cnt = int(ns - t0 < kSdfTile ? ns - t0 : kSdfTile);
            __syncthreads();
            for (int a = threadIdx.x; a < cnt; a += kSdfBlock) {
                const int64_t s = t0 + a;
                sq2[a] = v4<T>{T(st.qs[3 * s] - cx), T(st.qs[3 * s + 1] - cy), T(st.qs[3 * s + 2] - cz), T(0)};
                sn2[a] = v4<T>{T(st.wn[3 * s]), T(st.wn[3 * s + 1]), T(0), T(0)};
                sidx[a] = int(s);
            }
            __syncthreads();
            if (valid) {
#pragma unroll 4
                for (int a = 0; a < cnt; ++a) {
                    const v4<T> sp = sq2[a];
                    const T dx = prx - sp.x, dy = pry - sp.y, dz = prz - sp.z;
                    const T d2 = dx * dx + dy * dy + dz * dz;
                    bool in = d2 <= hi2a && d2 >= lo2b;
                    if (!in && d2 <= hi2b && d2 >= lo2a) {  // near a shell edge: decide in FP64
                        const int64_t sj = sidx[a];
                        const double ex = px - st.qs[3 * sj], ey = py - st.qs[3 * sj + 1], ez = pz - st.qs[3 * sj + 2];
                        const double e2 = ex * ex + ey * ey + ez * ez;
                        in = e2 <= hi2 && e2 >= lo2;
                    }
                    if (in) {
                        const v4<T> cw = sn2[a];
                        const T u = sqrt(d2) * inv_r_gs - gs;
                        const T G = dev_exp2(-u * u);
                        acc_re += cw.x * G;
                        acc_im += cw.y * G;
                    }
                }
            }
        }
    }
    if (valid) {
        const T c = T(1.0 / (2.5066282746310002 * prm.sigma));
        out[(int64_t(k) * g.ny + j) * g.nx + i] = mk(acc_re * c, acc_im * c);
    }
}

// skin (+R n_j, weight (lambda1 w_j, 0)) and core (-R n_j, (0, lambda2 w_j))
// offset points of the samples, FP64, as a sample set of 2n points
__global__ void offset_points_kernel(const double* __restrict__ q, const double* __restrict__ nrm,
                                     const double* __restrict__ w, int64_t n, double R, double l1, double l2,
                                     double* __restrict__ q2, double* __restrict__ c2, double* __restrict__ w2) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q2[3 * j + a] = q[3 * j + a] + R * nrm[3 * j + a];
        q2[3 * (n + j) + a] = q[3 * j + a] - R * nrm[3 * j + a];
    }
    c2[3 * j] = l1;
    c2[3 * j + 1] = 0.0;
    c2[3 * j + 2] = 0.0;
    c2[3 * (n + j)] = 0.0;
    c2[3 * (n + j) + 1] = l2;
    c2[3 * (n + j) + 2] = 0.0;
    w2[j] = w[j];
    w2[n + j] = w[j];
}

// ---- adjoint with respect to the boundary samples
// L = Re sum_p g(p) rho(p).  With the nearest sample, membership and contact
// ball of every node held (FP64 throughout; the cotangent g comes in the
// context's precision), at a live node with nearest sample q* at xi:
//   d rho / d w_j = A c_j K(r_j),   d rho / d n_j = A w_j K(r_j) u_j,
//   d rho / d q_j = A w_j [-K(r_j) (n_j - c_j u_j) / eta_j - c_j K'(r_j) u_j / xi],
//   d rho / d xi  = -(2 rho + A sum_j w_j c_j K'(r_j) r_j) / xi,   d xi / d q* = -u*,
// with A = lambda / (2 pi sigma xi^2), K = G P / (1 + r^2)^2 as in the sum and
//   K' = K (-(r - 1) / sigma^2 - 4 r / (1 + r^2)) + G (-2 r + i s) / (1 + r^2)^2.
//
// The kernels below use FP64 exp, rsqrt and reciprocals of a few instructions
// (errors of about one unit in the last place): the sums are bound by them.

// exp(t), t <= 0: t = n ln 2 + f with ln 2 in two parts (Cody and Waite), |f| <= ln 2 / 2, Taylor to
// f^13 / 13! (4e-18)
__device__ __forceinline__ double exp_neg(double t) {
    t = fmax(t, -745.0);
    const double n = rint(t * 1.4426950408889634);
    const double f = __builtin_fma(n, -1.9082149292705877e-10, __builtin_fma(n, -0.6931471803691238, t));
    double p = 1.0 / 6227020800.0;
    p = __builtin_fma(p, f, 1.0 / 479001600.0);
    p = __builtin_fma(p, f, 1.0 / 39916800.0);
    p = __builtin_fma(p, f, 1.0 / 3628800.0);
    p = __builtin_fma(p, f, 1.0 / 362880.0);
    p = __builtin_fma(p, f, 1.0 / 40320.0);
    p = __builtin_fma(p, f, 1.0 / 5040.0);
    p = __builtin_fma(p, f, 1.0 / 720.0);
    p = __builtin_fma(p, f, 1.0 / 120.0);
    p = __builtin_fma(p, f, 1.0 / 24.0);
    p = __builtin_fma(p, f, 1.0 / 6.0);
    p = __builtin_fma(p, f, 0.5);
    p = __builtin_fma(p, f, 1.0);
    p = __builtin_fma(p, f, 1.0);
    return __builtin_amdgcn_ldexp(p, int(n));
}
// x^(-1/2) and 1 / x for normal x > 0: the hardware estimate (about 24 bits) and one cubic Newton step
__device__ __forceinline__ double rsqrt_step(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-x * y, y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp_step(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, __builtin_fma(e, e, e), y);
}

// sum over each row of 16 lanes, in every lane of the row
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double v) {
    v += row_move<0xb1>(v);   // quad_perm [1, 0, 3, 2]
    v += row_move<0x4e>(v);   // quad_perm [2, 3, 0, 1]
    v += row_move<0x124>(v);  // row_ror 4
    v += row_move<0x128>(v);  // row_ror 8
    return v;
}

// nearest samples and xi sums of the nodes in brick order
struct NearData {
    double* d2;
    double* sum;
    int* at;
};

// Node m of brick blk: 16 groups of 16 nodes, as the build's waves take them.
struct BrickNode {
    int i, j, k;
    bool valid;
    double x, y, z;
};
__device__ __forceinline__ BrickNode brick_node(const GridDesc& g, int64_t blk, int m) {
    const Brick br = brick_shape(g.nz);
    const int nbx = (g.nx + br.bx - 1) / br.bx, nby = (g.ny + br.by - 1) / br.by;
    const int grp = m >> 4, n = m & 15;
    const bool planar = g.nz == 1;
    BrickNode o;
    o.i = int(blk % nbx) * br.bx + (planar ? 4 * (grp & 3) : 4 * (grp & 1)) + (n & 3);
    o.j = int(blk / nbx % nby) * br.by +
          (planar ? 4 * (grp >> 2) + (n >> 2) : 2 * ((grp >> 1) & 3) + ((n >> 2) & 1));
    o.k = planar ? 0 : int(blk / (nbx * nby)) * br.bz + 2 * (grp >> 3) + (n >> 3);
    o.valid = o.i < g.nx && o.j < g.ny && o.k < g.nz;
    o.x = g.ox + g.h * o.i;
    o.y = g.oy + g.h * o.j;
    o.z = g.oz + g.h * o.k;
    return o;
}

// Pass 1 of the adjoint on its own: the nearest sample of every node in brick
// order (squared distance, place in tree order or -1), one wave per 16 nodes,
// and the nodes' xi sums cleared.
template <int WPB>
__global__ __launch_bounds__(64 * WPB) void adjoint_nearest_kernel(const double* __restrict__ qs,
                                                                   const int* __restrict__ js,
                                                                   const TreeNode* __restrict__ nodes, SampleTree tr,
                                                                   int64_t ns, GridDesc g, int64_t turn,
                                                                   NearData near) {
    __shared__ double sh_best[WPB == 4 ? 256 : 1];
    __shared__ int sh_idx[WPB == 4 ? 256 : 1];
    const int64_t grp = scattered_tile(blockIdx.x, gridDim.x, turn);
    const int lane = int(threadIdx.x) & 63, sub = WPB == 1 ? 0 : uniform(int(threadIdx.x) >> 6);
    const BrickNode b = brick_node(g, grp >> 4, int(grp & 15) * 16 + (lane & 15));
    double best;
    int sbest;
    wave_nearest<WPB>(qs, js, nodes, tr, ns, b.x, b.y, b.z, b.valid, sub, best, sbest, nullptr);
    if constexpr (WPB == 4) {
        sh_best[threadIdx.x] = best;
        sh_idx[threadIdx.x] = sbest;
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) nearer(sh_best[64 * wv + lane], sh_idx[64 * wv + lane], js, best, sbest);
    }
    if (sub == 0 && lane < 16) {
        near.d2[16 * grp + lane] = best;
        near.at[16 * grp + lane] = sbest;
        near.sum[16 * grp + lane] = 0.0;
    }
}

// xi term of the nearest sample: -(d rho / d xi) u*, u* = e / xi
__device__ __forceinline__ void add_xi_term(const double* __restrict__ q, int64_t jb, double x, double y, double z,
                                            double inv_xi, double sum, double* __restrict__ gq) {
    const double coef = inv_xi * inv_xi * sum;
    atomicAdd(gq + 3 * jb, coef * (x - q[3 * jb]));
    atomicAdd(gq + 3 * jb + 1, coef * (y - q[3 * jb + 1]));
    atomicAdd(gq + 3 * jb + 2, coef * (z - q[3 * jb + 2]));
}
__global__ __launch_bounds__(kSdfBlock) void adjoint_xi_kernel(const double* __restrict__ q,
                                                               const int* __restrict__ js, GridDesc g, NearData near,
                                                               double* __restrict__ gq) {
    const int64_t slot = int64_t(blockIdx.x) * kSdfBlock + threadIdx.x;
    const double sum = near.sum[slot];
    const int at = sum != 0.0 ? near.at[slot] : -1;
    const BrickNode b = brick_node(g, blockIdx.x, int(threadIdx.x));
    const double coef = sum / near.d2[slot];
    // lanes whose nearest sample is the same add up first: neighbours share
    // few, and one atomic each made them queue (58 -> 28 us at 64^3)
    unsigned long long todo = __ballot(at >= 0);
    while (todo) {
        const int first = __builtin_ctzll(todo);
        const int who = uniform(__shfl(at, first));
        const bool mine = at == who;
        todo &= ~__ballot(mine);
        const int64_t jb = js[who];
        double v[3] = {mine ? coef * (b.x - q[3 * jb]) : 0.0, mine ? coef * (b.y - q[3 * jb + 1]) : 0.0,
                       mine ? coef * (b.z - q[3 * jb + 2]) : 0.0};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[a] = row_sum(v[a]);
            v[a] += __shfl_xor(v[a], 16);
            v[a] += __shfl_xor(v[a], 32);
        }
        if ((threadIdx.x & 63) < 3)
            atomicAdd(gq + 3 * jb + (threadIdx.x & 63), (threadIdx.x & 63) == 0 ? v[0] : ((threadIdx.x & 63) == 1 ? v[1] : v[2]));
    }
}

// A block per brick of 256 nodes and range of leaves.  Every node's data goes
// to LDS (NEAR: its nearest sample is known, else pass 1 runs here); then each
// wave takes leaves: a lane owns one of the 64 samples and walks
// the nodes whose ball reaches the leaf, so that one evaluation of a pair's
// kernel serves both sums: the sample's seven gradient components stay in the
// lane's registers, and the node's xi term,
//   Re(g d rho / d xi) = -(1 / xi) sum_j w_j c_j Re(A g (2 K(r_j) + K'(r_j) r_j)),
// one value per pair, is summed over the lanes.  Samples are added to the
// gradients once per leaf and block by FP64 atomics (their order varies, so the
// last bits may vary between runs); blocks start at different leaves, so they
// do not add to the same addresses at a time.
// Bound by FP64 VALU issue, about 100 instructions per pair (a pass over the
// nodes and one over the samples, with the library's exp, took some 220), and
// on small grids by how evenly the pairs fall: bricks at the surface hold many
// times the mean.  There the leaves are split over more blocks than run at a
// time, which needs pass 1 done once, by itself: 3.9k samples on 64^3 nodes
// 2.2 ms with one block a brick, 1.85 in the bricks' order, 1.25 in a scattered one
// (the three kernels), 5.2 before all of this.
template <typename T, bool NEAR>
__global__ __launch_bounds__(kSdfBlock) void sdf_adjoint_kernel(const double* __restrict__ q,
                                                                const double* __restrict__ nrm,
                                                                const double* __restrict__ w,
                                                                const double* __restrict__ qs,
                                                                const int* __restrict__ js,
                                                                const TreeNode* __restrict__ nodes, SampleTree tr,
                                                                int64_t ns, GridDesc g, ParamDesc prm,
                                                                const cplx<T>* __restrict__ cot,
                                                                double* __restrict__ gq, double* __restrict__ gn,
                                                                double* __restrict__ gw, int64_t turn,
                                                                NearData near) {
    __shared__ v4<double> nodep[kSdfBlock];  // (px, py, pz, 1 / xi)
    __shared__ v4<double> nodeg[kSdfBlock];  // (A g.re, A g.im, ball radius^2 or -1, s)
    __shared__ double nsum[kSdfBlock];
    __shared__ int nnear[kSdfBlock];
    __shared__ double red[kSdfBlock / 64];

    const int64_t blk = scattered_tile(blockIdx.x, gridDim.x, turn);
    const int lane = int(threadIdx.x) & 63, wave = uniform(int(threadIdx.x) >> 6);
    const double sig2inv = 1.0 / (prm.sigma * prm.sigma);

    auto put_node = [&](const BrickNode& b, int m, double best, int sbest) {
        const int64_t jb = sbest >= 0 ? js[sbest] : 0;
        const double dot = (b.x - q[3 * jb]) * nrm[3 * jb] + (b.y - q[3 * jb + 1]) * nrm[3 * jb + 1] +
                           (b.z - q[3 * jb + 2]) * nrm[3 * jb + 2];
        const int pmc = dot > 0.0 ? 1 : (dot < 0.0 ? -1 : 0);
        const double xi = sqrt(best);
        const cplx<T> gt = b.valid ? cot[(int64_t(b.k) * g.ny + b.j) * g.nx + b.i] : mk(T(0), T(0));
        const double g_re = double(gt.re), g_im = double(gt.im);
        const bool act = b.valid && pmc != 0 && xi >= prm.xi_floor && (g_re != 0.0 || g_im != 0.0);
        const double lam = pmc > 0 ? prm.lambda1 : -prm.lambda2;
        const double A = lam / (2.0 * 3.14159265358979323846 * prm.sigma * best);
        nodep[m] = v4<double>{b.x, b.y, b.z, 1.0 / xi};
        nodeg[m] = v4<double>{A * g_re, A * g_im, act ? (1.0 + prm.eps) * (1.0 + prm.eps) * best : -1.0,
                              pmc > 0 ? -2.0 : 2.0};
        nnear[m] = int(jb);
        nsum[m] = 0.0;
    };
    if constexpr (NEAR) {
        const int m = int(threadIdx.x);
        put_node(brick_node(g, blk, m), m, near.d2[blk * kSdfBlock + m], near.at[blk * kSdfBlock + m]);
    } else {
        for (int grp = 4 * wave; grp < 4 * wave + 4; ++grp) {
            const int m = 16 * grp + (lane & 15);
            const BrickNode b = brick_node(g, blk, m);
            double best;
            int sbest;
            wave_nearest<1>(qs, js, nodes, tr, ns, b.x, b.y, b.z, b.valid, 0, best, sbest, nullptr);
            if (lane < 16) put_node(b, m, best, sbest);
        }
    }
    __syncthreads();
    const double r2brick = block_reduce<true>(nodeg[threadIdx.x].z, red) * (1.0 + 1e-9);
    if (r2brick < 0.0) return;  // uniform: no node of the brick contributes
    const Brick br = brick_shape(g.nz);
    const BrickNode b0 = brick_node(g, blk, 0);
    const double bl[3] = {b0.x, b0.y, b0.z};
    const double bh[3] = {bl[0] + g.h * (min(br.bx, g.nx - b0.i) - 1), bl[1] + g.h * (min(br.by, g.ny - b0.j) - 1),
                          bl[2] + g.h * (min(br.bz, g.nz - b0.k) - 1)};

    // this wave's leaves: every (4 splits)-th, walked from an offset of its own
    const int nleaf = tr.cnt[0], step = 4 * int(gridDim.y), first = 4 * int(blockIdx.y) + wave;
    const int own = first < nleaf ? (nleaf - first + step - 1) / step : 0;
    for (int t0 = 0; t0 < own; t0 += 64) {
        int lf = -1;
        if (t0 + lane < own) lf = first + step * int((unsigned(t0 + lane) + unsigned(blk)) % unsigned(own));
        const bool hit = lf >= 0 && box_gap2(bl, bh, nodes[lf]) <= r2brick;
        unsigned long long todo = __ballot(hit);
        while (todo) {
            const int from = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int leaf = uniform(__shfl(lf, from));
            const TreeNode& tn = nodes[leaf];
            const int64_t sidx = int64_t(leaf) * kLeaf + lane;
            const bool have = sidx < ns;
            const int64_t sj = js[have ? sidx : int64_t(leaf) * kLeaf];
            const double qx = q[3 * sj], qy = q[3 * sj + 1], qz = q[3 * sj + 2];
            const double nx = nrm[3 * sj], ny = nrm[3 * sj + 1], nz = nrm[3 * sj + 2];
            const double wj = w[sj];
            // sums of gk u, of e u, of -gk / eta and of c gk (see below)
            double b0 = 0.0, b1 = 0.0, b2 = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0, s1 = 0.0, aw = 0.0;
            bool any = false;
            for (int c0 = 0; c0 < kSdfBlock; c0 += 64) {
                const v4<double> np0 = nodep[c0 + lane];
                const unsigned long long reach =
                    __ballot(node_dmin2(tn, np0.x, np0.y, np0.z) <= nodeg[c0 + lane].z * (1.0 + 1e-9));
                for (int sg = 0; sg < 64; sg += 16) {
                    int bits = int(reach >> sg) & 0xffff;
                    if (!bits) continue;
                    double nacc = 0.0;
                    while (bits) {
                        const int b = __builtin_ctz(unsigned(bits));
                        bits &= bits - 1;
                        const v4<double> np = nodep[c0 + sg + b], ng = nodeg[c0 + sg + b];
                        const double dx = np.x - qx, dy = np.y - qy, dz = np.z - qz;
                        const double d2 = dist2(dx, dy, dz);
                        const bool in = have && d2 <= ng.z;
                        const double ie = rsqrt_step(d2);
                        const double ux = dx * ie, uy = dy * ie, uz = dz * ie;
                        const double c = ux * nx + uy * ny + uz * nz;
                        const double r = d2 * ie * np.w;
                        const double x = r - 1.0;
                        const double G = exp_neg(-0.5 * sig2inv * x * x);
                        const double iden = rcp_step(1.0 + r * r);
                        const double gi = G * iden * iden;
                        const double kre = gi * (1.0 - r * r), kim = gi * (ng.w * r);
                        const double f = -x * sig2inv - 4.0 * r * iden;
                        const double dre = kre * f - 2.0 * r * gi, dim = kim * f + ng.w * gi;
                        // Re(A g K), Re(A g K')
                        const double gk = in ? ng.x * kre - ng.y * kim : 0.0;
                        const double gkp = in ? ng.x * dre - ng.y * dim : 0.0;
                        any |= in;
                        aw += c * gk;
                        b0 += gk * ux;
                        b1 += gk * uy;
                        b2 += gk * uz;
                        // d rho / d q_j = w [t1 (n - c u) + t2 u] = w [t1 n + e u]
                        const double t1 = -gk * ie, e = -c * gkp * np.w - t1 * c;
                        s1 += t1;
                        e0 += e * ux;
                        e1 += e * uy;
                        e2 += e * uz;
                        const double v = row_sum(in ? wj * c * (2.0 * gk + r * gkp) : 0.0);
                        if ((lane & 15) == b) nacc = v;
                    }
                    if (nacc != 0.0) atomicAdd(nsum + c0 + sg + (lane & 15), nacc);
                }
            }
            if (any) {
                atomicAdd(gq + 3 * sj, wj * (s1 * nx + e0));
                atomicAdd(gq + 3 * sj + 1, wj * (s1 * ny + e1));
                atomicAdd(gq + 3 * sj + 2, wj * (s1 * nz + e2));
                atomicAdd(gn + 3 * sj, wj * b0);
                atomicAdd(gn + 3 * sj + 1, wj * b1);
                atomicAdd(gn + 3 * sj + 2, wj * b2);
                atomicAdd(gw + sj, aw);
            }
        }
    }
    __syncthreads();
    const double nv = nsum[threadIdx.x];
    if (nodeg[threadIdx.x].z >= 0.0 && nv != 0.0) {
        const v4<double> np = nodep[threadIdx.x];
        if constexpr (NEAR) atomicAdd(near.sum + blk * kSdfBlock + threadIdx.x, nv);
        else add_xi_term(q, nnear[threadIdx.x], np.x, np.y, np.z, np.w, nv, gq);
    }
}

// ---- Hilbert order and the sample tree
// 30-bit Hilbert index of a cell given by 10 bits per axis (Skilling's
// transpose algorithm, 2004)
__device__ __forceinline__ unsigned hilbert30(unsigned x, unsigned y, unsigned z) {
    unsigned X[3] = {x, y, z};
#pragma unroll
    for (unsigned Q = 512; Q > 1; Q >>= 1) {
        const unsigned P = Q - 1;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (X[a] & Q) {
                X[0] ^= P;
            } else {
                const unsigned t = (X[0] ^ X[a]) & P;
                X[0] ^= t;
                X[a] ^= t;
            }
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    unsigned t = 0;
#pragma unroll
    for (unsigned Q = 512; Q > 1; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1;
    unsigned key = 0;
#pragma unroll
    for (int b = 9; b >= 0; --b)
#pragma unroll
        for (int a = 0; a < 3; ++a) key = (key << 1) | (((X[a] ^ t) >> b) & 1u);
    return key;
}

// 10 bits per axis over the grid's box widened by 4 h (outside samples clamp)
__device__ __forceinline__ unsigned sample_key(const double* __restrict__ q, int64_t j, double ox, double oy,
                                               double oz, double inv_cell) {
    const double o[3] = {ox, oy, oz};
    unsigned c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double f = (q[3 * j + a] - o[a]) * inv_cell;
        c[a] = !(f > 0.0) ? 0u : (f >= 1023.0 ? 1023u : unsigned(f));
    }
    return hilbert30(c[0], c[1], c[2]);
}

__global__ void hilbert_key_kernel(const double* __restrict__ q, int64_t n, double ox, double oy, double oz,
                                   double inv_cell, unsigned* __restrict__ key, int* __restrict__ val) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
    key[j] = sample_key(q, j, ox, oy, oz, inv_cell);
    val[j] = int(j);
}

// Up to kSmallSort samples: keys and order in one launch.  Every block computes
// all keys, and ranks 64 samples: a wave counts the keys of its sixteenth that
// come before each lane's (equal keys keep their input order), and the sixteen
// counts add up to the sample's place.  n^2 comparisons, but spread over n / 64
// CUs and without a barrier between them, where a bitonic sort in one block is a
// chain of 45 to 78 LDS round trips: 512 samples 12.7 -> 5.5 us, 3.9k 41 ->
// 15; the radix sort's twenty launches take more than either.
constexpr int kSmallSort = 4096;
__global__ __launch_bounds__(1024) void small_order_kernel(const double* __restrict__ q, int n, double ox, double oy,
                                                           double oz, double inv_cell, int* __restrict__ order) {
    __shared__ __align__(16) unsigned key[kSmallSort];
    __shared__ int place[64];
    const int lane = int(threadIdx.x) & 63, wave = uniform(int(threadIdx.x) >> 6);
    const int n64 = (n + 63) & ~63;  // keys past the last are larger than any (30 bits)
    for (int j = int(threadIdx.x); j < n64; j += 1024)
        key[j] = j < n ? sample_key(q, j, ox, oy, oz, inv_cell) : ~0u;
    if (threadIdx.x < 64) place[threadIdx.x] = 0;
    __syncthreads();
    const int group = int(blockIdx.x), own = 64 * group + lane;
    const unsigned mine = key[own];
    int before = 0;
    for (int g = wave; g < n64 / 64; g += 16) {
        if (g != group) {
            const unsigned bound = mine + (g < group ? 1u : 0u);  // equal keys of earlier groups come before
#pragma unroll 4
            for (int i = 0; i < 64; i += 4) {
                const uint4 k = *reinterpret_cast<const uint4*>(key + 64 * g + i);
                before += int(k.x < bound) + int(k.y < bound) + int(k.z < bound) + int(k.w < bound);
            }
        } else {
            for (int i = 0; i < 64; ++i) {
                const unsigned k = key[64 * g + i];
                before += int(k < mine || (k == mine && i < lane));
            }
        }
    }
    atomicAdd(place + lane, before);
    __syncthreads();
    if (threadIdx.x < 64 && own < n) order[place[lane]] = own;
}

__device__ __forceinline__ double wave_min(double v) {
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    return v;
}

// grid-lattice point nearest v (node differences from it are exact for h a
// power of two)
__device__ __forceinline__ double lattice(double v, double o, double h) { return o + h * rint((v - o) / h); }

// MFMA records of a point: rec1 = (-2 q, |q|^2), rec2 = (w, -q.w), stored per
// 16 points component by component, so a wave's operand is one 256-byte load.
// A node that is not concerned multiplies them by zero, so records of matrix
// items have to be finite (true: all values are, with room for the sums of 2^30
// samples in the interpolation points).
constexpr float kRecordMax = 1e18f;
__device__ __forceinline__ bool put_record(float* __restrict__ rec1, float* __restrict__ rec2, int64_t at, float x,
                                           float y, float z, float wx, float wy, float wz) {
    const int64_t o = (at >> 4) * 64 + (at & 15);
    rec1[o] = -2.f * x;
    rec1[o + 16] = -2.f * y;
    rec1[o + 32] = -2.f * z;
    const float q2 = float(double(x) * x + double(y) * y + double(z) * z);
    const float qw = -float(double(x) * wx + double(y) * wy + double(z) * wz);
    rec1[o + 48] = q2;
    rec2[o] = wx;
    rec2[o + 16] = wy;
    rec2[o + 32] = wz;
    rec2[o + 48] = qw;
    // (a comparison with NaN is false)
    return q2 <= kRecordMax && fabsf(wx) + fabsf(wy) + fabsf(wz) + fabsf(qw) <= kRecordMax;
}

// One wave per leaf: samples gathered in Hilbert order, the leaf's box, and
// its FP32 records relative to the lattice point nearest the box centre.
template <bool FAST>
__global__ __launch_bounds__(kSdfBlock) void leaf_kernel(const double* __restrict__ q,
                                                         const double* __restrict__ nrm,
                                                         const double* __restrict__ w,
                                                         const int* __restrict__ order, int64_t n, int64_t nleaf,
                                                         GridDesc g, double* __restrict__ qs,
                                                         double* __restrict__ wn, TreeNode* __restrict__ node,
                                                         float* __restrict__ rec1, float* __restrict__ rec2) {
    const int64_t leaf = int64_t(blockIdx.x) * (kSdfBlock / 64) + (threadIdx.x >> 6);
    const int lane = int(threadIdx.x) & 63;
    if (leaf >= nleaf) return;
    const int64_t ix = leaf * kLeaf + lane;
    const bool own = ix < n;
    const int64_t s = order[own ? ix : leaf * kLeaf];  // lanes past the end repeat the first sample, weight 0
    double p[3], v[3], c[3];
    TreeNode t;
    bool finite = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        p[a] = q[3 * s + a];
        v[a] = own ? w[s] * nrm[3 * s + a] : 0.0;
        finite &= fabs(p[a]) < INFINITY;
        if (own) {
            qs[3 * ix + a] = p[a];
            wn[3 * ix + a] = v[a];
        }
    }
    const bool all = __ballot(!finite) == 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = wave_min(finite ? p[a] : INFINITY), hi = wave_max(finite ? p[a] : -INFINITY);
        const double mid = 0.5 * (lo + hi);
        const double o = a == 0 ? g.ox : (a == 1 ? g.oy : g.oz);
        c[a] = fabs(mid) < INFINITY ? lattice(mid, o, g.h) : 0.0;
        // a sample that is not finite never counts: the leaf is then always visited, and its infinite qmax2
        // has it tested pair by pair (below)
        t.lo[a] = all ? lo : -INFINITY;
        t.hi[a] = all ? hi : INFINITY;
        t.c[a] = c[a];
    }
    const float x = float(p[0] - c[0]), y = float(p[1] - c[1]), z = float(p[2] - c[2]);
    bool plain = all;
    if constexpr (FAST)
        plain &= __ballot(!put_record(rec1, rec2, ix, x, y, z, float(v[0]), float(v[1]), float(v[2]))) == 0;
    const double m2 = wave_max(finite ? double(x) * x + double(y) * y + double(z) * z : 0.0);
    if (lane == 0) {
        t.reach2 = -1.f;
        t.qmax2 = plain ? float(m2 * 1.0001) : INFINITY;
        t.px = 0;
        t.order = 0x111;
        node[leaf] = t;
    }
}

// 256-sample tile boxes (lo, hi) from the leaves
__global__ void tile_box_kernel(const TreeNode* __restrict__ node, int64_t nleaf, int64_t ntile,
                                double* __restrict__ box) {
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= ntile) return;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double lo = INFINITY, hi = -INFINITY;
        for (int64_t c = kFan * t; c < kFan * (t + 1) && c < nleaf; ++c) {
            lo = fmin(lo, node[c].lo[a]);
            hi = fmax(hi, node[c].hi[a]);
        }
        box[6 * t + a] = lo;
        box[6 * t + 3 + a] = hi;
    }
}

// Layout of the interpolation points: per level 1 and up, every node has room
// for cap points; `at` is the level's first record group, `part` its first
// partial sum, `blk` its first block of the weight kernel.
struct InterpLayout {
    int cap[kMaxLevels];
    int split[kMaxLevels];
    int64_t at[kMaxLevels];
    int64_t part[kMaxLevels];
    int64_t blk[kMaxLevels + 1];
};

// smallest order whose Chebyshev interpolation error rho^-p over half-width
// tau (in units of the distance to the nearest singularity) is below kInterpEps
__device__ int interp_order(double tau) {
    if (tau < 1e-7) return 1;
    const double d = 1.0 / tau;
    const double lr = log(d + sqrt(fmax(d * d - 1.0, 0.0)));
    if (!(lr > 0.0)) return 99;
    const int p = int(ceil(-log(kInterpEps) / lr));
    return p < 2 ? 2 : p;
}

// Nodes of one or more levels from their children (one block per launch runs
// the levels [l0, l1), or many blocks one level), 16 lanes a node.  With FAST,
// lane k tries tau = 0.6 0.87^k, and the node takes the largest (the smallest
// reach = half-width / tau) whose tensor grid stays within `share` of its
// samples.
constexpr int kTauTries = 14;
template <bool FAST>
__global__ __launch_bounds__(kSdfBlock) void tree_up_kernel(TreeNode* __restrict__ node, SampleTree tr, int l0,
                                                            int l1, int64_t n, GridDesc g, InterpLayout lay,
                                                            double share) {
    const int k = int(threadIdx.x) & 15, per = kSdfBlock / 16;
    for (int l = l0; l < l1; ++l) {
        if (l > l0) __syncthreads();  // one block: the level below is complete
        // every lane of a wave runs the same rounds: the choice of tau is a ballot
        for (int i0 = int(blockIdx.x) * per; i0 < tr.cnt[l]; i0 += int(gridDim.x) * per) {
            const int i = i0 + (int(threadIdx.x) >> 4);
            const bool own = i < tr.cnt[l];
            TreeNode t;
            double half[3], hmax = 0.0;
            t.qmax2 = 0.f;
            for (int c = kFan * i; c < kFan * (i + 1) && c < tr.cnt[l - 1]; ++c)
                if (node[tr.off[l - 1] + c].qmax2 == INFINITY) t.qmax2 = INFINITY;
            bool ok = own && t.qmax2 == 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double lo = INFINITY, hi = -INFINITY;
                for (int c = kFan * i; c < kFan * (i + 1) && c < tr.cnt[l - 1]; ++c) {
                    lo = fmin(lo, node[tr.off[l - 1] + c].lo[a]);
                    hi = fmax(hi, node[tr.off[l - 1] + c].hi[a]);
                }
                t.lo[a] = lo;
                t.hi[a] = hi;
                const double mid = 0.5 * (lo + hi);
                const double o = a == 0 ? g.ox : (a == 1 ? g.oy : g.oz);
                t.c[a] = fabs(mid) < INFINITY ? lattice(mid, o, g.h) : 0.0;
                half[a] = 0.5 * (hi - lo);
                ok &= half[a] * half[a] < double(kRecordMax) / 4.0;  // the points' records are plain too
                hmax = fmax(hmax, half[a]);
            }
            t.reach2 = -1.f;
            t.px = 0;
            t.order = 0x111;
            int pick = 0;
            if constexpr (FAST) {
                const int64_t size = int64_t(kLeaf) << (2 * l);
                const double have = double(n - size * i < size ? n - size * i : size);
                t.px = int(lay.at[l] + int64_t(i) * (lay.cap[l] / 16));
                double tau = 0.6;
                for (int e = 0; e < k; ++e) tau *= 0.87;
                const double reach = hmax / tau;
                int p[3], most = 1;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    p[a] = hmax > 0.0 ? interp_order(half[a] / reach) : 1;
                    most = p[a] > most ? p[a] : most;
                }
                const double m = double(p[0]) * p[1] * p[2];
                const bool fits = ok && k < kTauTries && most <= kInterpMax && m <= share * have;
                const int tries = int(__ballot(fits) >> (int(threadIdx.x) & 48)) & 0xffff;
                if (fits) {
                    t.reach2 = float(reach * reach * 1.0001);
                    t.order = p[0] | (p[1] << 4) | (p[2] << 8);
                }
                pick = tries ? __builtin_ctz(unsigned(tries)) : 0;
            }
            if (own && k == pick) node[tr.off[l] + i] = t;
        }
        if (l + 1 < l1) __threadfence_block();
    }
}

// Sums sum_j L_m(q_j) w_j n_j of 64 interpolation points of one node over up to
// kInterpSplit of its samples, FP64.  Lanes own points, the block's waves a
// quarter of the samples each; a wave tabulates the Lagrange factors of 16
// samples at a time in LDS.
__global__ __launch_bounds__(kSdfBlock) void interp_sum_kernel(const TreeNode* __restrict__ node, SampleTree tr,
                                                               InterpLayout lay, const double* __restrict__ qs,
                                                               const double* __restrict__ wn, int64_t n,
                                                               double* __restrict__ part, int64_t blk0) {
    __shared__ double tab[4][16][3][kInterpMax];
    __shared__ double sums[4][64][3];
    const int64_t blk = blk0 + blockIdx.x;
    int l = 1;
    while (l + 1 < tr.levels && blk >= lay.blk[l + 1]) ++l;
    const int chunks = (lay.cap[l] + 63) / 64;
    const int64_t b = blk - lay.blk[l];
    const int chunk = int(b % chunks), split = int((b / chunks) % lay.split[l]);
    const int i = int(b / (int64_t(chunks) * lay.split[l]));
    const TreeNode t = node[tr.off[l] + i];
    const int count = t.reach2 < 0.f ? 0 : order_count(t.order);
    if (64 * chunk >= count) return;  // uniform across the block
    const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
    const int p0 = t.order & 15, p1 = (t.order >> 4) & 15, p2 = (t.order >> 8) & 15;
    const int m = 64 * chunk + lane;
    const bool own = m < count;
    const int m0 = own ? m % p0 : 0, m1 = own ? (m / p0) % p1 : 0, m2 = own ? m / (p0 * p1) : 0;
    const int64_t size = int64_t(kLeaf) << (2 * l);
    const int64_t first = size * i + int64_t(split) * kInterpSplit;
    int64_t last = size * i + size < n ? size * i + size : n;
    if (last > first + kInterpSplit) last = first + kInterpSplit;
    // this lane's role in the tables: axis la of sample lane % 16
    const int la = lane >> 4;
    const int pl = la == 0 ? p0 : (la == 1 ? p1 : p2);
    const double lo = la == 0 ? t.lo[0] : (la == 1 ? t.lo[1] : t.lo[2]);
    const double hi = la == 0 ? t.hi[0] : (la == 1 ? t.hi[1] : t.hi[2]);
    const double mid = 0.5 * (lo + hi), inv = hi > lo ? 2.0 / (hi - lo) : 0.0;
    double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
    for (int64_t s0 = first + 16 * wave; s0 < first + kInterpSplit; s0 += 64) {
        __syncthreads();
        if (la < 3 && s0 + (lane & 15) < last) {
            const double x = (qs[3 * (s0 + (lane & 15)) + la] - mid) * inv;
            double* L = tab[wave][lane & 15][la];
            // L_m(x) = w_m prod_{k != m} (x - x_k), x_k = cos((2k + 1) pi / 2p),
            // w_m = (-1)^m 2^(p - 1) sin((2m + 1) pi / 2p) / p
            const double sc = exp2(double(pl - 1)) / pl;
            double run = 1.0;
            for (int k = 0; k < pl; ++k) {
                L[k] = run;
                run *= x - cospi((2 * k + 1) / (2.0 * pl));
            }
            run = sc;
            for (int k = pl - 1; k >= 0; --k) {
                const double a = (2 * k + 1) / (2.0 * pl);
                L[k] *= run * ((k & 1) ? -sinpi(a) : sinpi(a));
                run *= x - cospi(a);
            }
        }
        __syncthreads();
        const int cnt = int(last - s0 < 16 ? last - s0 : 16);
        for (int a = 0; a < cnt; ++a) {
            const double f = tab[wave][a][0][m0] * tab[wave][a][1][m1] * tab[wave][a][2][m2];
            const int64_t s = s0 + a;
            acc0 += f * wn[3 * s];
            acc1 += f * wn[3 * s + 1];
            acc2 += f * wn[3 * s + 2];
        }
    }
    sums[wave][lane][0] = acc0;
    sums[wave][lane][1] = acc1;
    sums[wave][lane][2] = acc2;
    __syncthreads();
    if (wave == 0 && own) {
        double* o = part + (lay.part[l] + (int64_t(i) * lay.split[l] + split) * lay.cap[l] + m) * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) o[a] = (sums[0][lane][a] + sums[1][lane][a]) + (sums[2][lane][a] + sums[3][lane][a]);
    }
}

// Records of the interpolation points of level 1 + blockIdx.y: position, and
// the splits' sums; points past the count repeat the first with weight 0.
__global__ __launch_bounds__(kSdfBlock) void interp_record_kernel(const TreeNode* __restrict__ node, SampleTree tr,
                                                                  InterpLayout lay,
                                                                  const double* __restrict__ part,
                                                                  float* __restrict__ rec1,
                                                                  float* __restrict__ rec2) {
    const int l = 1 + int(blockIdx.y);
    const int64_t id = int64_t(blockIdx.x) * kSdfBlock + threadIdx.x;
    const int i = int(id / lay.cap[l]), m = int(id % lay.cap[l]);
    if (i >= tr.cnt[l]) return;
    const TreeNode t = node[tr.off[l] + i];
    const int count = t.reach2 < 0.f ? 0 : order_count(t.order);
    if (m >= (count + 15) / 16 * 16) return;
    const int mm = m < count ? m : 0;
    const int p[3] = {t.order & 15, (t.order >> 4) & 15, (t.order >> 8) & 15};
    const int at[3] = {mm % p[0], (mm / p[0]) % p[1], mm / (p[0] * p[1])};
    float x[3], w[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double node_x = 0.5 * (t.lo[a] + t.hi[a]) +
                              (p[a] > 1 ? 0.5 * (t.hi[a] - t.lo[a]) * cospi((2 * at[a] + 1) / (2.0 * p[a])) : 0.0);
        x[a] = float(node_x - t.c[a]);
        double v = 0.0;
        if (m < count)
            for (int sp = 0; sp < lay.split[l]; ++sp)
                v += part[(lay.part[l] + (int64_t(i) * lay.split[l] + sp) * lay.cap[l] + m) * 3 + a];
        w[a] = float(v);
    }
    put_record(rec1, rec2, int64_t(t.px) * 16 + m, x[0], x[1], x[2], w[0], w[1], w[2]);
}

SampleTree tree_layout(int64_t n, int64_t* nodes) {
    SampleTree tr{};
    int64_t c = (n + kLeaf - 1) / kLeaf, off = 0;
    for (;;) {
        tr.off[tr.levels] = int(off);
        tr.cnt[tr.levels] = int(c);
        ++tr.levels;
        off += c;
        if (c <= kFan) break;
        c = (c + kFan - 1) / kFan;
    }
    *nodes = off;
    return tr;
}

// Workspace carve-up (256-byte aligned pieces).  The sort's buffers are free
// once the samples are gathered: the tree and the tile boxes reuse them.  The
// second part, for the FP32 kernels' fast pass 2, is optional.
struct SdfWs {
    size_t keys_in, vals_in, qs, wn, keys_out, vals_out, temp, tree, box, total;
    size_t rec1, rec2, part, fast_total;
    InterpLayout lay;
};
inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }
inline SdfWs sdf_ws_layout(int64_t n) {
    SdfWs L{};
    const int64_t ntile = (n + kSdfTile - 1) / kSdfTile;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += al256(bytes);
        return at;
    };
    L.vals_in = take(size_t(n) * 4);
    L.qs = take(size_t(n) * 24);
    L.wn = take(size_t(n) * 24);
    const size_t reuse = off;
    L.keys_in = take(size_t(n) * 4);
    L.keys_out = take(size_t(n) * 4);
    L.vals_out = take(size_t(n) * 4);
    L.temp = take(sort_temp_bytes(n));
    const size_t sort_end = off;
    off = reuse;
    int64_t nodes = 0;
    const SampleTree tr = tree_layout(n, &nodes);
    L.tree = take(size_t(nodes) * sizeof(TreeNode));
    L.box = take(size_t(ntile) * 48);
    off = std::max(off, sort_end);
    L.total = off;
    int64_t groups = int64_t(tr.cnt[0]) * (kLeaf / 16), parts = 0, blocks = 0;
    for (int l = 1; l < tr.levels; ++l) {
        const int64_t size = int64_t(kLeaf) << (2 * l);
        L.lay.cap[l] = interp_cap(size);
        L.lay.split[l] = int((size + kInterpSplit - 1) / kInterpSplit);
        L.lay.at[l] = groups;
        L.lay.part[l] = parts;
        L.lay.blk[l] = blocks;
        groups += int64_t(tr.cnt[l]) * (L.lay.cap[l] / 16);
        parts += int64_t(tr.cnt[l]) * L.lay.split[l] * L.lay.cap[l];
        blocks += int64_t(tr.cnt[l]) * L.lay.split[l] * ((L.lay.cap[l] + 63) / 64);
    }
    L.lay.blk[tr.levels] = blocks;
    L.rec1 = take(size_t(groups) * 256);
    L.rec2 = take(size_t(groups) * 256);
    L.part = take(size_t(parts) * 24);
    L.fast_total = off;
    return L;
}

struct Prepared {
    SampleTiles st;       // sorted samples, and 256-sample tiles (radial kernel)
    SampleTree tr;
    const TreeNode* node;
    const float *rec1, *rec2;
};

// a launch has fewer than 2^32 threads along x: more go into several
constexpr int64_t kLaunchThreads = int64_t(1) << 31;

// Hilbert order, sorted copies, sample tree; with `fast` the records of the FP32
// sum, with `interp` its interpolation points, with `tiles` the 256-sample tile boxes
hipError_t prepare_samples(const double* q, const double* n, const double* w, int64_t ns, const GridDesc& g, void* ws,
                           bool fast, bool interp, bool tiles, hipStream_t s, Prepared* out) {
    const SdfWs L = sdf_ws_layout(ns);
    char* base = static_cast<char*>(ws);
    auto* qs = reinterpret_cast<double*>(base + L.qs);
    auto* wn = reinterpret_cast<double*>(base + L.wn);
    auto* node = reinterpret_cast<TreeNode*>(base + L.tree);
    auto* box = reinterpret_cast<double*>(base + L.box);
    auto* rec1 = reinterpret_cast<float*>(base + L.rec1);
    auto* rec2 = reinterpret_cast<float*>(base + L.rec2);
    auto* part = reinterpret_cast<double*>(base + L.part);
    auto* vals_in = reinterpret_cast<int*>(base + L.vals_in);
    const double ext = g.h * (std::max(g.nx, std::max(g.ny, g.nz)) + 8);
    const double ox = g.ox - 4 * g.h, oy = g.oy - 4 * g.h, oz = g.oz - 4 * g.h, inv_cell = 1024.0 / ext;
    int* order = vals_in;
    if (ns <= kSmallSort) {
        hipLaunchKernelGGL(small_order_kernel, dim3(unsigned((ns + 63) / 64)), dim3(1024), 0, s, q, int(ns), ox, oy, oz,
                           inv_cell, order);
    } else {
        auto* keys_in = reinterpret_cast<unsigned*>(base + L.keys_in);
        auto* keys_out = reinterpret_cast<unsigned*>(base + L.keys_out);
        auto* vals_out = reinterpret_cast<int*>(base + L.vals_out);
        hipLaunchKernelGGL(hilbert_key_kernel, dim3(unsigned((ns + 255) / 256)), dim3(256), 0, s, q, ns, ox, oy, oz,
                           inv_cell, keys_in, vals_in);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        unsigned* keys_sorted = nullptr;
        // four passes of 8 bits: the result is back in the first pair of buffers
        e = launch_sort_pairs(keys_in, vals_in, keys_out, vals_out, ns, 30, base + L.temp, s, &keys_sorted, &order);
        if (e != hipSuccess) return e;
        if (order != vals_in) return hipErrorUnknown;
    }
    int64_t nodes = 0;
    const SampleTree tr = tree_layout(ns, &nodes);
    const int64_t nleaf = tr.cnt[0], ntile = (ns + kSdfTile - 1) / kSdfTile;
    const dim3 lg(unsigned((nleaf + 3) / 4));
    if (fast)
        hipLaunchKernelGGL(leaf_kernel<true>, lg, dim3(kSdfBlock), 0, s, q, n, w, order, ns, nleaf, g, qs, wn, node,
                           rec1, rec2);
    else
        hipLaunchKernelGGL(leaf_kernel<false>, lg, dim3(kSdfBlock), 0, s, q, n, w, order, ns, nleaf, g, qs, wn, node,
                           nullptr, nullptr);
    // levels of many nodes by a launch each, the rest by one block
    int l = 1;
    while (l < tr.levels) {
        const bool many = tr.cnt[l] > 64;
        const int l1 = many ? l + 1 : tr.levels;
        const dim3 ug(many ? unsigned((tr.cnt[l] + kSdfBlock / 16 - 1) / (kSdfBlock / 16)) : 1u);
        if (fast)
            hipLaunchKernelGGL(tree_up_kernel<true>, ug, dim3(kSdfBlock), 0, s, node, tr, l, l1, ns, g, L.lay,
                               interp ? kInterpShare : 0.0);
        else
            hipLaunchKernelGGL(tree_up_kernel<false>, ug, dim3(kSdfBlock), 0, s, node, tr, l, l1, ns, g, L.lay, 0.0);
        l = l1;
    }
    if (fast && interp && tr.levels > 1) {
        for (int64_t b0 = 0; b0 < L.lay.blk[tr.levels]; b0 += kLaunchThreads / kSdfBlock) {
            const int64_t count = std::min(L.lay.blk[tr.levels] - b0, kLaunchThreads / kSdfBlock);
            hipLaunchKernelGGL(interp_sum_kernel, dim3(unsigned(count)), dim3(kSdfBlock), 0, s, node, tr, L.lay, qs, wn,
                               ns, part, b0);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        int64_t pts = 0;
        for (int lv = 1; lv < tr.levels; ++lv) pts = std::max(pts, int64_t(tr.cnt[lv]) * L.lay.cap[lv]);
        const dim3 rg{unsigned((pts + kSdfBlock - 1) / kSdfBlock), unsigned(tr.levels - 1), 1u};
        hipLaunchKernelGGL(interp_record_kernel, rg, dim3(kSdfBlock), 0, s, node, tr, L.lay, part, rec1, rec2);
    }
    if (tiles)
        hipLaunchKernelGGL(tile_box_kernel, dim3(unsigned((ntile + 63) / 64)), dim3(64), 0, s, node, nleaf, ntile,
                           box);
    *out = Prepared{SampleTiles{qs, wn, order, box, ntile}, tr, node, rec1, rec2};
    return hipGetLastError();
}

// node-sample pairs from which interpolation repays its own launches
constexpr double kInterpPairs = 1e8;
// Grids of at most this many bricks give each brick's samples to four waves,
// where one wave per brick would leave the 1024 SIMDs too few waves to hide a
// walk's loads.  The fast kernel keeps a SIMD busy with two waves and pays the
// shared walk: 4 waves / 1 wave take 130 / 150 us at 2048 bricks (32^3, 0.9k
// samples), 211 / 192 us at 4000, 1196 / 773 us at 16384 (64^3, 3.9k).  The
// FP64 one, bound by the latency of its serial pair loop, crosses later:
// 386 / 420 us at 4000, 2350 / 2630 us at 16384, 4030 / 3960 us at 23328.
template <bool FAST>
constexpr int64_t kShareBricks = FAST ? 2500 : 20000;

int64_t brick_count(const GridDesc& g) {
    const Brick br = brick_shape(g.nz);
    return int64_t((g.nx + br.bx - 1) / br.bx) * ((g.ny + br.by - 1) / br.by) * ((g.nz + br.bz - 1) / br.bz);
}

// zeroed by a kernel, not hipMemsetAsync, so the call can be captured in a graph
__global__ void zero_grads_kernel(double* __restrict__ gq, double* __restrict__ gn, double* __restrict__ gw,
                                  int64_t ns) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < 3 * ns; i += int64_t(gridDim.x) * blockDim.x) {
        gq[i] = 0.0;
        gn[i] = 0.0;
        if (i < ns) gw[i] = 0.0;
    }
}

template <typename T, int PHI>
void enqueue_few(const double* q, const double* n, const double* w, int64_t ns, const GridDesc& g, const ParamDesc& p,
                 cplx<T>* out, hipStream_t s) {
    const int64_t bricks = brick_count(g);
    for (int64_t b0 = 0; b0 < bricks; b0 += kLaunchThreads / kSdfBlock) {
        const int64_t count = std::min(bricks - b0, kLaunchThreads / kSdfBlock);
        hipLaunchKernelGGL((sdf_few_kernel<T, PHI>), dim3(unsigned(count)), dim3(kSdfBlock), 0, s, q, n, w, int(ns), g, p,
                           out, b0);
    }
}
// Up to how many samples that is the faster way.  On small grids it is a serial
// chain of 0.25 us a sample: 64 samples on 32^3 nodes 20.6 us (the tree 33.5), 200
// 57 (45), on 8^3 64 19 (20), FP64 24 (18).  On large ones the tree's walk costs a wave of 16 nodes as much as some
// hundred pairs of each: on 128^3 nodes 1 sample takes 19 us (the tree 169), 64 142
// (393), 300 610 (900), 500 1006 (1079); FP64 64 340 (483), 300 1536 (1543), 400
// 2040 (1916); on 64^3 300 116 (150), 500 190 (190).  The signed distance alone
// (double skin layer): 500 on 8^3 32 (32), on 128^3 315 (440).
bool few_samples(int64_t ns, const GridDesc& g, int phi, bool wide) {
    const int64_t nodes = int64_t(g.nx) * g.ny * g.nz;
    if (brick_count(g) * kSdfBlock > 2 * nodes) return ns <= 64 && nodes <= 4096;  // thin grids fill few lanes
    if (phi == kPhiDsl) return ns <= 512;
    if (nodes < (1 << 18)) return ns <= (wide ? 32 : 64);
    return ns <= (wide || nodes < (1 << 20) ? 300 : kFewMax);
}

template <typename T, int PHI, bool FAST, bool STATS = false>
void enqueue_build(const double* q, const double* n, const Prepared& P, int64_t ns, const GridDesc& g,
                   const ParamDesc& p, cplx<T>* out, unsigned long long* stats, hipStream_t s) {
    const BrickGrid bg = wave_bricks(g.nx, g.ny, g.nz);
    const int64_t bricks = int64_t(bg.nx) * bg.ny * bg.nz;
    auto run = [&](auto kernel, int waves) {
        for (int64_t b0 = 0; b0 < bricks; b0 += kLaunchThreads / (64 * waves)) {
            const int64_t count = std::min<int64_t>(bricks - b0, kLaunchThreads / (64 * waves));
            hipLaunchKernelGGL(kernel, dim3(unsigned(count)), dim3(64 * waves), 0, s, q, n, P.st.qs, P.st.wn, P.st.js,
                               P.node, P.tr, P.rec1, P.rec2, ns, g, p, out, stats, b0);
        }
    };
    if (bricks <= kShareBricks<FAST>) run(sdf_build_kernel<T, PHI, FAST, 4, STATS>, 4);
    else run(sdf_build_kernel<T, PHI, FAST, 1, STATS>, 1);
}

}  // namespace

size_t sdf_build_workspace_bytes(int64_t ns, int phi) {
    // the radial kernel tiles the 2 n offset points, held (positions, weight
    // slots, weights) ahead of the tile layout
    if (phi == kPhiRadial) return al256(size_t(ns) * 2 * 7 * sizeof(double)) + sdf_ws_layout(2 * ns).total;
    return sdf_ws_layout(ns).total;
}

size_t sdf_build_fast_bytes(int64_t ns) { return sdf_ws_layout(ns).fast_total; }

namespace {

// Leaf ranges per brick of the adjoint: about kAdjointBlocks blocks in all, at
// least a leaf for each wave.  Larger grids have bricks enough to even out.
constexpr int64_t kAdjointBlocks = 8192;
// Groups of 16 nodes up to which four waves look for their nearest samples, as
// the build's bricks (shape gradients: 630 / 670 us at 2048 groups, 1445 / 1455
// at 6912, 1875 / 1855 at 15360, 2830 / 2805 at 16384).
constexpr int64_t kShareNearest = 10000;
struct AdjointSplit {
    int64_t bricks, splits;
};
AdjointSplit adjoint_split(int64_t ns, const GridDesc& g) {
    const int64_t bricks = brick_count(g), leaves = (ns + kLeaf - 1) / kLeaf;
    return {bricks, std::max<int64_t>(1, std::min<int64_t>(kAdjointBlocks / bricks, (leaves + 3) / 4))};
}

}  // namespace

size_t sdf_adjoint_bytes(int64_t ns, const GridDesc& g) {
    const AdjointSplit sp = adjoint_split(ns, g);
    return sdf_ws_layout(ns).total + (sp.splits > 1 ? size_t(sp.bricks) * kSdfBlock * 20 : 0);
}

template <typename T>
hipError_t launch_sdf_build(const double* q, const double* n, const double* w, int64_t ns, const GridDesc& g,
                            const ParamDesc& p, int phi, void* rho_out, void* ws, size_t ws_bytes, hipStream_t s,
                            unsigned long long* stats) {
    Prepared P{};
    auto* out = static_cast<cplx<T>*>(rho_out);
    if (phi == kPhiRadial) {
        double* q2 = static_cast<double*>(ws);
        double* c2 = q2 + 6 * ns;
        double* w2 = c2 + 6 * ns;
        hipLaunchKernelGGL(offset_points_kernel, dim3(unsigned((ns + 255) / 256)), dim3(256), 0, s, q, n, w, ns,
                           p.radius, p.lambda1, p.lambda2, q2, c2, w2);
        void* ws2 = static_cast<char*>(ws) + al256(size_t(ns) * 2 * 7 * sizeof(double));
        hipError_t e = prepare_samples(q2, c2, w2, 2 * ns, g, ws2, false, false, true, s, &P);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(sdf_radial_kernel<T>, dim3(unsigned(brick_count(g))), dim3(kSdfBlock), 0, s, P.st, 2 * ns,
                           g, p, out);
        return hipGetLastError();
    }
    if (!stats && few_samples(ns, g, phi, std::is_same<T, double>::value)) {
        if (phi == kPhiDsl) enqueue_few<T, kPhiDsl>(q, n, w, ns, g, p, out, s);
        else if (phi == kPhiInverseSquare) enqueue_few<T, kPhiInverseSquare>(q, n, w, ns, g, p, out, s);
        else enqueue_few<T, kPhiSkeletal>(q, n, w, ns, g, p, out, s);
        return hipGetLastError();
    }
    const bool sums = phi == kPhiSkeletal || phi == kPhiInverseSquare;
    const bool fast = std::is_same<T, float>::value && sums && ws_bytes >= sdf_build_fast_bytes(ns);
    const bool interp = fast && double(ns) * g.nx * g.ny * g.nz >= kInterpPairs;
    hipError_t e = prepare_samples(q, n, w, ns, g, ws, fast, interp, false, s, &P);
    if (e != hipSuccess) return e;
    if constexpr (std::is_same<T, float>::value) {
        if (fast) {
            if (stats) enqueue_build<T, kPhiSkeletal, true, true>(q, n, P, ns, g, p, out, stats, s);
            else if (phi == kPhiSkeletal) enqueue_build<T, kPhiSkeletal, true>(q, n, P, ns, g, p, out, nullptr, s);
            else enqueue_build<T, kPhiInverseSquare, true>(q, n, P, ns, g, p, out, nullptr, s);
            return hipGetLastError();
        }
    }
    if (stats) enqueue_build<T, kPhiSkeletal, false, true>(q, n, P, ns, g, p, out, stats, s);
    else if (phi == kPhiDsl) enqueue_build<T, kPhiDsl, false>(q, n, P, ns, g, p, out, nullptr, s);
    else if (phi == kPhiInverseSquare) enqueue_build<T, kPhiInverseSquare, false>(q, n, P, ns, g, p, out, nullptr, s);
    else enqueue_build<T, kPhiSkeletal, false>(q, n, P, ns, g, p, out, nullptr, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_sdf_adjoint(const double* q, const double* n, const double* w, int64_t ns, const GridDesc& g,
                              const ParamDesc& p, const void* cot, double* grad_q, double* grad_n, double* grad_w,
                              void* ws, size_t ws_bytes, hipStream_t s) {
    hipLaunchKernelGGL(zero_grads_kernel, dim3(unsigned(std::min<int64_t>((3 * ns + 255) / 256, 4096))), dim3(256), 0, s,
                       grad_q, grad_n, grad_w, ns);
    Prepared P{};
    hipError_t e = prepare_samples(q, n, w, ns, g, ws, false, false, false, s, &P);
    if (e != hipSuccess) return e;
    const AdjointSplit sp = adjoint_split(ns, g);
    const int64_t turn = tile_step(sp.bricks);
    auto run = [&](auto kernel, int64_t splits, const NearData& near) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(sp.bricks), unsigned(splits)), dim3(kSdfBlock), 0, s, q, n, w,
                           P.st.qs, P.st.js, P.node, P.tr, ns, g, p, static_cast<const cplx<T>*>(cot), grad_q, grad_n,
                           grad_w, turn, near);
    };
    const int64_t slots = sp.bricks * kSdfBlock;
    if (sp.splits > 1 && ws_bytes >= sdf_adjoint_bytes(ns, g)) {
        auto* d2 = reinterpret_cast<double*>(static_cast<char*>(ws) + sdf_ws_layout(ns).total);
        const NearData near{d2, d2 + slots, reinterpret_cast<int*>(d2 + 2 * slots)};
        auto nearest = [&](auto kernel, int waves) {
            hipLaunchKernelGGL(kernel, dim3(unsigned(16 * sp.bricks)), dim3(64 * waves), 0, s, P.st.qs, P.st.js, P.node,
                               P.tr, ns, g, tile_step(16 * sp.bricks), near);
        };
        if (16 * sp.bricks <= kShareNearest) nearest(adjoint_nearest_kernel<4>, 4);
        else nearest(adjoint_nearest_kernel<1>, 1);
        run(sdf_adjoint_kernel<T, true>, sp.splits, near);
        hipLaunchKernelGGL(adjoint_xi_kernel, dim3(unsigned(sp.bricks)), dim3(kSdfBlock), 0, s, q, P.st.js, g, near,
                           grad_q);
    } else {
        run(sdf_adjoint_kernel<T, false>, 1, NearData{});
    }
    return hipGetLastError();
}

template hipError_t launch_sdf_adjoint<float>(const double*, const double*, const double*, int64_t, const GridDesc&,
                                              const ParamDesc&, const void*, double*, double*, double*, void*,
                                              size_t, hipStream_t);
template hipError_t launch_sdf_adjoint<double>(const double*, const double*, const double*, int64_t,
                                               const GridDesc&, const ParamDesc&, const void*, double*, double*,
                                               double*, void*, size_t, hipStream_t);
template hipError_t launch_sdf_build<float>(const double*, const double*, const double*, int64_t, const GridDesc&,
                                            const ParamDesc&, int, void*, void*, size_t, hipStream_t,
                                            unsigned long long*);
template hipError_t launch_sdf_build<double>(const double*, const double*, const double*, int64_t, const GridDesc&,
                                             const ParamDesc&, int, void*, void*, size_t, hipStream_t,
                                             unsigned long long*);

}  // namespace sdf
