// Pose value and adjoint for gradient-based refinement of placements.
//
//   f(t, q) = Re sum_k c_k Phi(R x_k / h + t),  Phi(y) = sum_p rho_F(p) B3(p - y),
//   df/dt   = Re sum_k c_k grad Phi(y_k)                      (g_k = Re c_k grad Phi(y_k)),
//   df/dq   from the torque tau = sum_k (R x_k / h) x g_k:    for a unit quaternion u the
//             rotated point moves by 2 vec(e_c u*) x (R x) + (radial part) along u_c,
//             so df/du_c = 2 vec(e_c u*) . tau on the tangent space of |u| = 1,
//   df/dw_k = sum_b s_b Re(rho_M(x_k) Phi_b(y_k)).
//
// Block (sample tile, pose tile): threads own body samples and walk the poses
// of the tile, gathering the 4^3 stencil of rho_F around each moved sample
// (the stencil weights are recomputed here, never stored).  Per pose the 7
// sums (f, df/dt, tau) are accumulated in FP64 and reduced per block into
// partials; a second kernel reduces the partials per pose and applies the
// quaternion chain rule in FP64.  Per-sample weight gradients stay in
// registers across the pose tile and are written once per tile.
#include <algorithm>
#include <limits>
#include <type_traits>

#include "block_order.hpp"
#include "common.hpp"
#include "launch.hpp"
#include "tile_spread.hpp"

namespace sdf {

namespace {

constexpr int kGBlock = 256;
constexpr int kSPT = 4;           // samples per thread of the tile kernel (1 where blocks are few)
constexpr int kPosesPerBlock = 16;  // at most, in both pose kernels
constexpr int kNAcc = 7;  // f, dt[3], tau[3]

__device__ __forceinline__ void quat_rot(const double* q, double r[9]) {
    double w = q[0], x = q[1], y = q[2], z = q[3];
    const double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
    w *= inv;
    x *= inv;
    y *= inv;
    z *= inv;
    r[0] = 1 - 2 * (y * y + z * z);
    r[1] = 2 * (x * y - w * z);
    r[2] = 2 * (x * z + w * y);
    r[3] = 2 * (x * y + w * z);
    r[4] = 1 - 2 * (x * x + z * z);
    r[5] = 2 * (y * z - w * x);
    r[6] = 2 * (x * z - w * y);
    r[7] = 2 * (y * z + w * x);
    r[8] = 1 - 2 * (x * x + y * y);
}

// Sum of v over each row of 16 lanes, left in every lane of the row (DPP
// quad permutations and row rotations; no LDS traffic).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row16_sum(double v) {
    v += dpp_f64<0xb1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_f64<0x4e>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_f64<0x124>(v);  // row_ror 4
    v += dpp_f64<0x128>(v);  // row_ror 8
    return v;
}

// The sums of v[0 .. 6] over each row of 16 lanes: lane l of a row ends with
// those of values a and a + 1, a = 4 (l & 1) + (l & 2).  Two exchanges halve
// the values a lane carries, so 54 instructions do the work of 84.
__device__ __forceinline__ void row16_sum8(const double v[7], int lane, double out[2]) {
    const bool b0 = lane & 1, b1 = lane & 2;
    double h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double hi = i < 3 ? v[i + 4] : 0.0;
        h[i] = (b0 ? hi : v[i]) + dpp_f64<0xb1>(b0 ? v[i] : hi);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        double x = (b1 ? h[i + 2] : h[i]) + dpp_f64<0x4e>(b1 ? h[i] : h[i + 2]);
        x += dpp_f64<0x124>(x);  // the four quads of the row
        x += dpp_f64<0x128>(x);
        out[i] = x;
    }
}
__device__ __forceinline__ double warp_sum(double v) {
    for (int off = warpSize / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Bound by the latency of its gathers where a call is small: a block of 1024
// samples walked 16 poses one after the other, and 25 poses of 4096 planar
// FP64 samples ran 8 blocks on 256 CUs.  SPT samples a thread and `per` poses
// a block come from grad_split; that call: 163 -> 8 us with gradients.
template <typename T, bool GRAD, int SPT>
__global__ __launch_bounds__(kGBlock) void grad_tile_kernel(const cplx<T>* __restrict__ rho_f, int N, int planar,
                                                            const cplx<T>* __restrict__ rho_m,
                                                            const T* __restrict__ w_m, int n_m,
                                                            const double* __restrict__ poses, int64_t B,
                                                            const double* __restrict__ gscale,
                                                            double* __restrict__ part, int nsb,
                                                            T* __restrict__ wpart, int want_w, int pb0, int per) {
    const int sb = blockIdx.x, pb = pb0 + int(blockIdx.y);
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const int nz = planar ? 1 : N;
    const T half = T(0.5) * T(n_m);

    // this thread's samples
    int64_t ks[SPT];
    T xb[SPT][3];
    cplx<T> ck[SPT], rm[SPT];
    T gw[SPT], gwi[SPT];  // wmode 1: Re(rho_M Phi) sums; 2: Phi sums (re, im)
#pragma unroll
    for (int s = 0; s < SPT; ++s) {
        const int64_t k = (int64_t(sb) * SPT + s) * kGBlock + threadIdx.x;
        ks[s] = k;
        const int64_t kk = k < K ? k : 0;
        xb[s][0] = T(int(kk % n_m)) - half;
        xb[s][1] = T(int((kk / n_m) % n_m)) - half;
        xb[s][2] = planar ? T(0) : T(int(kk / (int64_t(n_m) * n_m))) - half;
        rm[s] = k < K ? rho_m[kk] : mk(T(0), T(0));
        ck[s] = rm[s] * (k < K ? w_m[kk] : T(0));
        gw[s] = T(0);
        gwi[s] = T(0);
    }

    __shared__ double red[kGBlock / 16][kNAcc];

    const int64_t b0 = int64_t(pb) * per;
    for (int pi = 0; pi < per; ++pi) {
        const int64_t b = b0 + pi;
        if (b >= B) break;  // uniform across the block
        const double* pose = poses + 7 * b;
        double r64[9];
        quat_rot(pose + 3, r64);
        T r[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) r[a] = T(r64[a]);
        // split t into an integer and a fractional part so that positions are
        // formed in the sample's local frame (keeps FP32 stencils accurate)
        double tint[3];
        T tfr[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            tint[a] = floor(pose[a]);
            tfr[a] = T(pose[a] - tint[a]);
        }
        const double sc = gscale ? gscale[b] : 1.0;
        double acc[kNAcc];
#pragma unroll
        for (int a = 0; a < kNAcc; ++a) acc[a] = 0.0;

#pragma unroll
        for (int s = 0; s < SPT; ++s) {
            if (ks[s] >= K) continue;
            T y[3];
#pragma unroll
            for (int a = 0; a < 3; ++a)
                y[a] = tfr[a] + r[3 * a] * xb[s][0] + r[3 * a + 1] * xb[s][1] + r[3 * a + 2] * xb[s][2];
            T fl[3], wgt[3][4], dw[3][4];
            int base[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                fl[a] = dev_floor(y[a]);
                base[a] = int(fl[a]) + int(tint[a]) - 1;
                bspline3_weights(y[a] - fl[a], wgt[a]);
                if (GRAD) bspline3_dweights(y[a] - fl[a], dw[a]);
            }
            cplx<T> phi = mk(T(0), T(0)), gx = phi, gy = phi, gz = phi;
            const int zc = planar ? 1 : 4;
            for (int cz = 0; cz < zc; ++cz) {
                const int iz = planar ? 0 : wrap(base[2] + cz, nz);
                const T wz = planar ? T(1) : wgt[2][cz];
                const T dz = planar ? T(0) : (GRAD ? dw[2][cz] : T(0));
#pragma unroll
                for (int cy = 0; cy < 4; ++cy) {
                    const int iy = wrap(base[1] + cy, N);
                    const cplx<T>* row = rho_f + (int64_t(iz) * N + iy) * N;
                    cplx<T> rx = mk(T(0), T(0)), rdx = rx;
#pragma unroll
                    for (int cx = 0; cx < 4; ++cx) {
                        const cplx<T> v = row[wrap(base[0] + cx, N)];
                        rx = rx + v * wgt[0][cx];
                        if (GRAD) rdx = rdx + v * dw[0][cx];
                    }
                    phi = phi + rx * (wgt[1][cy] * wz);
                    if (GRAD) {
                        gx = gx + rdx * (wgt[1][cy] * wz);
                        gy = gy + rx * (dw[1][cy] * wz);
                        gz = gz + rx * (wgt[1][cy] * dz);
                    }
                }
            }
            const cplx<T> v = ck[s] * phi;
            acc[0] += double(v.re);
            if (GRAD) {
                const double g0 = double((ck[s] * gx).re), g1 = double((ck[s] * gy).re),
                             g2 = double((ck[s] * gz).re);
                acc[1] += g0;
                acc[2] += g1;
                acc[3] += g2;
                // rotated body position R x (without t) and torque (R x) x g
                double wv[3];
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    wv[a] = double(r[3 * a]) * double(xb[s][0]) + double(r[3 * a + 1]) * double(xb[s][1]) +
                            double(r[3 * a + 2]) * double(xb[s][2]);
                acc[4] += wv[1] * g2 - wv[2] * g1;
                acc[5] += wv[2] * g0 - wv[0] * g2;
                acc[6] += wv[0] * g1 - wv[1] * g0;
                if (want_w == 1) gw[s] += T(sc) * (rm[s] * phi).re;
                if (want_w == 2) {
                    gw[s] += T(sc) * phi.re;
                    gwi[s] += T(sc) * phi.im;
                }
            }
        }
        // block reduction of the per-pose sums (FP64): rows of 16 lanes, then the rows;
        // a single sum over the wave (FP64, 4096 poses of 32^3: values alone 12.4 ms, with
        // the rows, where the compiler gathers with other registers, 14.3)
        constexpr int nacc = GRAD ? kNAcc : 1;
#pragma unroll
        for (int a = 0; a < nacc; ++a) {
            if constexpr (GRAD) {
                const double v = row16_sum(acc[a]);
                if ((threadIdx.x & 15) == 0) red[threadIdx.x >> 4][a] = v;
            } else {
                const double v = warp_sum(acc[a]);
                if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][a] = v;
            }
        }
        __syncthreads();
        if (threadIdx.x < nacc) {
            double v = 0.0;
#pragma unroll
            for (int rw = 0; rw < kGBlock / (GRAD ? 16 : 64); ++rw) v += red[rw][threadIdx.x];
            part[(b * nsb + sb) * kNAcc + threadIdx.x] = v;
        }
        __syncthreads();
    }
    if (GRAD && want_w) {
#pragma unroll
        for (int s = 0; s < SPT; ++s)
            if (ks[s] < K) {
                if (want_w == 1) wpart[int64_t(pb) * K + ks[s]] = gw[s];
                else {
                    wpart[2 * (int64_t(pb) * K + ks[s])] = gw[s];
                    wpart[2 * (int64_t(pb) * K + ks[s]) + 1] = gwi[s];
                }
            }
    }
}

// 3D FP32 variant with the fixed field staged in LDS.  Block (8 x 8 x 8
// sample tile, pose tile), one sample per thread.  Per pose the block loads
// into LDS the box of rho_F cells that the tile's 4^3 stencils can touch:
// the tile's corners bound its moved positions (widened by 1e-3 cell, far
// above the FP32 rounding of a moved position), so the stencil floors span at
// most ceil(7 |row of R|_1) + 1 <= 14 values and the box is at most 17 cells
// per axis.  The box has fixed pitches (18 cells per row, 312 per plane: of
// the pitches timed, the best over both uniformly spread and clustered
// rotations, whose stencil gathers meet different LDS bank conflicts), so the
// 64 stencil reads of a sample sit at constant offsets from one address.
// Staging gives each wave two planes of the box and three rows per load
// instruction (54 lanes): the lanes' offsets within a plane serve both planes,
// a plane is a buffer descriptor, and its bounds and kBufferNone stand for the
// masks.  All of a wave's loads come before its LDS stores.
// Bound by VALU issue (650 instructions per wave and pose, of which the stencil
// and its weights need 370) and the gathers' LDS cycles, half of them bank
// conflicts, each nine tenths of the time.  1024 poses of a 64^3 body: 4.9 ms;
// 5.6 with row and plane found anew for each load and every sum reduced over
// the 16 lanes of a row by itself (810 instructions).
constexpr int kBoxTile = 8;
constexpr int kBoxBlock = kBoxTile * kBoxTile * kBoxTile;
constexpr int kBoxWaves = kBoxBlock / 64;
constexpr int kBoxMax = 17;
constexpr int kBoxRow = 18;
constexpr int kBoxPlane = 312;
constexpr int kBoxCells = kBoxPlane * kBoxMax;
constexpr int kBoxSlotRows = 3;                                            // rows per wave load
constexpr int kBoxSlotsY = (kBoxMax + kBoxSlotRows - 1) / kBoxSlotRows;       // loads per plane
constexpr float kBoxMargin = 1e-3f;
static_assert(kBoxRow >= kBoxMax && kBoxPlane >= kBoxRow * kBoxMax, "box pitches");
static_assert(kBoxRow * kBoxSlotRows <= 64, "staging rows per wave");
static_assert(kBoxMax == 2 * kBoxWaves + 1 && kBoxSlotsY <= kBoxWaves, "two planes a wave, and one more");

// Per-pose constants of the box kernel, computed once per pose: R in FP32,
// t split into floor and fraction, and the offsets of the moved 8^3 tile's
// bounding box from its moved corner, sum_c min(0, 7 R_ac) and
// sum_c max(0, 7 R_ac).
struct BoxPose {
    float r[9];
    float tfr[3];
    int tint[3];
    float dmin[3];
    float dmax[3];
    float pad[3];
};
static_assert(sizeof(BoxPose) == 96, "BoxPose layout");

__global__ void box_pose_kernel(const double* __restrict__ poses, int64_t B, BoxPose* __restrict__ out) {
    const int64_t b = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double* pose = poses + 7 * b;
    double r64[9];
    quat_rot(pose + 3, r64);
    BoxPose P;
#pragma unroll
    for (int a = 0; a < 9; ++a) P.r[a] = float(r64[a]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double ti = floor(pose[a]);
        P.tint[a] = int(ti);
        P.tfr[a] = float(pose[a] - ti);
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float e = float(kBoxTile - 1) * P.r[3 * a + c];
            lo += fminf(e, 0.f);
            hi += fmaxf(e, 0.f);
        }
        P.dmin[a] = lo;
        P.dmax[a] = hi;
        P.pad[a] = 0.f;
    }
    out[b] = P;
}

// REAL (pose gradients without weight gradients): only Re(c_k Phi) and the
// real parts of c_k times Phi's derivatives are needed, so the stencil
// contracts u = Re(c_k v) per cell, one real product chain instead of a
// complex one from the y sums on (16 fewer VALU instructions per plane).
template <bool GRAD, bool REAL = false>
__global__ __launch_bounds__(kBoxBlock, 2) void grad_box_kernel(const cplx<float>* __restrict__ rho_f, int N,
                                                                const cplx<float>* __restrict__ rho_m,
                                                                const float* __restrict__ w_m, int n_m,
                                                                const BoxPose* __restrict__ bpose, int64_t B,
                                                                const double* __restrict__ gscale,
                                                                double* __restrict__ part, int nsb,
                                                                float* __restrict__ wpart, int want_w, int pb0,
                                                                int per) {
    __shared__ cplx<float> box[kBoxCells];
    __shared__ double red[kBoxBlock / 16][kNAcc];
    const int sb = blockIdx.x, pb = pb0 + int(blockIdx.y);
    const int nt = (n_m + kBoxTile - 1) / kBoxTile;
    const int t0x = (sb % nt) * kBoxTile, t0y = ((sb / nt) % nt) * kBoxTile, t0z = (sb / (nt * nt)) * kBoxTile;
    const int64_t K = int64_t(n_m) * n_m * n_m;
    const float half = 0.5f * float(n_m);
    // this thread's sample: a wave covers a 4 x 4 x 4 sub-block of the tile
    // (compact in 3D, which spreads its stencil gathers over more LDS banks
    // than an 8 x 8 x 1 slice)
    const int wq = int(threadIdx.x >> 6), ln = int(threadIdx.x & 63);
    const int i = t0x + 4 * (wq & 1) + (ln & 3), j = t0y + 4 * ((wq >> 1) & 1) + ((ln >> 2) & 3),
              k = t0z + 4 * (wq >> 2) + (ln >> 4);
    const bool ok = i < n_m && j < n_m && k < n_m;
    const int64_t ks = ok ? (int64_t(k) * n_m + j) * n_m + i : 0;
    const float xb0 = float(i) - half, xb1 = float(j) - half, xb2 = float(k) - half;
    const cplx<float> rm = ok ? rho_m[ks] : mk(0.f, 0.f);
    const cplx<float> ck = rm * (ok ? w_m[ks] : 0.f);
    float gw = 0.f, gwi = 0.f;  // wmode 1: Re(rho_M Phi) sum; 2: Phi sum (re, im)
    // body coordinates of the tile corner (a clipped tile keeps the full
    // tile's bounds, which contain its samples)
    const float xlo0 = float(t0x) - half, xlo1 = float(t0y) - half, xlo2 = float(t0z) - half;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    // staging lane roles: row j_s of a slot of three rows, cell cx_s of the row
    const int js = lane / kBoxRow, cxs = lane - js * kBoxRow;
    const int64_t b0 = int64_t(pb) * per;
    for (int pi = 0; pi < per; ++pi) {
        const int64_t b = b0 + pi;
        if (b >= B) break;  // uniform across the block
        const BoxPose& P = bpose[b];
        float r[9], tfr[3];
        int tint[3], lo[3], ext[3];
#pragma unroll
        for (int a = 0; a < 9; ++a) r[a] = P.r[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            tint[a] = P.tint[a];
            tfr[a] = P.tfr[a];
            const float y0 = tfr[a] + r[3 * a] * xlo0 + r[3 * a + 1] * xlo1 + r[3 * a + 2] * xlo2;
            const int fmin = int(floorf(y0 + P.dmin[a] - kBoxMargin));
            lo[a] = __builtin_amdgcn_readfirstlane(fmin - 1 + tint[a]);
            // at most kBoxMax for any rotation (see above); the clamp only guards
            // non-finite poses, whose conversions give in-range but meaningless boxes
            ext[a] = __builtin_amdgcn_readfirstlane(
                min(int(floorf(y0 + P.dmax[a] + kBoxMargin)) - fmin + 4, kBoxMax));
        }
        // stage the box: a wave takes planes wid and wid + 8, a load rows 3 q .. 3 q + 2
        // of one (lane = kBoxRow j + cx: row 3 q + j, cell cx)
        {
            const unsigned Nu = unsigned(N), plane_bytes = Nu * Nu * unsigned(sizeof(cplx<float>));
            const unsigned wx = unsigned(wrap(lo[0], N)), wy = unsigned(wrap(lo[1], N)), wz = unsigned(wrap(lo[2], N));
            unsigned gx = wx + unsigned(cxs);
            gx = min(gx, gx - Nu);
            const bool lane_ok = js < kBoxSlotRows && cxs < ext[0];
            auto offset = [&](int q) {  // of this lane's cell within a plane
                const int cy = q * kBoxSlotRows + js;
                unsigned gy = wy + unsigned(cy);
                gy = min(gy, gy - Nu);
                return lane_ok && cy < ext[1] ? (__umul24(gy, Nu) + gx) * unsigned(sizeof(cplx<float>)) : kBufferNone;
            };
            auto plane = [&](int cz) {  // no bytes past the box
                unsigned gz = wz + unsigned(cz);
                gz = min(gz, gz - Nu);
                return buffer_rsrc(rho_f + size_t(gz) * Nu * Nu, cz < ext[2] ? plane_bytes : 0u);
            };
            const auto r0 = plane(wid), r1 = plane(wid + kBoxWaves);
            cplx<float> v0[kBoxSlotsY], v1[kBoxSlotsY];
#pragma unroll
            for (int q = 0; q + 1 < kBoxSlotsY; ++q) {
                const unsigned at = offset(q);
                v0[q] = buffer_load_cf(r0, at, 0);
                v1[q] = buffer_load_cf(r1, at, 0);
            }
            const bool tall = ext[1] > (kBoxSlotsY - 1) * kBoxSlotRows;
            if (tall) {
                const unsigned at = offset(kBoxSlotsY - 1);
                v0[kBoxSlotsY - 1] = buffer_load_cf(r0, at, 0);
                v1[kBoxSlotsY - 1] = buffer_load_cf(r1, at, 0);
            }
            cplx<float>* dst = box + wid * kBoxPlane + lane;
            if (lane < kBoxSlotRows * kBoxRow) {
#pragma unroll
                for (int q = 0; q + 1 < kBoxSlotsY; ++q) {
                    dst[q * (kBoxSlotRows * kBoxRow)] = v0[q];
                    dst[kBoxWaves * kBoxPlane + q * (kBoxSlotRows * kBoxRow)] = v1[q];
                }
            }
            constexpr int kLastRows = kBoxMax - (kBoxSlotsY - 1) * kBoxSlotRows;
            if (tall && lane < kLastRows * kBoxRow) {
                dst[(kBoxSlotsY - 1) * (kBoxSlotRows * kBoxRow)] = v0[kBoxSlotsY - 1];
                dst[kBoxWaves * kBoxPlane + (kBoxSlotsY - 1) * (kBoxSlotRows * kBoxRow)] = v1[kBoxSlotsY - 1];
            }
            // the seventeenth plane: a load for each of the first waves
            if (ext[2] > 2 * kBoxWaves && wid < kBoxSlotsY) {
                const cplx<float> v = buffer_load_cf(plane(2 * kBoxWaves), offset(wid), 0);
                if (lane < (wid + 1 < kBoxSlotsY ? kBoxSlotRows : kLastRows) * kBoxRow)
                    box[2 * kBoxWaves * kBoxPlane + wid * (kBoxSlotRows * kBoxRow) + lane] = v;
            }
        }
        __syncthreads();
        const double sc = gscale ? gscale[b] : 1.0;
        double acc[kNAcc];
#pragma unroll
        for (int a = 0; a < kNAcc; ++a) acc[a] = 0.0;
        if (ok) {
            float wgt[3][4], dw[3][4], wv[3];
            int lb[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                wv[a] = r[3 * a] * xb0 + r[3 * a + 1] * xb1 + r[3 * a + 2] * xb2;
                const float y = tfr[a] + wv[a];
                const float fl = floorf(y);
                lb[a] = int(fl) + tint[a] - 1 - lo[a];  // in [0, ext - 4]
                bspline3_weights(y - fl, wgt[a]);
                if (GRAD) bspline3_dweights(y - fl, dw[a]);
            }
            const cplx<float>* base = box + lb[2] * kBoxPlane + lb[1] * kBoxRow + lb[0];
            if constexpr (REAL) {
                // separable contraction of u = Re(c_k v): x, then y, then z
                float phi = 0.f, gx = 0.f, gy = 0.f, gz = 0.f;
#pragma unroll 1
                for (int cz = 0; cz < 4; ++cz) {
                    float wz = wgt[2][0], dz = dw[2][0];
#pragma unroll
                    for (int q = 1; q < 4; ++q)
                        if (cz == q) {
                            wz = wgt[2][q];
                            dz = dw[2][q];
                        }
                    const cplx<float>* plane = base + cz * kBoxPlane;
                    float ay = 0.f, by = 0.f, cy_ = 0.f;
#pragma unroll
                    for (int cy = 0; cy < 4; ++cy) {
                        float rx = 0.f, rdx = 0.f;
#pragma unroll
                        for (int cx = 0; cx < 4; ++cx) {
                            const cplx<float> v = plane[cy * kBoxRow + cx];
                            const float u = ck.re * v.re - ck.im * v.im;
                            rx += u * wgt[0][cx];
                            rdx += u * dw[0][cx];
                        }
                        ay += rx * wgt[1][cy];
                        by += rdx * wgt[1][cy];
                        cy_ += rx * dw[1][cy];
                    }
                    phi += ay * wz;
                    gx += by * wz;
                    gy += cy_ * wz;
                    gz += ay * dz;
                }
                const double g0 = double(gx), g1 = double(gy), g2 = double(gz);
                const double w0 = double(wv[0]), w1 = double(wv[1]), w2 = double(wv[2]);
                acc[0] = double(phi);
                acc[1] = g0;
                acc[2] = g1;
                acc[3] = g2;
                acc[4] = w1 * g2 - w2 * g1;
                acc[5] = w2 * g0 - w0 * g2;
                acc[6] = w0 * g1 - w1 * g0;
            } else {
                // separable contraction: x, then y, then z
                cplx<float> phi = mk(0.f, 0.f), gx = phi, gy = phi, gz = phi;
#pragma unroll 1
                for (int cz = 0; cz < 4; ++cz) {
                    float wz = wgt[2][0], dz = GRAD ? dw[2][0] : 0.f;
#pragma unroll
                    for (int q = 1; q < 4; ++q)
                        if (cz == q) {
                            wz = wgt[2][q];
                            if (GRAD) dz = dw[2][q];
                        }
                    const cplx<float>* plane = base + cz * kBoxPlane;
                    cplx<float> ay = mk(0.f, 0.f), by = ay, cy_ = ay;
#pragma unroll
                    for (int cy = 0; cy < 4; ++cy) {
                        cplx<float> rx = mk(0.f, 0.f), rdx = rx;
#pragma unroll
                        for (int cx = 0; cx < 4; ++cx) {
                            const cplx<float> v = plane[cy * kBoxRow + cx];
                            rx = rx + v * wgt[0][cx];
                            if (GRAD) rdx = rdx + v * dw[0][cx];
                        }
                        ay = ay + rx * wgt[1][cy];
                        if (GRAD) {
                            by = by + rdx * wgt[1][cy];
                            cy_ = cy_ + rx * dw[1][cy];
                        }
                    }
                    phi = phi + ay * wz;
                    if (GRAD) {
                        gx = gx + by * wz;
                        gy = gy + cy_ * wz;
                        gz = gz + ay * dz;
                    }
                }
                acc[0] = double((ck * phi).re);
                if (GRAD) {
                    const double g0 = double((ck * gx).re), g1 = double((ck * gy).re), g2 = double((ck * gz).re);
                    const double w0 = double(wv[0]), w1 = double(wv[1]), w2 = double(wv[2]);
                    acc[1] = g0;
                    acc[2] = g1;
                    acc[3] = g2;
                    acc[4] = w1 * g2 - w2 * g1;
                    acc[5] = w2 * g0 - w0 * g2;
                    acc[6] = w0 * g1 - w1 * g0;
                    if (want_w == 1) gw += float(sc) * (rm * phi).re;
                    if (want_w == 2) {
                        gw += float(sc) * phi.re;
                        gwi += float(sc) * phi.im;
                    }
                }
            }
        }
        // block reduction: rows of 16 lanes (DPP), then 32 row sums per value
        constexpr int nacc = GRAD ? kNAcc : 1;
        if constexpr (GRAD) {
            double two[2];
            row16_sum8(acc, lane, two);
            const int a = 4 * (lane & 1) + (lane & 2);  // this lane holds sums a and a + 1
            if ((lane & 15) < 4) {
                red[wid * 4 + (lane >> 4)][a] = two[0];
                if (a + 1 < nacc) red[wid * 4 + (lane >> 4)][a + 1] = two[1];
            }
        } else {
            const double v = row16_sum(acc[0]);
            if ((lane & 15) == 0) red[wid * 4 + (lane >> 4)][0] = v;
        }
        __syncthreads();  // also: every thread is done reading the box
        if (threadIdx.x < nacc) {
            double v = 0.0;
#pragma unroll
            for (int rw = 0; rw < kBoxBlock / 16; ++rw) v += red[rw][threadIdx.x];
            part[(b * nsb + sb) * kNAcc + threadIdx.x] = v;
        }
    }
    if (GRAD && want_w == 1 && ok) wpart[int64_t(pb) * K + ks] = gw;
    if (GRAD && want_w == 2 && ok) {
        wpart[2 * (int64_t(pb) * K + ks)] = gw;
        wpart[2 * (int64_t(pb) * K + ks) + 1] = gwi;
    }
}

// Per pose: reduce the sample-tile partials, apply the chain rule through
// R(q / |q|) (FP64), write the score and the 7 pose derivatives.
template <typename T, bool GRAD>
__global__ void grad_finish_kernel(const double* __restrict__ part, int nsb, const double* __restrict__ poses,
                                   int64_t B, T* __restrict__ score, double* __restrict__ grad_pose) {
    // one wave per pose: lanes stride over the sample tiles (a pose's partials
    // are contiguous, so a wave's loads are too), then a wave reduction
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    if (b >= B) return;  // uniform across the wave
    double acc[kNAcc];
#pragma unroll
    for (int a = 0; a < kNAcc; ++a) acc[a] = 0.0;
    constexpr int nacc = GRAD ? kNAcc : 1;
    const double* pb = part + b * nsb * kNAcc;
    for (int sb = lane; sb < nsb; sb += 64)
#pragma unroll
        for (int a = 0; a < nacc; ++a) acc[a] += pb[sb * kNAcc + a];
#pragma unroll
    for (int a = 0; a < nacc; ++a) acc[a] = warp_sum(acc[a]);
    if (lane != 0) return;
    score[b] = T(acc[0]);
    if (!GRAD || !grad_pose) return;
    const double* q = poses + 7 * b + 3;
    const double nq = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double w = q[0] / nq, x = q[1] / nq, y = q[2] / nq, z = q[3] / nq;
    // df/du_c = 2 vec(e_c u*) . tau (plus a radial part that the projection
    // below removes), u = (w, x, y, z):
    //   vec(1 u*) = (-x, -y, -z), vec(i u*) = (w, z, -y),
    //   vec(j u*) = (-z, w, x),   vec(k u*) = (y, -x, w)
    const double om[4][3] = {{-x, -y, -z}, {w, z, -y}, {-z, w, x}, {y, -x, w}};
    double gu[4];
    for (int c = 0; c < 4; ++c) gu[c] = 2.0 * (om[c][0] * acc[4] + om[c][1] * acc[5] + om[c][2] * acc[6]);
    // d/dq = (I - u u^T) / |q| applied to d/du
    const double u[4] = {w, x, y, z};
    const double ug = u[0] * gu[0] + u[1] * gu[1] + u[2] * gu[2] + u[3] * gu[3];
    double* g = grad_pose + 7 * b;
    g[0] = acc[1];
    g[1] = acc[2];
    g[2] = acc[3];
    for (int c = 0; c < 4; ++c) g[3 + c] = (gu[c] - u[c] * ug) / nq;
}

template <typename T>
__global__ void wsum_kernel(const T* __restrict__ wpart, int npb, int64_t K, T* __restrict__ grad_w) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    T s = T(0);
    for (int p = 0; p < npb; ++p) s += wpart[int64_t(p) * K + k];
    grad_w[k] = s;
}

// complex tile partials: grad_c[k] = sum over pose tiles of Phi sums
template <typename T>
__global__ void csum_kernel(const T* __restrict__ wpart, int npb, int64_t K, T* __restrict__ grad_c) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    T re = T(0), im = T(0);
    for (int p = 0; p < npb; ++p) {
        re += wpart[2 * (int64_t(p) * K + k)];
        im += wpart[2 * (int64_t(p) * K + k) + 1];
    }
    grad_c[2 * k] = re;
    grad_c[2 * k + 1] = im;
}

// grad_w[k] = Re(rho_M[k] grad_c[k])
template <typename T>
__global__ void w_from_c_kernel(const cplx<T>* __restrict__ rho_m, const T* __restrict__ grad_c, int64_t K,
                                T* __restrict__ grad_w) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    grad_w[k] = rho_m[k].re * grad_c[2 * k] - rho_m[k].im * grad_c[2 * k + 1];
}

// ---- chain-rule products for automatic differentiation
// out[b][j] = gp[b][j] * s[b] (FP64; may be in place)
__global__ void pose_chain_kernel(const double* __restrict__ gp, const double* __restrict__ s, int64_t B,
                                  double* __restrict__ out) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= 7 * B) return;
    out[i] = gp[i] * s[i / 7];
}

// cotangent of rho_M from that of c_k = w_k rho_M(x_k): w_k G_k (complex)
template <typename T>
__global__ void rho_from_c_kernel(const T* __restrict__ w_m, const T* __restrict__ grad_c, int64_t K,
                                  T* __restrict__ grad_rho) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    grad_rho[2 * k] = w_m[k] * grad_c[2 * k];
    grad_rho[2 * k + 1] = w_m[k] * grad_c[2 * k + 1];
}

// ---- cotangent of the scores with respect to rho_F (the adjoint of the
// gather): G(p) = sum_b s_b sum_k c_k B3(p - y_kb), periodic, y_kb = R_b x_k + t_b.
// Per pose: R (FP64).
__device__ __forceinline__ void put_rotation(const double* __restrict__ poses, int64_t b, double* __restrict__ out) {
    double r[9];
    quat_rot(poses + 7 * b + 3, r);
#pragma unroll
    for (int a = 0; a < 9; ++a) out[9 * b + a] = r[a];
}
// Rotations, and the maxima of fixed_max_kernel cleared.
__global__ void fixed_pose_kernel(const double* __restrict__ poses, int64_t B, double* __restrict__ out,
                                  unsigned long long* __restrict__ maxima) {
    const int64_t b = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (b < 2) maxima[b] = 0;
    if (b < B) put_rotation(poses, b, out);
}

// maxima[0] = largest |Re c_k| or |Im c_k| of the finite rho_M and w_M (infinite where their product
// overflows), as the bits of a non-negative double (which order like integers); maxima[1] = 1 if some
// rho_M or w_M is not finite.  Small calls do the rotations and both maxima in one block and launch.
template <typename T, int BLOCK>
__device__ __forceinline__ void coefficient_maxima(const cplx<T>* __restrict__ rho_m, const T* __restrict__ w_m,
                                                   int64_t K, unsigned long long* __restrict__ maxima) {
    __shared__ double sh[BLOCK / 64];
    double m = 0.0;
    bool odd = false;
#pragma unroll 4
    for (int64_t k = int64_t(blockIdx.x) * BLOCK + threadIdx.x; k < K; k += int64_t(gridDim.x) * BLOCK) {
        const cplx<T> r = rho_m[k];
        const T w = w_m[k];
        const bool plain = (r.re - r.re) + (r.im - r.im) + (w - w) == T(0);
        odd |= !plain;
        if (plain) m = fmax(m, fmax(fabs(double(r.re) * double(w)), fabs(double(r.im) * double(w))));
    }
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    const bool any = __syncthreads_or(odd);
    if (threadIdx.x != 0) return;
    for (int wv = 1; wv < BLOCK / 64; ++wv) m = fmax(m, sh[wv]);
    const unsigned long long bits = __double_as_longlong(m);
    if (gridDim.x == 1) {
        maxima[0] = bits;
        maxima[1] = any;
    } else {
        atomicMax(maxima, bits);
        if (any) atomicMax(maxima + 1, 1ull);
    }
}
template <typename T>
__global__ __launch_bounds__(256) void fixed_max_kernel(const cplx<T>* __restrict__ rho_m, const T* __restrict__ w_m,
                                                        int64_t K, unsigned long long* __restrict__ maxima) {
    coefficient_maxima<T, 256>(rho_m, w_m, K, maxima);
}
template <typename T>
__global__ __launch_bounds__(1024) void fixed_prep_kernel(const cplx<T>* __restrict__ rho_m, const T* __restrict__ w_m,
                                                          int64_t K, const double* __restrict__ poses, int64_t B,
                                                          double* __restrict__ out,
                                                          unsigned long long* __restrict__ maxima) {
    for (int64_t b = threadIdx.x; b < B; b += 1024) put_rotation(poses, b, out);
    coefficient_maxima<T, 1024>(rho_m, w_m, K, maxima);
}

// A block owns a tile of the fixed grid and a range of poses: for every pose
// and every periodic image of the tile that the turned box reaches, the samples
// in reach (DENSE: all samples, or a part of them, wrapped) add their taps to LDS
// sums; each node is stored once, to out or to a partial grid.  It replaces one global atomic
// pair per tap, at 23 billion a second: 32 poses of a 32^3 box on 64^3 nodes
// 5.9 -> 0.26 ms.  Bound by LDS adds and VALU issue.
// Sums of a pose are 64-bit integers in units of at most 2^-57 max|c_k| |s_b|, and
// move to FP64 registers after each pose, in order: runs repeat bit for bit, and
// poses of any scale keep their digits beside larger ones (one scale for all
// poses left three of a pose at 1e-6 of the largest, in FP32).  Moving costs 200
// instructions a wave, a pose's samples some thousands.  On the torus at most 8
// images of the body meet, the splines of each sum to little over 1, and 2^58 an
// image leaves room for 32 before a sum reaches 2^63.
// A term that is not finite is a flag of its node, for an infinity of either sign
// or, as both, NaN.
constexpr double kFixedTop = 288230376151711744.0;  // 2^58
template <typename T>
__device__ __forceinline__ void flag_term(unsigned* flags, int words, int node, T v) {
    const unsigned bit = 1u << (node % 32);
    if (!(v < T(0))) atomicOr(flags + node / 32, bit);
    if (!(v > T(0))) atomicOr(flags + words + node / 32, bit);
}
__device__ __forceinline__ double flagged(const unsigned* flags, int words, int node) {
    const bool up = (flags[node / 32] >> (node % 32)) & 1, down = (flags[words + node / 32] >> (node % 32)) & 1;
    return up ? (down ? NAN : INFINITY) : (down ? -INFINITY : 0.0);
}
template <typename T, bool PLANAR, int BLOCK, bool DENSE>
__global__ __launch_bounds__(BLOCK, BLOCK == kTileBlock ? 3 : 1)
void fixed_tile_kernel(const cplx<T>* __restrict__ rho_m, const T* __restrict__ w_m, int n_m,
                       const double* __restrict__ rot, const double* __restrict__ poses,
                       const double* __restrict__ gscale, int64_t B, int64_t per, int grids, int parts, int N,
                       int64_t tiles, int64_t step, const unsigned long long* __restrict__ maxima,
                       cplx<T>* __restrict__ out) {
    using S = SpreadTile<PLANAR>;
    constexpr int OWN = S::X * S::Y * S::Z / BLOCK;  // nodes a thread stores
    __shared__ unsigned long long acc[S::WORDS];
    constexpr int FLAGS = S::X * S::Y * S::Z / 32;  // words per sign and part
    __shared__ unsigned bad[4 * FLAGS];
    const int ntx = (N + S::X - 1) / S::X, nty = (N + S::Y - 1) / S::Y;
    const int grid = int(blockIdx.x % unsigned(grids)), range = grid / parts;
    const int tile = int(scattered_tile(int64_t(blockIdx.x / unsigned(grids)), tiles, step));
    const int t0[3] = {(tile % ntx) * S::X, ((tile / ntx) % nty) * S::Y, PLANAR ? 0 : (tile / (ntx * nty)) * S::Z};
    const int dim[3] = {min(S::X, N - t0[0]), min(S::Y, N - t0[1]), PLANAR ? 1 : min(S::Z, N - t0[2])};
    const double cm = __longlong_as_double((long long)maxima[0]);
    for (int i = int(threadIdx.x); i < S::WORDS; i += BLOCK) acc[i] = 0;
    for (int i = int(threadIdx.x); i < 4 * FLAGS; i += BLOCK) bad[i] = 0;
    double sr[OWN], si[OWN];
#pragma unroll
    for (int o = 0; o < OWN; ++o) sr[o] = si[o] = 0.0;
    __syncthreads();
    auto flush = [&](double inv) {
        __syncthreads();
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            const int nd = o * BLOCK + int(threadIdx.x);
            unsigned long long* a = acc + (nd / S::X) * S::PITCH + nd % S::X;
            sr[o] += double((long long)a[0]) * inv;
            si[o] += double((long long)a[S::IMAG]) * inv;
            a[0] = a[S::IMAG] = 0;
        }
        __syncthreads();
    };
    const Fixed64 fixed;
    const T half_box = T(0.5) * T(n_m);
    const int64_t b0 = int64_t(range) * per, b1 = b0 + per < B ? b0 + per : B;
    for (int64_t b = b0; b < b1; ++b) {
        const double* P = rot + 9 * b;
        const double* pose = poses + 7 * b;
        T r[9], tfr[3];
        float rf[9], ylo[3], yhi[3];
        int tw[3];  // floor of t on the grid
        const T sb = T(gscale ? gscale[b] : 1.0);
        bool finite = true;
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            r[a] = T(P[a]);
            rf[a] = float(P[a]);
            finite &= fabs(P[a]) < INFINITY;
        }
#pragma unroll
        for (int a = 0; a < (PLANAR ? 2 : 3); ++a) {
            const double ti = floor(pose[a]);
            finite &= fabs(ti) < INFINITY;
            tfr[a] = T(pose[a] - ti);
            tw[a] = int(ti - double(N) * floor(ti / double(N)));
            // reach of the turned box, and the tile's images m N it meets
            const float h = 0.5f * float(n_m), e = h - 1.f;
            ylo[a] = yhi[a] = float(tfr[a]);
#pragma unroll
            for (int q = 0; q < (PLANAR ? 2 : 3); ++q) {
                ylo[a] += fminf(-h * rf[3 * a + q], e * rf[3 * a + q]);
                yhi[a] += fmaxf(-h * rf[3 * a + q], e * rf[3 * a + q]);
            }
        }
        if (!finite) {  // uniform: every weight of a sample's stencil is NaN, and the stencil lies where the
                        // conversions put it; a sample without a term (a pose of scale zero) reaches nothing
            const int64_t K = sb == T(0) && !maxima[1] ? 0 : int64_t(n_m) * n_m * (PLANAR ? 1 : n_m);
            for (int64_t kk = int64_t(threadIdx.x); kk < K; kk += BLOCK) {
                const cplx<T> ck = rho_m[kk] * (w_m[kk] * sb);
                if (ck.re == T(0) && ck.im == T(0)) continue;
                const int64_t row = kk / n_m;
                const T xb[3] = {T(int(kk - row * n_m)) - half_box, T(int(row % n_m)) - half_box,
                                 PLANAR ? T(0) : T(int(row / n_m)) - half_box};
                unsigned first[3] = {0, 0, 0};  // sums of large conversions wrap
#pragma unroll
                for (int a = 0; a < (PLANAR ? 2 : 3); ++a) {
                    const double ti = floor(pose[a]);
                    const T y = T(pose[a] - ti) + r[3 * a] * xb[0] + r[3 * a + 1] * xb[1] + r[3 * a + 2] * xb[2];
                    first[a] = unsigned(int(dev_floor(y))) + unsigned(int(ti)) - 1u;
                }
                for (int tap = 0; tap < (PLANAR ? 16 : 64); ++tap) {
                    const int ix = wrap(int(first[0] + (tap & 3)), N) - t0[0],
                              iy = wrap(int(first[1] + ((tap >> 2) & 3)), N) - t0[1],
                              iz = PLANAR ? 0 : wrap(int(first[2] + (tap >> 4)), N) - t0[2];
                    if (unsigned(ix) >= unsigned(dim[0]) || unsigned(iy) >= unsigned(dim[1]) ||
                        unsigned(iz) >= unsigned(dim[2]))
                        continue;
                    const int nd = (iz * S::Y + iy) * S::X + ix;
                    flag_term(bad, FLAGS, nd, T(NAN));
                    flag_term(bad + 2 * FLAGS, FLAGS, nd, T(NAN));
                }
            }
            continue;
        }
        // (terms that are finite are at most the largest finite T)
        const double most = fmin(cm * fabs(double(sb)), double(std::numeric_limits<T>::max()));
        const double pow2 = pow2_below(fmin(kFixedTop / most, 1e300));
        bool touched = false;  // uniform
        // a tap's node within the tile: on the torus where the sample's stencil was
        // wrapped as a whole, else that of its image
        auto tap = [&](int a, int at) { return DENSE && at >= N - t0[a] ? at - N : at; };
        auto add_sample = [&](int i, int j, int k, const int o[3]) {
            const int kk = (k * n_m + j) * n_m + i;
            cplx<T> ck = rho_m[kk] * (w_m[kk] * sb);
            if (ck.re == T(0) && ck.im == T(0)) return;
            const bool fin_re = ck.re - ck.re == T(0), fin_im = ck.im - ck.im == T(0);
            const double vr = fin_re ? double(ck.re) * pow2 : 0.0, vi = fin_im ? double(ck.im) * pow2 : 0.0;
            const T xb[3] = {T(i) - half_box, T(j) - half_box, PLANAR ? T(0) : T(k) - half_box};
            int b3[3] = {0, 0, 0};
            T wgt[3][4];
#pragma unroll
            for (int a = 0; a < (PLANAR ? 2 : 3); ++a) {
                const T y = tfr[a] + r[3 * a] * xb[0] + r[3 * a + 1] * xb[1] + r[3 * a + 2] * xb[2];
                const T fl = dev_floor(y);
                b3[a] = int(fl) - 1 - o[a];
                if constexpr (DENSE) b3[a] = wrap(b3[a] + t0[a], N) - t0[a];
                bspline3_weights(y - fl, wgt[a]);
            }
#pragma unroll
            for (int cz = 0; cz < (PLANAR ? 1 : 4); ++cz) {
                const int iz = PLANAR ? 0 : tap(2, b3[2] + cz);
                if (unsigned(iz) >= unsigned(dim[2])) continue;
#pragma unroll
                for (int cy = 0; cy < 4; ++cy) {
                    const int iy = tap(1, b3[1] + cy);
                    if (unsigned(iy) >= unsigned(dim[1])) continue;
                    const T wyz = PLANAR ? wgt[1][cy] : wgt[1][cy] * wgt[2][cz];
                    const double row_re = vr * double(wyz), row_im = vi * double(wyz);
                    const int row = iz * S::Y + iy;
#pragma unroll
                    for (int cx = 0; cx < 4; ++cx) {
                        const int ix = tap(0, b3[0] + cx);
                        if (unsigned(ix) >= unsigned(dim[0])) continue;
                        unsigned long long* a = acc + row * S::PITCH + ix;
                        if (!(fin_re && fin_im)) {
                            const T wt = wgt[0][cx] * wyz;
                            const int nd = row * S::X + ix;
                            if (!fin_re) flag_term(bad, FLAGS, nd, ck.re * wt);
                            if (!fin_im) flag_term(bad + 2 * FLAGS, FLAGS, nd, ck.im * wt);
                        }
                        atomicAdd(a, fixed(row_re * double(wgt[0][cx])));
                        atomicAdd(a + S::IMAG, fixed(row_im * double(wgt[0][cx])));
                    }
                }
            }
        };
        if constexpr (DENSE) {  // every sample of the body reaches the tile, or nearly
            const int o[3] = {t0[0] - tw[0], t0[1] - tw[1], PLANAR ? 0 : t0[2] - tw[2]};
            const int K = n_m * n_m * (PLANAR ? 1 : n_m);
            for (int kk = grid % parts * BLOCK + int(threadIdx.x); kk < K; kk += parts * BLOCK)
                add_sample(kk % n_m, kk / n_m % n_m, PLANAR ? 0 : kk / (n_m * n_m), o);
            touched = true;
        } else {
            int m0[3] = {0, 0, 0}, m1[3] = {0, 0, 0};
#pragma unroll
            for (int a = 0; a < (PLANAR ? 2 : 3); ++a) {
                const float base = float(t0[a] - tw[a]);
                m0[a] = uniform(int(ceilf((ylo[a] - 0.05f - (base + float(dim[a] + 1))) / float(N))));
                m1[a] = uniform(int(floorf((yhi[a] + 0.05f - (base - 2.f)) / float(N))));
            }
            for (int mz = m0[2]; mz <= m1[2]; ++mz)
                for (int my = m0[1]; my <= m1[1]; ++my)
                    for (int mx = m0[0]; mx <= m1[0]; ++mx) {
                        const int o[3] = {t0[0] - tw[0] + mx * N, t0[1] - tw[1] + my * N,
                                          PLANAR ? 0 : t0[2] - tw[2] + mz * N};
                        float lo[3], hi[3];
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            const float f = PLANAR && a == 2 ? 0.f : float(tfr[a]);
                            lo[a] = float(o[a] - 2) - f;
                            hi[a] = float(o[a] + dim[a] + 1) - f;
                        }
                        touched |= box_samples<PLANAR>(rf, n_m, lo, hi, uniform(int(threadIdx.x) >> 6), BLOCK / 64,
                                                       [&](int i, int j, int k) { add_sample(i, j, k, o); });
                    }
        }
        if (touched) flush(1.0 / pow2);
    }
    __syncthreads();  // flags of a pose that is not finite
    const int64_t G = PLANAR ? int64_t(N) * N : int64_t(N) * N * N;
    cplx<T>* dst = out + int64_t(grid) * G;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
        const int nd = o * BLOCK + int(threadIdx.x);
        const int ix = nd % S::X, iy = (nd / S::X) % S::Y, iz = nd / (S::X * S::Y);
        if (ix >= dim[0] || iy >= dim[1] || iz >= dim[2]) continue;
        dst[(int64_t(t0[2] + iz) * N + t0[1] + iy) * N + t0[0] + ix] =
            mk(T(sr[o] + flagged(bad, FLAGS, nd)), T(si[o] + flagged(bad + 2 * FLAGS, FLAGS, nd)));
    }
}

// out = sum of the partial grids, in order
template <typename T>
__global__ void fixed_sum_kernel(const T* __restrict__ part, int ranges, int64_t count, T* __restrict__ out) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += int64_t(gridDim.x) * blockDim.x) {
        double s = 0.0;
        for (int r = 0; r < ranges; ++r) s += double(part[int64_t(r) * count + i]);
        out[i] = T(s);
    }
}

// tiles of a fixed grid
int64_t fixed_tiles(int N, bool planar) {
    auto up = [&](int s) { return int64_t((N + s - 1) / s); };
    return planar ? up(SpreadTile<true>::X) * up(SpreadTile<true>::Y)
                  : up(SpreadTile<false>::X) * up(SpreadTile<false>::Y) * up(SpreadTile<false>::Z);
}

// R of every pose, then the maxima in the last 16 bytes
constexpr size_t kFixedTail = 16;
size_t fixed_table_bytes(int64_t B) { return (sizeof(double) * 9 * size_t(B) + 15) / 16 * 16 + kFixedTail; }

}  // namespace

// the LDS-staged kernel serves 3D FP32 poses; FP64 and planar use the tile kernel
template <typename T>
bool use_box(bool planar, int N) {
    return std::is_same<T, float>::value && !planar && N >= kBoxMax && N <= 1024;
}

// Blocks of a pose kernel: nsb sample tiles (of 256 spt samples, or the box
// kernel's 8^3) x npb groups of `per` poses.  A block that walks 16 poses
// reuses its samples' registers, which pays while the chip is full; below
// kFewBlocks blocks the walk is a serial chain on a part of the CUs, so the
// groups shrink and, at one pose a block, the tile kernel's samples go one to
// a thread.  Weight gradients hold one partial per group and sample and a last
// kernel walks them, so they keep to 64 groups.  64 tiles of 32 poses (box
// kernel, gradients of poses and samples): 90 us in 128 blocks, 35 us in 1024.
constexpr int64_t kFewBlocks = 1024;
constexpr int64_t kFewGroups = 64;
struct GradSplit {
    int64_t nsb, npb;
    int spt, per;
};
template <typename T>
GradSplit grad_split(int64_t B, int N, int n_m, bool planar, int wmode, bool fine) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const int64_t nt = (n_m + kBoxTile - 1) / kBoxTile;
    const bool box = use_box<T>(planar, N);
    auto tiles = [&](int spt) { return box ? nt * nt * nt : (K + kGBlock * spt - 1) / (kGBlock * spt); };
    GradSplit g{tiles(kSPT), 0, kSPT, kPosesPerBlock};
    if (fine) {
        const int64_t least = std::min<int64_t>(wmode ? (B + kFewGroups - 1) / kFewGroups : 1, kPosesPerBlock);
        if (g.nsb * ((B + least - 1) / least) < kFewBlocks) {
            g.per = int(least);
            g.spt = 1;
            g.nsb = tiles(1);
        } else {  // at most kFewBlocks: four a CU and no fifth to wait for
            const int64_t per = (g.nsb * B + kFewBlocks - 1) / kFewBlocks;
            g.per = int(std::min<int64_t>(std::max(per, least), kPosesPerBlock));
        }
    }
    g.npb = (B + g.per - 1) / g.per;
    return g;
}

template <typename T>
size_t grad_workspace_bytes(int64_t B, int N, int n_m, bool planar, int wmode, bool fine) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const GradSplit g = grad_split<T>(B, N, n_m, planar, wmode, fine);
    size_t bytes = size_t(B * g.nsb * kNAcc) * sizeof(double);
    bytes = (bytes + 255) / 256 * 256;
    if (wmode) bytes += (size_t(g.npb * K) * sizeof(T) * size_t(wmode) + 255) / 256 * 256;
    if (use_box<T>(planar, N)) bytes += size_t(B) * sizeof(BoxPose);
    return bytes + 256;
}

template <typename T>
hipError_t launch_score_grad(const void* rho_f, int N, bool planar, const void* rho_m, const T* w_m, int n_m,
                             const double* poses, int64_t B, T* score, double* grad_pose, T* grad_w, T* grad_c,
                             const double* grad_scale, void* ws, size_t ws_bytes, hipStream_t s) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    // weight mode: 2 sums Phi (complex) per sample, from which grad_w follows;
    // 1 sums Re(rho_M Phi) directly
    const int ww = grad_c ? 2 : (grad_w ? 1 : 0);
    const bool fine = ws_bytes >= grad_workspace_bytes<T>(B, N, n_m, planar, ww, true);
    const GradSplit gs = grad_split<T>(B, N, n_m, planar, ww, fine);
    const int nsb = int(gs.nsb), npb = int(gs.npb), per = gs.per;
    double* part = static_cast<double*>(ws);
    size_t off = size_t(B * nsb * kNAcc) * sizeof(double);
    off = (off + 255) / 256 * 256;
    T* wpart = reinterpret_cast<T*>(static_cast<char*>(ws) + off);
    if (ww) off += (size_t(gs.npb * K) * sizeof(T) * size_t(ww) + 255) / 256 * 256;
    BoxPose* bpose = reinterpret_cast<BoxPose*>(static_cast<char*>(ws) + off);
    if (use_box<T>(planar, N)) {
        hipLaunchKernelGGL(box_pose_kernel, dim3(unsigned((B + 127) / 128)), dim3(128), 0, s, poses, B, bpose);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool grad = grad_pose != nullptr || ww != 0;
    const auto* rf = static_cast<const cplx<T>*>(rho_f);
    const auto* rm = static_cast<const cplx<T>*>(rho_m);
    // pose tiles run in launches of at most 65535 along grid y
    for (int pb0 = 0; pb0 < npb; pb0 += 65535) {
        const dim3 grid{unsigned(nsb), unsigned(std::min(npb - pb0, 65535)), 1u};
        if constexpr (std::is_same<T, float>::value) {
            if (use_box<T>(planar, N)) {
                if (grad && ww == 0)
                    hipLaunchKernelGGL((grad_box_kernel<true, true>), grid, dim3(kBoxBlock), 0, s, rf, N, rm, w_m, n_m,
                                       bpose, B, grad_scale, part, nsb, wpart, 0, pb0, per);
                else if (grad)
                    hipLaunchKernelGGL((grad_box_kernel<true>), grid, dim3(kBoxBlock), 0, s, rf, N, rm, w_m, n_m, bpose,
                                       B, grad_scale, part, nsb, wpart, ww, pb0, per);
                else
                    hipLaunchKernelGGL((grad_box_kernel<false>), grid, dim3(kBoxBlock), 0, s, rf, N, rm, w_m, n_m,
                                       bpose, B, grad_scale, part, nsb, wpart, 0, pb0, per);
            }
        }
        if (!use_box<T>(planar, N)) {
            auto tile = [&](auto kernel, int want_w) {
                hipLaunchKernelGGL(kernel, grid, dim3(kGBlock), 0, s, rf, N, planar ? 1 : 0, rm, w_m, n_m, poses, B,
                                   grad_scale, part, nsb, wpart, want_w, pb0, per);
            };
            if (gs.spt == 1) {
                if (grad) tile(grad_tile_kernel<T, true, 1>, ww);
                else tile(grad_tile_kernel<T, false, 1>, 0);
            } else {
                if (grad) tile(grad_tile_kernel<T, true, kSPT>, ww);
                else tile(grad_tile_kernel<T, false, kSPT>, 0);
            }
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 g2(unsigned((B + 3) / 4));  // 4 waves of 64 lanes per block, one pose per wave
    if (grad)
        hipLaunchKernelGGL((grad_finish_kernel<T, true>), g2, dim3(256), 0, s, part, nsb, poses, B, score, grad_pose);
    else
        hipLaunchKernelGGL((grad_finish_kernel<T, false>), g2, dim3(256), 0, s, part, nsb, poses, B, score, nullptr);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 gk(unsigned((K + 255) / 256));
    if (ww == 1) {
        hipLaunchKernelGGL(wsum_kernel<T>, gk, dim3(256), 0, s, wpart, npb, K, grad_w);
    } else if (ww == 2) {
        hipLaunchKernelGGL(csum_kernel<T>, gk, dim3(256), 0, s, wpart, npb, K, grad_c);
        if (grad_w) hipLaunchKernelGGL(w_from_c_kernel<T>, gk, dim3(256), 0, s, rm, grad_c, K, grad_w);
    }
    return hipGetLastError();
}

// How the fixed cotangent's work is cut.  Grids of few tiles split the poses into
// ranges so that about 4096 blocks run (the tiles a small box reaches are few, so
// one range per resident block leaves some CUs with two busy tiles and most with
// none).  Where a tile with its stencils is half of the torus or more, or few
// blocks would run at all, a block walks all samples, wrapped: the many images of
// a small torus each cost a search of the body's lines.  With few blocks it walks
// a part of them.  Each pose range and part has a partial grid.  FP32 calls: one
// pose of a 16^3 body on 16^3 nodes 154 us by images, 63 by samples, 27 in four
// parts; 3 of 17^3 on 17^3 158, 95, 47; one of 8^3 on 8^3 87, 22; but 25 of 16^3 on
// 32^3 65, 116.
constexpr int kDenseBlock = 1024;
struct FixedSplit {
    int64_t ranges, per, parts;  // per: poses of a range
    bool dense;
    int64_t grids() const { return ranges * parts; }
};
FixedSplit fixed_split(int64_t B, int N, int n_m, bool planar, bool split) {
    const int64_t tiles = fixed_tiles(N, planar), K = int64_t(n_m) * n_m * (planar ? 1 : n_m);
    FixedSplit f{1, B, 1, N <= (planar ? 48 : 20)};
    if (!split) return f;
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(4096 / tiles, std::min<int64_t>(B, 64)));
    f.per = (B + most - 1) / most;
    f.ranges = (B + f.per - 1) / f.per;
    const int64_t blocks = tiles * f.ranges;
    f.dense |= blocks <= 64 && N <= (planar ? 64 : 48);
    // a part of 1024 samples (planar, a quarter of the taps: 4096) repays its sum
    if (f.dense) f.parts = std::max<int64_t>(1, std::min(K / (planar ? 4 * kDenseBlock : kDenseBlock), 256 / blocks));
    return f;
}
template <typename T>
size_t fixed_cotangent_bytes(int64_t B, int N, int n_m, bool planar, bool split) {
    const size_t G = size_t(N) * N * (planar ? 1 : N);
    const int64_t g = fixed_split(B, N, n_m, planar, split).grids();
    return fixed_table_bytes(B) + (g > 1 ? size_t(g) * G * 2 * sizeof(T) : 0);
}

template <typename T>
hipError_t launch_fixed_cotangent(const void* rho_m, const T* w_m, int n_m, bool planar, int N, const double* poses,
                                  int64_t B, const double* grad_scale, void* grad_f, void* ws, size_t ws_bytes,
                                  hipStream_t s) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const int64_t G = planar ? int64_t(N) * N : int64_t(N) * N * N;
    double* rot = static_cast<double*>(ws);
    auto* maxima = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + fixed_table_bytes(B) - kFixedTail);
    auto* part = reinterpret_cast<cplx<T>*>(static_cast<char*>(ws) + fixed_table_bytes(B));
    const auto* rm = static_cast<const cplx<T>*>(rho_m);
    if (K <= 16384 && B <= 2048) {  // one launch of a chain of three or four
        hipLaunchKernelGGL(fixed_prep_kernel<T>, dim3(1), dim3(1024), 0, s, rm, w_m, K, poses, B, rot, maxima);
    } else {
        hipLaunchKernelGGL(fixed_pose_kernel, dim3(unsigned((B + 127) / 128)), dim3(128), 0, s, poses, B, rot, maxima);
        const unsigned blocks = unsigned(std::min<int64_t>((K + 255) / 256, 256));
        hipLaunchKernelGGL(fixed_max_kernel<T>, dim3(blocks), dim3(256), 0, s, rm, w_m, K, maxima);
    }
    const int64_t tiles = fixed_tiles(N, planar);
    const FixedSplit f =
        fixed_split(B, N, n_m, planar, ws_bytes >= fixed_cotangent_bytes<T>(B, N, n_m, planar, true));
    cplx<T>* dst = f.grids() > 1 ? part : static_cast<cplx<T>*>(grad_f);
    // the ranges of a tile side by side and the tiles scattered, so that every
    // CU gets its share of the body's tiles (64^3 field, 32 poses of a 32^3
    // body: 334 us with the tiles in order, 213 so, of FP32 terms rounded to one
    // word; 265 with the two-word ones)
    const int64_t step = tile_step(tiles);
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(f.grids() * tiles)), dim3(threads), 0, s, rm, w_m, n_m, rot, poses,
                           grad_scale, B, f.per, int(f.grids()), int(f.parts), N, tiles, step, maxima, dst);
    };
    if (f.dense) {
        if (planar) run(fixed_tile_kernel<T, true, kDenseBlock, true>, kDenseBlock);
        else run(fixed_tile_kernel<T, false, kDenseBlock, true>, kDenseBlock);
    } else {
        if (planar) run(fixed_tile_kernel<T, true, kTileBlock, false>, kTileBlock);
        else run(fixed_tile_kernel<T, false, kTileBlock, false>, kTileBlock);
    }
    if (f.grids() > 1)
        hipLaunchKernelGGL(fixed_sum_kernel<T>, dim3(unsigned(std::min<int64_t>((2 * G + 255) / 256, 4096))), dim3(256),
                           0, s, reinterpret_cast<const T*>(part), int(f.grids()), 2 * G, static_cast<T*>(grad_f));
    return hipGetLastError();
}

hipError_t launch_pose_chain(const double* gp, const double* scale, int64_t B, double* out, hipStream_t s) {
    hipLaunchKernelGGL(pose_chain_kernel, dim3(unsigned((7 * B + 255) / 256)), dim3(256), 0, s, gp, scale, B, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rho_from_c(const T* w_m, const void* grad_c, int64_t K, void* grad_rho, hipStream_t s) {
    hipLaunchKernelGGL(rho_from_c_kernel<T>, dim3(unsigned((K + 255) / 256)), dim3(256), 0, s, w_m,
                       static_cast<const T*>(grad_c), K, static_cast<T*>(grad_rho));
    return hipGetLastError();
}
template hipError_t launch_rho_from_c<float>(const float*, const void*, int64_t, void*, hipStream_t);
template hipError_t launch_rho_from_c<double>(const double*, const void*, int64_t, void*, hipStream_t);

template size_t fixed_cotangent_bytes<float>(int64_t, int, int, bool, bool);
template size_t fixed_cotangent_bytes<double>(int64_t, int, int, bool, bool);
template hipError_t launch_fixed_cotangent<float>(const void*, const float*, int, bool, int, const double*, int64_t,
                                                  const double*, void*, void*, size_t, hipStream_t);
template hipError_t launch_fixed_cotangent<double>(const void*, const double*, int, bool, int, const double*, int64_t,
                                                   const double*, void*, void*, size_t, hipStream_t);
template size_t grad_workspace_bytes<float>(int64_t, int, int, bool, int, bool);
template size_t grad_workspace_bytes<double>(int64_t, int, int, bool, int, bool);
template hipError_t launch_score_grad<float>(const void*, int, bool, const void*, const float*, int, const double*,
                                             int64_t, float*, double*, float*, float*, const double*, void*, size_t,
                                             hipStream_t);
template hipError_t launch_score_grad<double>(const void*, int, bool, const void*, const double*, int, const double*,
                                              int64_t, double*, double*, double*, double*, const double*, void*, size_t,
                                              hipStream_t);

}  // namespace sdf
