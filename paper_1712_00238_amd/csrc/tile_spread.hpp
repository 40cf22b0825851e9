// Spreading samples of a rotated body lattice onto a tile of grid nodes in
// LDS: the samples that reach a tile, found wave by wave, and the integer sums
// that take their terms.  Used by the multi-pass search (one rotation per tile)
// and by the fixed field's cotangent (all poses per tile).
#pragma once

#include "common.hpp"

namespace sdf {

namespace {

// Tile of nodes a block owns: 3D 16 x 16 x 8 (34 KiB of 64-bit sums: four
// blocks per CU; a sample is visited 1.9 times on average), planar 32 x 32.
template <bool PLANAR>
struct SpreadTile {
    static constexpr int X = PLANAR ? 32 : 16, Y = PLANAR ? 32 : 16, Z = PLANAR ? 1 : 8;
    static constexpr int PITCH = X + 1;
    // sums of the real parts, then of the imaginary parts: neighbouring nodes
    // one 8-byte slot apart ((re, im) pairs would leave every second slot idle
    // during each add)
    static constexpr int IMAG = Z * Y * PITCH;
    static constexpr int WORDS = 2 * IMAG;
};
constexpr int kTileBlock = 256;

// Calls f(i, j, k) for every body sample x = (i, j, k) - n_m / 2 whose position
// R x (r: FP32 rows of R) lies in the box [lo, hi), and for a few outside it
// (within 0.02, or on a line that an edge of the box nearly runs along: f tests
// exactly).  A wave takes 64 body lines along i at a time
// (every waves-th line, so that all of a block's waves share few lines); the
// box cuts each line to one run of samples, and the runs are laid end to end
// over the lanes, so f runs with full waves.  No barrier.  False (for all waves
// alike) if the box holds no line.
template <bool PLANAR, typename F>
__device__ __forceinline__ bool box_samples(const float r[9], int n_m, const float lo[3], const float hi[3], int wave,
                                            int waves, F&& f) {
    constexpr int D = PLANAR ? 2 : 3;
    const float half = 0.5f * float(n_m);
    int first[3], last[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (PLANAR && a == 2) {
            first[a] = last[a] = 0;
            continue;
        }
        float mid = half, ext = 0.05f;
#pragma unroll
        for (int b = 0; b < D; ++b) {
            mid += r[3 * b + a] * (0.5f * (lo[b] + hi[b]));
            ext += fabsf(r[3 * b + a]) * (0.5f * (hi[b] - lo[b]));
        }
        first[a] = max(0, int(ceilf(mid - ext)));
        last[a] = min(n_m - 1, int(floorf(mid + ext)));
        if (last[a] < first[a]) return false;  // uniform
    }
    const int nj = last[1] - first[1] + 1, lines = nj * (last[2] - first[2] + 1);
    const int lane = int(threadIdx.x) & 63;
    for (int l0 = wave; l0 < lines; l0 += 64 * waves) {
        const int l = l0 + lane * waves;
        const float bj = float(first[1] + l % nj) - half, bk = PLANAR ? 0.f : float(first[2] + l / nj) - half;
        float a = float(first[0]), b = float(last[0]);
        bool ok = l < lines;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float y0 = r[3 * c + 1] * bj + r[3 * c + 2] * bk - r[3 * c] * half, s = r[3 * c];
            if (fabsf(s) < 1e-4f) {  // all of the line or nothing: its samples lie between y0 and y0 + s n_m
                const float y1 = y0 + s * float(n_m);
                ok &= fmaxf(y0, y1) >= lo[c] - 0.04f && fminf(y0, y1) <= hi[c] + 0.04f;
            } else {
                const float inv = 1.f / s;
                const float q1 = (lo[c] - 0.02f - y0) * inv, q2 = (hi[c] + 0.02f - y0) * inv;
                a = fmaxf(a, fminf(q1, q2));
                b = fminf(b, fmaxf(q1, q2));
            }
        }
        const int ia = int(ceilf(a));
        int run = ok ? max(0, int(floorf(b)) - ia + 1) : 0;
        int sum = run;  // inclusive prefix sum over the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(sum, off);
            if (lane >= off) sum += o;
        }
        const int total = __builtin_amdgcn_readlane(sum, 63);
        for (int p0 = 0; p0 < total; p0 += 64) {
            const int p = p0 + lane;
            int q = 0;  // first line whose prefix sum exceeds p
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(sum, q + step - 1) <= p) q += step;
            q = min(q, 63);
            const int i = __shfl(ia, q) + p - (__shfl(sum, q) - __shfl(run, q));
            const int ql = l0 + q * waves;
            if (p < total) f(i, first[1] + ql % nj, first[2] + ql / nj);
        }
    }
    return true;
}

// 64-bit integer nearest v, |v| < 2^62, in two exact steps: adding m = 1.5 2^52
// leaves an integer in the low words.  The first step's m is short by the high
// word that the second leaves above its own, so the words meet in one add.  The
// constants are a kernel's variables that the compiler cannot see through: as
// literals they cost five moves a term, more than the arithmetic.
struct Fixed64 {
    double mh, ml, up;
    __device__ __forceinline__ Fixed64()
        : mh(6755399441055744.0 - 1127743488.0), ml(6755399441055744.0), up(2.3283064365386963e-10) {  // 0x43380000
        asm("" : "+v"(mh));
        asm("" : "+v"(ml));
        asm("" : "+s"(up));
    }
    __device__ __forceinline__ unsigned long long operator()(double v) const {
        const double hm = __builtin_fma(v, up, mh);
        const double l = __builtin_fma(hm - mh, -4294967296.0, v);
        const double lm = l + ml;  // l in [-2^31, 2^31]: the words of the signed integer l, plus m's high word
        unsigned hi = unsigned(__double2loint(hm)) + unsigned(__double2hiint(lm));
        asm("" : "+v"(hi));
        return (static_cast<unsigned long long>(hi) << 32) | unsigned(__double2loint(lm));
    }
};

// the largest power of two not above v (v > 0, normal): scaling by it rounds nothing
__device__ __forceinline__ double pow2_below(double v) {
    return __longlong_as_double(__double_as_longlong(v) & 0x7ff0000000000000ll);
}

}  // namespace

}  // namespace sdf
