// Plain multi-pass correlation path, one template for FP32 and FP64, every
// launch over a batch of rotations:
//   quaternions -> rotation matrices (FP64), c_k = w_k rho_M(x_k) and max |c_k|,
//   spread tile by tile in LDS (integers), x and y FFT passes, the z pass
//   forward, times the fixed spectrum and back in one kernel, the inverse y
//   pass, and the inverse x pass with the peak of its rows (planar grids: x,
//   then y with the product, then x).
// The FP64 search, full score volumes and the windowless reference run here;
// it is also what the fused FP32 kernels are compared with.

#include "common.hpp"
#include "fft.hpp"
#include "fft256.hpp"
#include "launch.hpp"
#include "tile_spread.hpp"
#include "twiddles.hpp"

namespace sdf {

namespace {

// ------------------------------------------------------------------ rotations
template <typename T>
__global__ void quat_to_rot_kernel(const double* __restrict__ quats, int64_t n, double* __restrict__ r64,
                                   T* __restrict__ rT, unsigned long long* __restrict__ cmax) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (cmax && i == 0) *cmax = 0;  // for coef_max_kernel
    if (i >= n) return;
    double w = quats[4 * i], x = quats[4 * i + 1], y = quats[4 * i + 2], z = quats[4 * i + 3];
    double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
    w *= inv;
    x *= inv;
    y *= inv;
    z *= inv;
    double r[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - w * z),     2 * (x * z + w * y),
                   2 * (x * y + w * z),     1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                   2 * (x * z - w * y),     2 * (y * z + w * x),     1 - 2 * (x * x + y * y)};
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        if (r64) r64[9 * i + a] = r[a];
        if (rT) rT[9 * i + a] = T(r[a]);
    }
}

template <typename T>
__global__ void coef_kernel(const cplx<T>* __restrict__ rho, const T* __restrict__ w, int64_t n,
                            cplx<T>* __restrict__ c) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) c[i] = rho[i] * w[i];
}

// the same, and the largest |Re c| or |Im c| as the bits of a non-negative double
// (which order like integers; infinities and NaN above every number)
template <typename T>
__global__ __launch_bounds__(256) void coef_max_kernel(const cplx<T>* __restrict__ rho, const T* __restrict__ w,
                                                       int64_t n, cplx<T>* __restrict__ c,
                                                       unsigned long long* __restrict__ cmax) {
    __shared__ unsigned long long wave_max[4];
    unsigned long long m = 0;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const cplx<T> v = rho[i] * w[i];
        c[i] = v;
        const unsigned long long a = __double_as_longlong(fabs(double(v.re))),
                                 b = __double_as_longlong(fabs(double(v.im)));
        m = max(m, max(a, b));
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned long long)__shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(cmax, max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3])));
}

template <typename T>
__global__ void zero_kernel(cplx<T>* __restrict__ p, int64_t n) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (; i < n; i += stride) p[i] = mk(T(0), T(0));
}

// ------------------------------------------------------------------ spread
// One thread per body sample: y = sign * R (k - n_m/2), 4^3 (planar: 4^2)
// B-spline stencil, periodic, accumulated with global atomics.
template <typename T>
__global__ void spread_atomic_kernel(const cplx<T>* __restrict__ c, int n_m, int planar, const T* __restrict__ R,
                                     T sign, int N, cplx<T>* __restrict__ out) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const cplx<T> ck = c[k];
    if (ck.re == T(0) && ck.im == T(0)) return;
    const int rot = blockIdx.y;
    const T* r = R + 9 * rot;
    const T half = T(0.5) * T(n_m);
    const T bx = T(int(k % n_m)) - half;
    const T by = T(int((k / n_m) % n_m)) - half;
    const T bz = planar ? T(0) : T(int(k / (int64_t(n_m) * n_m))) - half;
    const T yx = sign * (r[0] * bx + r[1] * by + r[2] * bz);
    const T yy = sign * (r[3] * bx + r[4] * by + r[5] * bz);
    const T yz = sign * (r[6] * bx + r[7] * by + r[8] * bz);
    const T fx0 = dev_floor(yx), fy0 = dev_floor(yy);
    T wx[4], wy[4], wz[4];
    bspline3_weights(yx - fx0, wx);
    bspline3_weights(yy - fy0, wy);
    const int ix = int(fx0) - 1, iy = int(fy0) - 1;
    const int64_t gsz = planar ? int64_t(N) * N : int64_t(N) * N * N;
    cplx<T>* g = out + rot * gsz;
    if (planar) {
        for (int b = 0; b < 4; ++b) {
            const int yy_i = wrap(iy + b, N);
            for (int a = 0; a < 4; ++a) {
                const int xx_i = wrap(ix + a, N);
                const T wt = wx[a] * wy[b];
                cplx<T>* p = g + int64_t(yy_i) * N + xx_i;
                atomicAdd(&p->re, ck.re * wt);
                atomicAdd(&p->im, ck.im * wt);
            }
        }
        return;
    }
    const T fz0 = dev_floor(yz);
    bspline3_weights(yz - fz0, wz);
    const int iz = int(fz0) - 1;
    for (int cz = 0; cz < 4; ++cz) {
        const int zz_i = wrap(iz + cz, N);
        for (int b = 0; b < 4; ++b) {
            const int yy_i = wrap(iy + b, N);
            const T wyz = wy[b] * wz[cz];
            for (int a = 0; a < 4; ++a) {
                const int xx_i = wrap(ix + a, N);
                const T wt = wx[a] * wyz;
                cplx<T>* p = g + (int64_t(zz_i) * N + yy_i) * N + xx_i;
                atomicAdd(&p->re, ck.re * wt);
                atomicAdd(&p->im, ck.im * wt);
            }
        }
    }
}

// ------------------------------------------------------------------ tile spread
// The search's spread: a block owns a tile of grid nodes of one rotation and
// gathers every body sample whose stencil reaches it, so each node is stored
// once, with no zero pass and no global atomics (FP64 global atomics took four
// fifths of the FP64 search: 17 million adds per rotation at 64^3 samples).
// The samples that reach the tile come wave by wave with full lanes
// (box_samples): each lane forms its sample's weights and adds the taps that
// lie in the tile to LDS.
// Sums are 64-bit integers in both precisions (their order does not matter, runs
// repeat bit for bit), in units of at most 2^-61 max|c|: finer than the rounding
// of an FP64 sum at nodes of 1/500 of the largest value and more, and of an FP32
// sum at any node that a coefficient of 2^-37 of the largest reaches (32-bit sums
// in units of 16 max|c| / 2^31 lost two digits on fields with one coefficient a
// hundred times the rest).  The B-splines of a whole lattice of unit density sum
// to at most 1.01 at any point, those of a part of it to less, so no sum reaches
// 2^63.  Nodes are centred coordinates [-N/2, N/2): the fit rule keeps every
// stencil inside, so no index wraps before the store.
// Bound by VALU issue (6 instructions per sum besides its LDS add).  FP64, 8
// rotations of 96^3 / 48^3: the whole search 6212 -> 461 us, 217 of them here;
// 36 rotations of 128^2 / 64^2: 1930 -> 65 us (with the batched and fused
// transform passes).
constexpr double kTileTop = 4611686018427387904.0;  // 2^62: |c| in units

// The r-th tile from the middle of the grid outwards.  The body's tiles take
// nearly all of the time; launched first, over all rotations, they spread over
// the CUs evenly and none is left for the end (FP64, 96^3, 8 rotations of a 48^3
// body: 420 us for the search in row order, 413 so, repeated on the same buffers;
// 12 of 128^3: 1300 and 1215).
// 3D tiles are half as thick as wide, and
// shell k of the nested boxes of 2k x 2k x 4k tiles holds its two lowest and two
// highest layers, then the rings of the layers between; grids of less than two
// tiles across are taken in order.
template <bool PLANAR>
__device__ __forceinline__ void tile_outwards(int r, int nx, int ny, int t[3]) {
    if (PLANAR) {
        auto from_middle = [](int i, int n) { return n / 2 + ((i & 1) ? -((i + 1) / 2) : i / 2); };
        t[0] = from_middle(r % nx, nx);
        t[1] = from_middle(r / nx, ny);
        t[2] = 0;
        return;
    }
    if (nx < 2) {
        t[0] = t[1] = 0;
        t[2] = r;
        return;
    }
    int k = 1;
    while (16 * k * k * k <= r) ++k;
    const int s = 2 * k, area = s * s, ring = 4 * s - 4;
    int q = r - 16 * (k - 1) * (k - 1) * (k - 1);
    if (q < 4 * area) {
        const int layer = q / area;
        q %= area;
        t[0] = q % s;
        t[1] = q / s;
        t[2] = layer < 2 ? layer : 2 * s - 4 + layer;
    } else {
        q -= 4 * area;
        t[2] = 2 + q / ring;
        q %= ring;
        t[0] = q < 2 * s ? q % s : ((q & 1) ? s - 1 : 0);
        t[1] = q < 2 * s ? (q < s ? 0 : s - 1) : 1 + (q - 2 * s) / 2;
    }
    t[0] += nx / 2 - k;
    t[1] += ny / 2 - k;
    t[2] += nx - s;
}

template <typename T, bool PLANAR, int BLOCK>
__global__ __launch_bounds__(BLOCK) void spread_tile_kernel(const cplx<T>* __restrict__ c, int n_m,
                                                                 const T* __restrict__ R, T sign, int N,
                                                                 const unsigned long long* __restrict__ cmax,
                                                                 cplx<T>* __restrict__ out) {
    using S = SpreadTile<PLANAR>;
    __shared__ unsigned long long acc[S::WORDS];
    const int sx = min(S::X, N), sy = min(S::Y, N), sz = PLANAR ? 1 : min(S::Z, N);
    const int ntx = N / sx, nty = N / sy;
    int tile[3];
    tile_outwards<PLANAR>(int(blockIdx.y), ntx, nty, tile);
    const int t0[3] = {tile[0] * sx - N / 2, tile[1] * sy - N / 2, PLANAR ? 0 : tile[2] * sz - N / 2};
    const int dim[3] = {sx, sy, sz};
    const int64_t G = PLANAR ? int64_t(N) * N : int64_t(N) * N * N;
    cplx<T>* g = out + int64_t(blockIdx.x) * G;
    const T* r = R + 9 * int64_t(blockIdx.x);
    const double cm = __longlong_as_double((long long)*cmax);
    const bool finite = cm < INFINITY;
    const double pow2 = pow2_below(fmin(kTileTop / cm, 1e300));
    const double scale = cm > 0.0 && finite ? pow2 : 0.0, inv = cm > 0.0 ? 1.0 / pow2 : 0.0;
    for (int i = int(threadIdx.x); i < S::WORDS; i += BLOCK) acc[i] = 0;
    __syncthreads();
    const T half_box = T(0.5) * T(n_m);
    const Fixed64 fixed;
    float rf[9], lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 9; ++a) rf[a] = float(sign * r[a]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = float(t0[a] - 2);
        hi[a] = float(t0[a] + dim[a] + 1);
    }
    box_samples<PLANAR>(rf, n_m, lo, hi, uniform(int(threadIdx.x) >> 6), BLOCK / 64, [&](int i, int j, int k) {
        const cplx<T> v = c[(k * n_m + j) * n_m + i];
        const double v_re = double(v.re) * scale, v_im = double(v.im) * scale;
        const T bx = T(i) - half_box, by = T(j) - half_box, bz = PLANAR ? T(0) : T(k) - half_box;
        T wt[3][4];
        int b[3];
#pragma unroll
        for (int a = 0; a < (PLANAR ? 2 : 3); ++a) {
            const T y = sign * (r[3 * a] * bx + r[3 * a + 1] * by + r[3 * a + 2] * bz);
            const T fl = dev_floor(y);
            b[a] = int(fl) - 1 - t0[a];
            bspline3_weights(y - fl, wt[a]);
        }
#pragma unroll
        for (int cz = 0; cz < (PLANAR ? 1 : 4); ++cz) {
            const int iz = PLANAR ? 0 : b[2] + cz;
            if (unsigned(iz) >= unsigned(sz)) continue;
#pragma unroll
            for (int cy = 0; cy < 4; ++cy) {
                const int iy = b[1] + cy;
                if (unsigned(iy) >= unsigned(sy)) continue;
                const double wyz = PLANAR ? double(wt[1][cy]) : double(wt[1][cy] * wt[2][cz]);
                const double row_re = v_re * wyz, row_im = v_im * wyz;
                unsigned long long* row = acc + (iz * S::Y + iy) * S::PITCH;
#pragma unroll
                for (int cx = 0; cx < 4; ++cx) {
                    const int ix = b[0] + cx;
                    if (unsigned(ix) >= unsigned(sx)) continue;
                    atomicAdd(row + ix, fixed(row_re * double(wt[0][cx])));
                    atomicAdd(row + S::IMAG + ix, fixed(row_im * double(wt[0][cx])));
                }
            }
        }
    });
    __syncthreads();
    for (int i = int(threadIdx.x); i < sx * sy * sz; i += BLOCK) {
        const int ix = i % sx, iy = (i / sx) % sy, iz = i / (sx * sy);
        const unsigned long long* a = acc + (iz * S::Y + iy) * S::PITCH + ix;
        const int ux = (t0[0] + ix + N) % N, uy = (t0[1] + iy + N) % N, uz = PLANAR ? 0 : (t0[2] + iz + N) % N;
        cplx<T> v = mk(T(double((long long)a[0]) * inv), T(double((long long)a[S::IMAG]) * inv));
        // a transform of any value that is not finite is NaN everywhere
        if (!finite) v = mk(T(NAN), T(NAN));
        g[(int64_t(uz) * N + uy) * N + ux] = v;
    }
}

// ------------------------------------------------------------------ direct reference
// Boundary samples of the moving part turned about its body-box centre c:
// q' = c + R (q - c), n' = R n (FP64, R row-major).
__global__ void rotate_samples_kernel(const double* __restrict__ q, const double* __restrict__ nrm, int64_t ns,
                                      const double* __restrict__ R, double cx, double cy, double cz,
                                      double* __restrict__ qo, double* __restrict__ no) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= ns) return;
    const double d[3] = {q[3 * j] - cx, q[3 * j + 1] - cy, q[3 * j + 2] - cz};
    const double c[3] = {cx, cy, cz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        qo[3 * j + a] = c[a] + R[3 * a] * d[0] + R[3 * a + 1] * d[1] + R[3 * a + 2] * d[2];
        no[3 * j + a] = R[3 * a] * nrm[3 * j] + R[3 * a + 1] * nrm[3 * j + 1] + R[3 * a + 2] * nrm[3 * j + 2];
    }
}

// Body-box values placed on the fixed grid without a window, reflected as
// the spread with sign -1 places them: node k (body position k - n_m / 2,
// n_m even) goes to u = -(k - n_m / 2) mod N.  Distinct nodes land on
// distinct grid nodes (n_m <= N), so plain stores suffice.
template <typename T>
__global__ void place_direct_kernel(const cplx<T>* __restrict__ rho, int n_m, int planar, T w_node, int N,
                                    cplx<T>* __restrict__ out) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const int h = n_m / 2;
    const int kx = int(k % n_m), ky = int((k / n_m) % n_m), kz = planar ? h : int(k / (int64_t(n_m) * n_m));
    const int ux = wrap(h - kx, N), uy = wrap(h - ky, N), uz = planar ? 0 : wrap(h - kz, N);
    out[(int64_t(uz) * N + uy) * N + ux] = rho[k] * w_node;
}

// ------------------------------------------------------------------ FFT passes

constexpr int kFftBlock = 256;

// Rows (x axis, contiguous): a block transforms conc = 256 / (N/8) rows.
template <typename T, int N, int S>
__global__ __launch_bounds__(kFftBlock) void fft_rows_kernel(cplx<T>* __restrict__ data, int64_t nrows, T scale) {
    constexpr int TPL = FFTShape<N>::TPL;
    constexpr int CONC = kFftBlock / TPL;
    __shared__ cplx<T> buf[CONC * N];
    __shared__ cplx<T> tw[N];
    table_twiddles<T, N>(tw);
    const int64_t row0 = int64_t(blockIdx.x) * CONC;
    const int nr = int(nrows - row0 < CONC ? nrows - row0 : CONC);
    cplx<T>* src = data + row0 * N;
    for (int i = threadIdx.x; i < nr * N; i += kFftBlock) buf[i] = src[i];
    __syncthreads();
    lds_fft_lines<T, N, S, false>(buf, 1, N, nr, tw);
    for (int i = threadIdx.x; i < nr * N; i += kFftBlock) src[i] = buf[i] * scale;
}

// Columns per block for the strided passes: the largest power of two that
// fits the block's lines and divides N.
template <int N>
constexpr int cols_width() {
    int w = 1;
    while (w * 2 <= kFftBlock / FFTShape<N>::TPL && N % (w * 2) == 0) w *= 2;
    return w;
}

// Strided axis (y: es = N, z: es = N^2): a block takes W consecutive x
// columns of one (other-axis) plane and transforms them along the axis.
template <typename T, int N, int S>
__global__ __launch_bounds__(kFftBlock) void fft_cols_kernel(cplx<T>* __restrict__ data, int64_t es, int64_t os,
                                                             int64_t gsz, T scale) {
    constexpr int W = cols_width<N>();
    __shared__ cplx<T> buf[N * W];
    __shared__ cplx<T> tw[N];
    table_twiddles<T, N>(tw);
    const int x0 = blockIdx.x * W;
    const int o = blockIdx.y;
    cplx<T>* base = data + int64_t(blockIdx.z) * gsz + int64_t(o) * os + x0;
    for (int i = threadIdx.x; i < N * W; i += kFftBlock) {
        const int e = i / W, xl = i % W;
        buf[i] = base[e * es + xl];
    }
    __syncthreads();
    lds_fft_lines<T, N, S, true>(buf, W, 1, W, tw);
    for (int i = threadIdx.x; i < N * W; i += kFftBlock) {
        const int e = i / W, xl = i % W;
        base[e * es + xl] = buf[i] * scale;
    }
}

// The last forward axis, the product with the fixed spectrum and the first
// inverse axis in one pass over the grid: W columns forward, times S, back.
template <typename T, int N>
__global__ __launch_bounds__(kFftBlock) void fft_cols_mul_kernel(cplx<T>* __restrict__ data, int64_t es, int64_t os,
                                                                 int64_t gsz, const cplx<T>* __restrict__ spec) {
    constexpr int W = cols_width<N>();
    __shared__ cplx<T> buf[N * W];
    __shared__ cplx<T> tw[N];
    table_twiddles<T, N>(tw);
    const int64_t off = int64_t(blockIdx.y) * os + int64_t(blockIdx.x) * W;
    cplx<T>* base = data + int64_t(blockIdx.z) * gsz + off;
    const cplx<T>* sb = spec + off;
    for (int i = threadIdx.x; i < N * W; i += kFftBlock) buf[i] = base[(i / W) * es + i % W];
    __syncthreads();
    lds_fft_lines<T, N, -1, true>(buf, W, 1, W, tw);
    for (int i = threadIdx.x; i < N * W; i += kFftBlock) buf[i] = buf[i] * sb[(i / W) * es + i % W];
    __syncthreads();
    lds_fft_lines<T, N, 1, true>(buf, W, 1, W, tw);
    for (int i = threadIdx.x; i < N * W; i += kFftBlock) base[(i / W) * es + i % W] = buf[i];
}

// Peaks kept by the inverse x pass: rows of a rotation store their real parts
// compactly at their own start (row r at reals 2 N r), and the first row of a
// block its best (value, flat index) in the free half behind.
template <typename T>
struct RowPeak {
    T v;
    int i;
};
template <typename T>
__device__ __forceinline__ RowPeak<T>* row_peak(T* rot, int N, int64_t row) {
    return reinterpret_cast<RowPeak<T>*>(rot + (2 * row + 1) * N);
}

// Inverse x pass of blockIdx.y's grid, real parts only: to vol (a volume per
// rotation), or (vol null) in place with the block's best value.
template <typename T, int N>
__global__ __launch_bounds__(kFftBlock) void fft_rows_real_kernel(cplx<T>* __restrict__ data, int nrows,
                                                                  T* __restrict__ vol) {
    constexpr int TPL = FFTShape<N>::TPL;
    constexpr int CONC = kFftBlock / TPL;
    __shared__ cplx<T> buf[CONC * N];
    __shared__ cplx<T> tw[N];
    __shared__ RowPeak<T> best[kFftBlock / 64];
    table_twiddles<T, N>(tw);
    const int row0 = int(blockIdx.x) * CONC;
    const int nr = min(CONC, nrows - row0);
    cplx<T>* rot = data + int64_t(blockIdx.y) * nrows * N;
    cplx<T>* src = rot + int64_t(row0) * N;
    for (int i = threadIdx.x; i < nr * N; i += kFftBlock) buf[i] = src[i];
    __syncthreads();
    lds_fft_lines<T, N, 1, false>(buf, 1, N, nr, tw);
    if (vol) {
        T* dst = vol + (int64_t(blockIdx.y) * nrows + row0) * N;
        for (int i = threadIdx.x; i < nr * N; i += kFftBlock) dst[i] = buf[i].re;
        return;
    }
    T* real = reinterpret_cast<T*>(rot);
    T bv = T(-INFINITY);
    int bi = 0x7fffffff;
    for (int i = threadIdx.x; i < nr * N; i += kFftBlock) {
        const T v = buf[i].re;
        real[(2 * int64_t(row0 + i / N)) * N + i % N] = v;
        if (v > bv) {  // i grows: the lowest index keeps a tie
            bv = v;
            bi = row0 * N + i;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const T ov = __shfl_xor(bv, off);
        const int oi = __shfl_xor(bi, off);
        if (ov > bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
        }
    }
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = RowPeak<T>{bv, bi};
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kFftBlock / 64; ++w)
            if (best[w].v > bv || (best[w].v == bv && best[w].i < bi)) {
                bv = best[w].v;
                bi = best[w].i;
            }
        *row_peak(real, N, row0) = RowPeak<T>{bv, bi};
    }
}

template <typename T, int N>
hipError_t fft3_impl(void* data, bool planar, int batch, int dir, double scale, hipStream_t s) {
    constexpr int TPL = FFTShape<N>::TPL;
    constexpr int CONC = kFftBlock / TPL;
    constexpr int W = cols_width<N>();
    cplx<T>* d = static_cast<cplx<T>*>(data);
    const int nz = planar ? 1 : N;
    const int64_t gsz = int64_t(N) * N * nz;
    const int64_t nrows = int64_t(N) * nz * batch;
    const T one = T(1), sc = T(scale);
    // x
    {
        dim3 grid(unsigned((nrows + CONC - 1) / CONC));
        if (dir < 0)
            hipLaunchKernelGGL((fft_rows_kernel<T, N, -1>), grid, dim3(kFftBlock), 0, s, d, nrows, one);
        else
            hipLaunchKernelGGL((fft_rows_kernel<T, N, 1>), grid, dim3(kFftBlock), 0, s, d, nrows, one);
    }
    // y: columns of each z plane
    {
        dim3 grid(N / W, nz, batch);
        const T scy = planar ? sc : one;
        if (dir < 0)
            hipLaunchKernelGGL((fft_cols_kernel<T, N, -1>), grid, dim3(kFftBlock), 0, s, d, int64_t(N),
                               int64_t(N) * N, gsz, scy);
        else
            hipLaunchKernelGGL((fft_cols_kernel<T, N, 1>), grid, dim3(kFftBlock), 0, s, d, int64_t(N),
                               int64_t(N) * N, gsz, scy);
    }
    // z: columns of each y row
    if (!planar) {
        dim3 grid(N / W, N, batch);
        if (dir < 0)
            hipLaunchKernelGGL((fft_cols_kernel<T, N, -1>), grid, dim3(kFftBlock), 0, s, d, int64_t(N) * N,
                               int64_t(N), gsz, sc);
        else
            hipLaunchKernelGGL((fft_cols_kernel<T, N, 1>), grid, dim3(kFftBlock), 0, s, d, int64_t(N) * N,
                               int64_t(N), gsz, sc);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ peak
constexpr int kPeakBlock = 256;

template <typename T>
__device__ __forceinline__ bool better(T v, int i, T bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

template <typename T>
__device__ __forceinline__ void block_argmax(T& v, int& idx) {
    __shared__ T sv[kPeakBlock];
    __shared__ int si[kPeakBlock];
    sv[threadIdx.x] = v;
    si[threadIdx.x] = idx;
    __syncthreads();
    for (int off = int(blockDim.x) / 2; off > 0; off >>= 1) {
        if (int(threadIdx.x) < off) {
            T ov = sv[threadIdx.x + off];
            int oi = si[threadIdx.x + off];
            if (better(ov, oi, sv[threadIdx.x], si[threadIdx.x])) {
                sv[threadIdx.x] = ov;
                si[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    v = sv[0];
    idx = si[0];
    __syncthreads();
}

// layouts of a volume: complex, or the inverse x pass's compact real rows
enum { kVolCplx, kVolRows };
template <typename T, int KIND>
__device__ __forceinline__ T vol_at(const void* vol, int64_t i, int N) {
    if (KIND == kVolCplx) return static_cast<const cplx<T>*>(vol)[i].re;
    return static_cast<const T*>(vol)[(i / N) * (2 * N) + i % N];
}

template <typename T>
__global__ __launch_bounds__(kPeakBlock) void peak_partial_kernel(const void* __restrict__ vol, int64_t nvox,
                                                                  int nparts, T* __restrict__ pval,
                                                                  int* __restrict__ pidx) {
    const int part = blockIdx.x, b = blockIdx.y;
    const int64_t chunk = (nvox + nparts - 1) / nparts;
    const int64_t lo = part * chunk;
    const int64_t hi = lo + chunk < nvox ? lo + chunk : nvox;
    const int64_t off = int64_t(b) * nvox;
    T bv = T(-INFINITY);
    int bi = 0x7fffffff;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kPeakBlock) {
        T v = vol_at<T, kVolCplx>(vol, off + i, 1);
        if (better(v, int(i), bv, bi)) {
            bv = v;
            bi = int(i);
        }
    }
    block_argmax(bv, bi);
    if (threadIdx.x == 0) {
        pval[int64_t(b) * nparts + part] = bv;
        pidx[int64_t(b) * nparts + part] = bi;
    }
}

// part_rows (kVolRows): rows per partial of the inverse x pass
template <typename T, int KIND>
__global__ __launch_bounds__(kPeakBlock) void peak_final_kernel(const void* __restrict__ vol, int N, int planar,
                                                                int nparts, int part_rows,
                                                                const T* __restrict__ pval,
                                                                const int* __restrict__ pidx, T* __restrict__ score,
                                                                int32_t* __restrict__ tout, T* __restrict__ nbhd,
                                                                double* __restrict__ refined) {
    const int b = blockIdx.x;
    const int nz = planar ? 1 : N;
    const int64_t nvox = int64_t(N) * N * nz;
    T bv = T(-INFINITY);
    int bi = 0x7fffffff;
    for (int i = threadIdx.x; i < nparts; i += kPeakBlock) {
        T v;
        int id;
        if constexpr (KIND == kVolRows) {
            T* rot = const_cast<T*>(static_cast<const T*>(vol)) + int64_t(b) * 2 * nvox;
            const RowPeak<T> p = *row_peak(rot, N, int64_t(i) * part_rows);
            v = p.v;
            id = p.i;
        } else {
            v = pval[int64_t(b) * nparts + i];
            id = pidx[int64_t(b) * nparts + i];
        }
        if (better(v, id, bv, bi)) {
            bv = v;
            bi = id;
        }
    }
    block_argmax(bv, bi);
    __shared__ T nb[27];
    const int tx = bi % N, ty = (bi / N) % N, tz = bi / (N * N);
    if (threadIdx.x < 27) {
        const int dz = threadIdx.x / 9 - 1, dy = (threadIdx.x / 3) % 3 - 1, dx = threadIdx.x % 3 - 1;
        const int zz = wrap(tz + dz, nz), yy = wrap(ty + dy, N), xx = wrap(tx + dx, N);
        nb[threadIdx.x] = vol_at<T, KIND>(vol, int64_t(b) * nvox + (int64_t(zz) * N + yy) * N + xx, N);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        score[b] = bv;
        tout[3 * b] = tx;
        tout[3 * b + 1] = ty;
        tout[3 * b + 2] = tz;
        if (nbhd)
            for (int a = 0; a < 27; ++a) nbhd[27 * int64_t(b) + a] = nb[a];
        if (refined) {
            // per-axis parabola through (f-, f0, f+), FP64
            const double f0 = double(nb[13]);
            const double fm[3] = {double(nb[12]), double(nb[10]), double(nb[4])};
            const double fp[3] = {double(nb[14]), double(nb[16]), double(nb[22])};
            const int ti[3] = {tx, ty, tz};
            for (int a = 0; a < 3; ++a) {
                const double den = fm[a] - 2.0 * f0 + fp[a];
                double d = 0.0;
                if (den < 0.0) {
                    d = (fm[a] - fp[a]) / (2.0 * den);
                    d = d < -0.5 ? -0.5 : (d > 0.5 ? 0.5 : d);
                }
                refined[3 * b + a] = double(ti[a]) + d;
            }
        }
    }
}

template <typename T>
__global__ void real_part_kernel(const cplx<T>* __restrict__ v, T* __restrict__ out, int64_t n) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (; i < n; i += stride) out[i] = v[i].re;
}

inline unsigned grid_for(int64_t n, int block, int cap = 65535 * 4) {
    int64_t g = (n + block - 1) / block;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    return unsigned(g);
}

}  // namespace

template <typename T>
hipError_t launch_quat_to_rot(const double* quats, int64_t n, double* r64, T* rT, hipStream_t s,
                              unsigned long long* cmax) {
    hipLaunchKernelGGL(quat_to_rot_kernel<T>, dim3(grid_for(n, 64)), dim3(64), 0, s, quats, n, r64, rT, cmax);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coef(const void* rho_m, const T* w_m, int64_t count, void* c_out, hipStream_t s) {
    hipLaunchKernelGGL(coef_kernel<T>, dim3(unsigned((count + 255) / 256)), dim3(256), 0, s,
                       static_cast<const cplx<T>*>(rho_m), w_m, count, static_cast<cplx<T>*>(c_out));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_zero(void* buf, int64_t count, hipStream_t s) {
    hipLaunchKernelGGL(zero_kernel<T>, dim3(grid_for(count, 256, 16384)), dim3(256), 0, s,
                       static_cast<cplx<T>*>(buf), count);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_spread_atomic(const void* c, int n_m, bool planar, const T* R, int n_rot, T sign, int N, void* out,
                                hipStream_t s) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    dim3 grid(unsigned((K + 255) / 256), unsigned(n_rot));
    hipLaunchKernelGGL(spread_atomic_kernel<T>, grid, dim3(256), 0, s, static_cast<const cplx<T>*>(c), n_m,
                       planar ? 1 : 0, R, sign, N, static_cast<cplx<T>*>(out));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_fft3(void* data, int N, bool planar, int batch, int dir, double scale, hipStream_t s) {
    switch (N) {
        case 8: return fft3_impl<T, 8>(data, planar, batch, dir, scale, s);
        case 16: return fft3_impl<T, 16>(data, planar, batch, dir, scale, s);
        case 32: return fft3_impl<T, 32>(data, planar, batch, dir, scale, s);
        case 64: return fft3_impl<T, 64>(data, planar, batch, dir, scale, s);
        case 96: return fft3_impl<T, 96>(data, planar, batch, dir, scale, s);
        case 128: return fft3_impl<T, 128>(data, planar, batch, dir, scale, s);
        case 256: return fft3_impl<T, 256>(data, planar, batch, dir, scale, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
int peak_parts(int N, bool planar) {
    const int64_t nvox = int64_t(N) * N * (planar ? 1 : N);
    int64_t p = (nvox + 4095) / 4096;
    if (p > 512) p = 512;
    if (p < 1) p = 1;
    return int(p);
}

template <typename T>
hipError_t launch_peak(const void* vol, int N, bool planar, int batch, T* part_val, int* part_idx, int nparts,
                       T* score, int32_t* t, T* nbhd, double* refined, hipStream_t s) {
    const int64_t nvox = int64_t(N) * N * (planar ? 1 : N);
    const dim3 g1{unsigned(nparts), unsigned(batch), 1u};
    hipLaunchKernelGGL(peak_partial_kernel<T>, g1, dim3(kPeakBlock), 0, s, vol, nvox, nparts, part_val, part_idx);
    hipLaunchKernelGGL((peak_final_kernel<T, kVolCplx>), dim3(unsigned(batch)), dim3(kPeakBlock), 0, s, vol, N,
                       planar ? 1 : 0, nparts, 0, part_val, part_idx, score, t, nbhd, refined);
    return hipGetLastError();
}

namespace {
template <typename T, int N>
hipError_t correlate_impl(void* data, const void* spec, bool planar, int batch, T* vol, T* score, int32_t* t, T* nbhd,
                          double* refined, hipStream_t s) {
    constexpr int CONC = kFftBlock / FFTShape<N>::TPL;
    constexpr int W = cols_width<N>();
    cplx<T>* d = static_cast<cplx<T>*>(data);
    const auto* sp = static_cast<const cplx<T>*>(spec);
    const int nz = planar ? 1 : N, rows = N * nz;
    const int64_t plane = int64_t(N) * N, gsz = plane * nz, all = int64_t(rows) * batch;
    hipLaunchKernelGGL((fft_rows_kernel<T, N, -1>), dim3(unsigned((all + CONC - 1) / CONC)), dim3(kFftBlock), 0, s, d,
                       all, T(1));
    if (planar) {
        hipLaunchKernelGGL((fft_cols_mul_kernel<T, N>), dim3(N / W, 1, batch), dim3(kFftBlock), 0, s, d, int64_t(N),
                           plane, gsz, sp);
    } else {
        const dim3 g(N / W, N, batch);
        hipLaunchKernelGGL((fft_cols_kernel<T, N, -1>), g, dim3(kFftBlock), 0, s, d, int64_t(N), plane, gsz, T(1));
        hipLaunchKernelGGL((fft_cols_mul_kernel<T, N>), g, dim3(kFftBlock), 0, s, d, plane, int64_t(N), gsz, sp);
        hipLaunchKernelGGL((fft_cols_kernel<T, N, 1>), g, dim3(kFftBlock), 0, s, d, int64_t(N), plane, gsz, T(1));
    }
    const int blocks = (rows + CONC - 1) / CONC;
    hipLaunchKernelGGL((fft_rows_real_kernel<T, N>), dim3(unsigned(blocks), unsigned(batch)), dim3(kFftBlock), 0, s, d,
                       rows, vol);
    if (!vol)
        hipLaunchKernelGGL((peak_final_kernel<T, kVolRows>), dim3(unsigned(batch)), dim3(kPeakBlock), 0, s, data, N,
                           planar ? 1 : 0, blocks, CONC, nullptr, nullptr, score, t, nbhd, refined);
    return hipGetLastError();
}
}  // namespace

template <typename T>
hipError_t launch_correlate(void* grid, const void* spec, int N, bool planar, int batch, T* vol, T* score, int32_t* t,
                            T* nbhd, double* refined, hipStream_t s) {
    switch (N) {
        case 8: return correlate_impl<T, 8>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        case 16: return correlate_impl<T, 16>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        case 32: return correlate_impl<T, 32>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        case 64: return correlate_impl<T, 64>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        case 96: return correlate_impl<T, 96>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        case 128: return correlate_impl<T, 128>(grid, spec, planar, batch, vol, score, t, nbhd, refined, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_spread_tiles(const void* c, int n_m, bool planar, const T* R, int n_rot, T sign, int N,
                               const unsigned long long* cmax, void* out, hipStream_t s) {
    const auto* cc = static_cast<const cplx<T>*>(c);
    auto* o = static_cast<cplx<T>*>(out);
    if (planar) {
        using S = SpreadTile<true>;
        const unsigned tx = unsigned(N / (S::X < N ? S::X : N)), ty = unsigned(N / (S::Y < N ? S::Y : N));
        hipLaunchKernelGGL((spread_tile_kernel<T, true, kTileBlock>), dim3(unsigned(n_rot), tx * ty), dim3(kTileBlock), 0, s, cc,
                           n_m, R, sign, N, cmax, o);
    } else {
        using S = SpreadTile<false>;
        const unsigned tx = unsigned(N / (S::X < N ? S::X : N)), ty = unsigned(N / (S::Y < N ? S::Y : N)),
                       tz = unsigned(N / (S::Z < N ? S::Z : N));
        // A call of few tiles ends with its slowest: eight waves a tile halve
        // that, where many tiles keep every CU busy with four (FP64, repeated: 413 /
        // 455 us for a search of 8 rotations at 96^3, 3456 tiles; 1214 / 1191 for 12 at
        // 128^3, 12288).
        const dim3 grid{unsigned(n_rot), tx * ty * tz, 1u};
        if (int64_t(n_rot) * tx * ty * tz <= 8192)
            hipLaunchKernelGGL((spread_tile_kernel<T, false, 2 * kTileBlock>), grid, dim3(2 * kTileBlock), 0, s, cc, n_m,
                               R, sign, N, cmax, o);
        else
            hipLaunchKernelGGL((spread_tile_kernel<T, false, kTileBlock>), grid, dim3(kTileBlock), 0, s, cc, n_m, R,
                               sign, N, cmax, o);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coef_max(const void* rho_m, const T* w_m, int64_t count, void* c_out, unsigned long long* cmax,
                           hipStream_t s) {
    // at most one block per CU: their maxima meet at one address
    hipLaunchKernelGGL(coef_max_kernel<T>, dim3(grid_for(count, 256, 256)), dim3(256), 0, s,
                       static_cast<const cplx<T>*>(rho_m), w_m, count, static_cast<cplx<T>*>(c_out), cmax);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_real_part(const void* vol, T* out, int64_t count, hipStream_t s) {
    hipLaunchKernelGGL(real_part_kernel<T>, dim3(grid_for(count, 256, 16384)), dim3(256), 0, s,
                       static_cast<const cplx<T>*>(vol), out, count);
    return hipGetLastError();
}

hipError_t launch_rotate_samples(const double* q, const double* nrm, int64_t ns, const double* R, const double c[3],
                                 double* qo, double* no, hipStream_t s) {
    hipLaunchKernelGGL(rotate_samples_kernel, dim3(unsigned((ns + 255) / 256)), dim3(256), 0, s, q, nrm, ns, R, c[0],
                       c[1], c[2], qo, no);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_place_direct(const void* rho, int n_m, bool planar, T w_node, int N, void* out, hipStream_t s) {
    const int64_t K = planar ? int64_t(n_m) * n_m : int64_t(n_m) * n_m * n_m;
    hipLaunchKernelGGL(place_direct_kernel<T>, dim3(unsigned((K + 255) / 256)), dim3(256), 0, s,
                       static_cast<const cplx<T>*>(rho), n_m, planar ? 1 : 0, w_node, N, static_cast<cplx<T>*>(out));
    return hipGetLastError();
}

#define SDF_INST(T)                                                                                              \
    template hipError_t launch_quat_to_rot<T>(const double*, int64_t, double*, T*, hipStream_t,                 \
                                              unsigned long long*);                                              \
    template hipError_t launch_coef<T>(const void*, const T*, int64_t, void*, hipStream_t);                      \
    template hipError_t launch_coef_max<T>(const void*, const T*, int64_t, void*, unsigned long long*,           \
                                           hipStream_t);                                                         \
    template hipError_t launch_zero<T>(void*, int64_t, hipStream_t);                                             \
    template hipError_t launch_place_direct<T>(const void*, int, bool, T, int, void*, hipStream_t);               \
    template hipError_t launch_spread_atomic<T>(const void*, int, bool, const T*, int, T, int, void*,           \
                                                hipStream_t);                                                    \
    template hipError_t launch_spread_tiles<T>(const void*, int, bool, const T*, int, T, int,                    \
                                               const unsigned long long*, void*, hipStream_t);                   \
    template hipError_t launch_correlate<T>(void*, const void*, int, bool, int, T*, T*, int32_t*, T*, double*,   \
                                            hipStream_t);                                                        \
    template hipError_t launch_fft3<T>(void*, int, bool, int, int, double, hipStream_t);                         \
    template int peak_parts<T>(int, bool);                                                                      \
    template hipError_t launch_peak<T>(const void*, int, bool, int, T*, int*, int, T*, int32_t*, T*, double*,   \
                                       hipStream_t);                                                             \
    template hipError_t launch_real_part<T>(const void*, T*, int64_t, hipStream_t);

SDF_INST(float)
SDF_INST(double)

}  // namespace sdf
