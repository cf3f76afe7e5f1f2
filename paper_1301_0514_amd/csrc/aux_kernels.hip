// aux_kernels.hip -- batched transposes, chirp tables, disk images and
// deterministic reductions for gfx950.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "aux_kernels.h"
#include "device_common.hpp"
#include "transpose_tile.hpp"

namespace scint {

// ---------------------------------------------------------------- transpose
// One 64 x 128 unit per workgroup of 256 threads (transpose_tile.hpp): grid
// x over units along the columns, y along the rows, z over the batch.
template <typename T>
__global__ __launch_bounds__(256) void transpose_pair_kernel(const T *__restrict__ in, T *__restrict__ out, int N) {
    __shared__ TransposeTile<T> tile;
    const int64_t base = (int64_t)blockIdx.z * N * N;
    transpose_unit<T, 256>(in + base, out + base, N, blockIdx.x, blockIdx.y, tile, threadIdx.x);
}

// complex128: one 16-byte element per lane, TILE x TILE tile.
template <typename T, int TILE>
__global__ __launch_bounds__(256) void transpose_kernel(const T *__restrict__ in, T *__restrict__ out, int N) {
    __shared__ T tile[TILE][TILE + 1];
    constexpr int ROWS = 256 / TILE;
    const int tx = threadIdx.x % TILE, ty = threadIdx.x / TILE;
    const int x0 = blockIdx.x * TILE, y0 = blockIdx.y * TILE;
    const int64_t base = (int64_t)blockIdx.z * N * N;
    const T *src = in + base;
    T *dst = out + base;
    // unguarded loads at clamped addresses (all in flight at once); the slots
    // filled for positions outside the matrix are never read
    T v[TILE / ROWS];
    const int xc = min(x0 + tx, N - 1);
#pragma unroll
    for (int k = 0; k < TILE / ROWS; ++k) v[k] = src[(int64_t)min(y0 + ty + k * ROWS, N - 1) * N + xc];
#pragma unroll
    for (int k = 0; k < TILE / ROWS; ++k) tile[ty + k * ROWS][tx] = v[k];
    __syncthreads();
#pragma unroll
    for (int r = ty; r < TILE; r += ROWS) {
        const int x = x0 + r, y = y0 + tx;
        if (x < N && y < N) dst[(int64_t)x * N + y] = tile[tx][r];
    }
}

struct alignas(8) Elem8 {
    float a, b;
};
struct alignas(16) Elem16 {
    double a, b;
};

hipError_t launch_transpose(const void *in, void *out, int N, int64_t nbatch, int elem_bytes,
                            hipStream_t stream) {
    if (N % 2 != 0) return hipErrorInvalidValue;
    for (int64_t b0 = 0; b0 < nbatch; b0 += 65535) {
        const int nb = (int)((nbatch - b0) < 65535 ? (nbatch - b0) : 65535);
        const int64_t off = b0 * (int64_t)N * N;
        const dim3 grid64(transpose_units_x(N), transpose_units_y(N), nb);
        if (elem_bytes == 4) {
            hipLaunchKernelGGL((transpose_pair_kernel<float>), grid64, dim3(256), 0, stream,
                               static_cast<const float *>(in) + off, static_cast<float *>(out) + off, N);
        } else if (elem_bytes == 8) {
            hipLaunchKernelGGL((transpose_pair_kernel<Elem8>), grid64, dim3(256), 0, stream,
                               static_cast<const Elem8 *>(in) + off, static_cast<Elem8 *>(out) + off, N);
        } else if (elem_bytes == 16) {
            constexpr int TILE = 32;
            dim3 grid((N + TILE - 1) / TILE, (N + TILE - 1) / TILE, nb);
            hipLaunchKernelGGL((transpose_kernel<Elem16, TILE>), grid, dim3(256), 0, stream,
                               static_cast<const Elem16 *>(in) + off, static_cast<Elem16 *>(out) + off, N);
        } else {
            return hipErrorInvalidValue;
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

__global__ __launch_bounds__(256) void transpose_units_kernel(const Elem8 *__restrict__ in, Elem8 *__restrict__ out, int N,
                                                              int64_t u0) {
    __shared__ TransposeTile<Elem8> tile;
    const int nx = transpose_units_x(N), ny = transpose_units_y(N);
    const int64_t u = u0 + blockIdx.x, z = u / ((int64_t)nx * ny);
    const int rem = (int)(u - z * ((int64_t)nx * ny)), uy = rem / nx, ux = rem - uy * nx;
    const int64_t base = z * (int64_t)N * N;
    transpose_unit<Elem8, 256>(in + base, out + base, N, ux, uy, tile, threadIdx.x);
}

hipError_t launch_transpose_units(const void *in, void *out, int N, int64_t u0, int64_t u1, hipStream_t stream) {
    if (N % 2 != 0 || u0 < 0 || u1 <= u0 || u1 - u0 > (1ll << 31) - 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(transpose_units_kernel, dim3((unsigned)(u1 - u0)), dim3(256), 0, stream,
                       static_cast<const Elem8 *>(in), static_cast<Elem8 *>(out), N, u0);
    return hipGetLastError();
}

// ---------------------------------------------------------------- low modes
struct LowModeArgs {
    int N, K;
    uint32_t r0, seed_lo, seed_hi;
    double amp0, neg_beta_4;
    int swap;  // the coefficients' kx' and ky' change places
    // chirp table built by the launch's last workgroups (chirp_value), or NULL
    cpx<float> *tab;
    double chirp_a, chirp_scale;
    int blocks;  // workgroups of the low modes, all screens
};

// scale exp(-2 pi i a k'^2), the turns formed and reduced in FP64
template <typename Real> __device__ __forceinline__ cpx<Real> chirp_value(int k, int N, double a, double scale) {
    const double kk = (double)(k < N / 2 ? k : k - N);
    const double turns = a * (kk * kk);
    double s, c;
    sincospi(2.0 * (turns - rint(turns)), &s, &c);
    return {(Real)(scale * c), (Real)(-scale * s)};
}

// G[b][y][k], k <= K <= 16: a workgroup takes kLowRows rows y, each thread one
// k of kLowPer of them; the coefficients and the factors exp(2 pi i ky' y / N)
// (argument reduced exactly in integers) come from LDS, each coefficient once
// for the thread's rows, and the thread sums B(k) and B(-k) of every row in a
// fixed order.  Bound by those LDS reads and their latency (a workgroup of 17
// threads per row, with the coefficients from memory, took 77 us for
// 16 x 2048 rows).  Every workgroup draws the (2K + 1)^2 coefficients itself,
// four or five per thread, and the call's chirp table is built by further
// workgroups of the launch: one launch instead of three (one FP32 256^2 screen
// + pattern 31.9 -> 28.4 us).  NT 1024 (one row per
// thread) where the grids have few rows, so that the drawing, one coefficient
// after the other, does not make the call wait; 256 and four rows else.
constexpr int kLowRows = 60, kLowW = 33;

template <int NT>
__global__ __launch_bounds__(NT) void low_modes_kernel(double2 *__restrict__ G, LowModeArgs a) {
    constexpr int kLowGroups = NT / (kLowW / 2 + 1), kLowPer = kLowRows / kLowGroups;
    static_assert(kLowGroups * kLowPer == kLowRows, "rows of a workgroup");
    __shared__ double2 c[kLowW * kLowW];
    __shared__ double2 e[kLowRows][kLowW];
    const int t = threadIdx.x;
    if ((int)blockIdx.x >= a.blocks) {
        const int k = ((int)blockIdx.x - a.blocks) * NT + t;
        if (k < a.N) a.tab[k] = chirp_value<float>(k, a.N, a.chirp_a, a.chirp_scale);
        return;
    }
    const int W = 2 * a.K + 1, K1 = a.K + 1;
    const int per = (a.N + kLowRows - 1) / kLowRows, b = (int)blockIdx.x / per, y0 = ((int)blockIdx.x - b * per) * kLowRows;
    for (int i = t; i < W * W; i += NT) {
        const int p = i / W, q = i - p * W;
        const int fx = (a.swap ? q : p) - a.K, fy = (a.swap ? p : q) - a.K;
        c[i] = spectrum_coeff_f64(fx < 0 ? fx + a.N : fx, fy < 0 ? fy + a.N : fy, a.N, a.r0 + (uint32_t)b, a.seed_lo,
                                  a.seed_hi, a.amp0, a.neg_beta_4);
    }
    for (int i = t; i < kLowRows * W; i += NT) {
        const int r = i / W, k = i - r * W;
        int m = (k - a.K) * (y0 + r) % a.N;  // (|k - K| <= 16: the product fits)
        if (m < 0) m += a.N;
        double sn, cs;
        sincospi(2.0 * (double)m / (double)a.N, &sn, &cs);
        e[r][k] = make_double2(cs, sn);
    }
    __syncthreads();
    const int g = t / K1, k = t - g * K1;
    if (g >= kLowGroups) return;
    const double2 *up = c + (a.K + k) * W, *down = c + (a.K - k) * W;  // rows kx' = k and -k
    double2 bp[kLowPer], bm[kLowPer];
#pragma unroll
    for (int q = 0; q < kLowPer; ++q) bp[q] = bm[q] = make_double2(0.0, 0.0);
    for (int j = 0; j < W; ++j) {
        const double2 u = up[j], v = down[j];
#pragma unroll
        for (int q = 0; q < kLowPer; ++q) {
            const double2 w = e[g * kLowPer + q][j];
            bp[q].x = fma(u.x, w.x, fma(-u.y, w.y, bp[q].x));
            bp[q].y = fma(u.x, w.y, fma(u.y, w.x, bp[q].y));
            bm[q].x = fma(v.x, w.x, fma(-v.y, w.y, bm[q].x));
            bm[q].y = fma(v.x, w.y, fma(v.y, w.x, bm[q].y));
        }
    }
    constexpr double kSqrt2 = 1.41421356237309504880;
#pragma unroll
    for (int q = 0; q < kLowPer; ++q) {
        const int y = y0 + g * kLowPer + q;
        if (y >= a.N) break;
        double2 s = bp[q];
        if (k > 0) s = make_double2(s.x + bm[q].x, s.y - bm[q].y);
        G[((int64_t)b * a.N + y) * K1 + k] = make_double2(kSqrt2 * s.x, kSqrt2 * s.y);
    }
}

hipError_t launch_low_modes(void *G, int N, int K, int nbatch, uint32_t r0, uint32_t seed_lo, uint32_t seed_hi,
                            double amp0, double neg_beta_4, hipStream_t stream, bool swap, void *chirp_tab,
                            double chirp_a, double chirp_scale) {
    if (K < 0 || 2 * K + 1 > kLowW || K >= N / 2 || nbatch < 1) return hipErrorInvalidValue;
    const int64_t per = (N + kLowRows - 1) / kLowRows;
    const bool small = per * nbatch <= 256;  // one per CU
    const int nt = small ? 1024 : 256;
    // (a grid's threads are counted in 32 bits)
    const int64_t most = (((1ll << 32) - 1) / nt - (N + nt - 1) / nt) / per;
    for (int64_t b0 = 0; b0 < nbatch; b0 += most) {
        const int64_t nb = nbatch - b0 < most ? nbatch - b0 : most;
        // (the chirp table with the first screens)
        const int64_t blocks = per * nb, chirp = chirp_tab && b0 == 0 ? (N + nt - 1) / nt : 0;
        LowModeArgs a{N, K, r0 + (uint32_t)b0, seed_lo, seed_hi, amp0, neg_beta_4, swap ? 1 : 0,
                      static_cast<cpx<float> *>(chirp_tab), chirp_a, chirp_scale, (int)blocks};
        double2 *Gb = static_cast<double2 *>(G) + b0 * N * (K + 1);
        if (small)
            hipLaunchKernelGGL((low_modes_kernel<1024>), dim3((unsigned)(blocks + chirp)), dim3(1024), 0, stream, Gb, a);
        else
            hipLaunchKernelGGL((low_modes_kernel<256>), dim3((unsigned)(blocks + chirp)), dim3(256), 0, stream, Gb, a);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- twiddles
struct TwiddleArgs {
    int n, total;
    int ns[8], R[8], off[8];
};

template <typename Real>
__global__ __launch_bounds__(256) void twiddle_table_kernel(cpx<Real> *tab, TwiddleArgs a) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= a.total) return;
    int s = 0;
    while (s + 1 < a.n && i >= a.off[s + 1]) ++s;
    const int j = i - a.off[s];
    const int64_t k = j / a.R[s], r = j - k * a.R[s];
    const int64_t M = (int64_t)a.ns[s] * a.R[s];
    const int64_t m = (r * k) % M;
    double sn, cs;
    sincospi(2.0 * (double)m / (double)M, &sn, &cs);
    tab[i] = {(Real)cs, (Real)(-sn)};
}

hipError_t launch_twiddle_table(void *tab, int n_stages, const int *ns, const int *R, const int *off, int total,
                                bool f64, hipStream_t stream) {
    if (n_stages < 0 || n_stages > 8 || total < 0) return hipErrorInvalidValue;
    if (total == 0) return hipSuccess;
    TwiddleArgs a{};
    a.n = n_stages;
    a.total = total;
    for (int s = 0; s < n_stages; ++s) {
        a.ns[s] = ns[s];
        a.R[s] = R[s];
        a.off[s] = off[s];
    }
    const dim3 grid((total + 255) / 256);
    if (f64)
        hipLaunchKernelGGL((twiddle_table_kernel<double>), grid, dim3(256), 0, stream, static_cast<cpx<double> *>(tab), a);
    else
        hipLaunchKernelGGL((twiddle_table_kernel<float>), grid, dim3(256), 0, stream, static_cast<cpx<float> *>(tab), a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- chirp
struct ChirpArgs {
    double a[64];
    double amp[64];
};

template <typename Real>
__global__ __launch_bounds__(256) void chirp_kernel(cpx<Real> *tab, int N, ChirpArgs args, int n, double scale) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int j = blockIdx.y;
    if (k >= N || j >= n) return;
    tab[(int64_t)j * N + k] = chirp_value<Real>(k, N, args.a[j], scale * args.amp[j]);
}

hipError_t launch_chirp_tables(void *tab, int N, const double *a, int n, double scale, bool f64,
                               hipStream_t stream, const double *amp) {
    if (n < 1 || n > 64) return hipErrorInvalidValue;
    ChirpArgs args{};
    for (int j = 0; j < n; ++j) {
        args.a[j] = a[j];
        args.amp[j] = amp ? amp[j] : 1.0;
    }
    dim3 grid((N + 255) / 256, n);
    if (f64)
        hipLaunchKernelGGL((chirp_kernel<double>), grid, dim3(256), 0, stream, static_cast<cpx<double> *>(tab), N,
                           args, n, scale);
    else
        hipLaunchKernelGGL((chirp_kernel<float>), grid, dim3(256), 0, stream, static_cast<cpx<float> *>(tab), N,
                           args, n, scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------- aperture
// A[j] = SF(j + 1/2) exp(i ((j - N/2)^2 / (2 rho^2) + pi j)) in FP64, rounded
// once.  The phase is formed in turns, (j - N/2)^2 exactly times
// 1/(4 pi rho^2), plus j/2, and reduced to [-1/2, 1/2] before sincospi.  The
// window is the raised sine over Lm pixels at each border (Lm = 0: none).
template <typename Real>
__global__ __launch_bounds__(256) void aperture_table_kernel(cpx<Real> *tab, int N, double a, double Lm) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    const double d = (double)(j - N / 2);
    const double turns = a * (d * d) + 0.5 * (double)(j & 1);
    const double f = turns - rint(turns);
    double s, c;
    sincospi(2.0 * f, &s, &c);
    const double x = (double)j + 0.5;
    double w = 1.0;
    if (Lm > 0.0) {
        if (x <= Lm)
            w = 0.5 * (1.0 - cospi(x / Lm));
        else if (x >= (double)N - Lm)
            w = 0.5 * (1.0 + cospi((x - (double)N + Lm) / Lm));
    }
    tab[j] = {(Real)(w * c), (Real)(w * s)};
}

hipError_t launch_aperture_table(void *tab, int N, double a, double Lm, bool f64, hipStream_t stream) {
    dim3 grid((N + 255) / 256);
    if (f64)
        hipLaunchKernelGGL((aperture_table_kernel<double>), grid, dim3(256), 0, stream,
                           static_cast<cpx<double> *>(tab), N, a, Lm);
    else
        hipLaunchKernelGGL((aperture_table_kernel<float>), grid, dim3(256), 0, stream,
                           static_cast<cpx<float> *>(tab), N, a, Lm);
    return hipGetLastError();
}

// ---------------------------------------------------------------- disk
template <typename Real>
__global__ __launch_bounds__(256) void disk_kernel(Real *img, int N, double r2, double value) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= N) return;
    const double dx = (double)(x < N / 2 ? x : x - N);
    const double dy = (double)(y < N / 2 ? y : y - N);
    img[(int64_t)y * N + x] = (dx * dx + dy * dy <= r2) ? (Real)value : (Real)0;
}

hipError_t launch_disk_image(void *img, int N, double r2, double value, bool f64, hipStream_t stream) {
    dim3 grid((N + 255) / 256, N);
    if (f64)
        hipLaunchKernelGGL((disk_kernel<double>), grid, dim3(256), 0, stream, static_cast<double *>(img), N, r2,
                           value);
    else
        hipLaunchKernelGGL((disk_kernel<float>), grid, dim3(256), 0, stream, static_cast<float *>(img), N, r2,
                           value);
    return hipGetLastError();
}

// ---------------------------------------------------------------- reductions
// Block tree over 256 FP64 partials in LDS (fixed order).
__device__ __forceinline__ double block_tree_sum(double v, double *red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

// Mean and variance of a w x h region in one read of it (bound by that read;
// two passes, the mean and then the squared deviations, took 42 + 27 us for
// two 4000^2 patterns).  Each thread sums x and, about its own first element
// c, x - c and (x - c)^2, in FP64; count, mean and sum of squared deviations
// of two sets combine as
//   M2 = M2a + M2b + (mean_b - mean_a)^2 n_a n_b / (n_a + n_b),
// which loses nothing to a mean far from zero, in a fixed order.
struct Moments {
    double n, sum, mean, m2;
};
__device__ __forceinline__ Moments merge(const Moments &a, const Moments &b) {
    if (b.n == 0.0) return a;
    if (a.n == 0.0) return b;
    const double n = a.n + b.n, d = b.mean - a.mean, f = b.n / n;
    return {n, a.sum + b.sum, a.mean + d * f, a.m2 + b.m2 + d * d * (a.n * f)};
}
__device__ __forceinline__ Moments block_merge(Moments v, Moments *red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = merge(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    return red[0];
}
struct MomentSums {
    double c, n, s0, s1, s2;
    __device__ __forceinline__ void add(double x) {
        if (n == 0.0) c = x;
        const double d = x - c;
        n += 1.0;
        s0 += x;
        s1 += d;
        s2 = fma(d, d, s2);
    }
    __device__ __forceinline__ Moments get() const {
        if (n == 0.0) return {0.0, 0.0, 0.0, 0.0};
        // (>= 0, NaN where a sum is, infinite where only the squares overflow)
        const double m2 = isinf(s2) && isfinite(s1) ? s2 : fmax(s2 - s1 * (s1 / n), 0.0 * s2);
        return {n, s0, c + s1 / n, m2};
    }
};

// VEC elements per load: 16 bytes for a contiguous run (w == row_stride, h
// rows of it), else 1.  Rows of a narrower region are walked by rows of
// 2^log_tx threads, as many as its width asks for, up to a workgroup's 256; up
// to there each thread keeps to one column (a 2 x 4096 strip by whole rows of
// 256, two of them busy: 396 us per call; with the rows dealt out to all 32).
template <typename Real, int VEC>
__global__ __launch_bounds__(256) void moments_kernel(const Real *__restrict__ x, int64_t batch_stride, int64_t w,
                                                      int64_t h, int64_t row_stride, int log_tx, Moments *partials) {
    __shared__ Moments red[256];
    const int b = blockIdx.y, nblk = gridDim.x;
    const Real *xb = x + (int64_t)b * batch_stride;
    MomentSums a{0.0, 0.0, 0.0, 0.0, 0.0};
    if constexpr (VEC > 1) {
        using Vec = Real __attribute__((ext_vector_type(VEC)));
        const Vec *xv = reinterpret_cast<const Vec *>(xb);
        const int64_t n = w * h / VEC, step = (int64_t)nblk * 256;
        int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
        for (; i + 3 * step < n; i += 4 * step) {  // four loads in flight
            const Vec v0 = xv[i], v1 = xv[i + step], v2 = xv[i + 2 * step], v3 = xv[i + 3 * step];
#pragma unroll
            for (int e = 0; e < VEC; ++e) a.add((double)v0[e]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) a.add((double)v1[e]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) a.add((double)v2[e]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) a.add((double)v3[e]);
        }
        for (; i < n; i += step) {
            const Vec v = xv[i];
#pragma unroll
            for (int e = 0; e < VEC; ++e) a.add((double)v[e]);
        }
    } else {
        if (w <= 256) {
            const int lane = threadIdx.x & ((1 << log_tx) - 1), rows = 256 >> log_tx;
            const int64_t step = (int64_t)nblk * rows;
            int64_t y = lane < w ? (int64_t)blockIdx.x * rows + (threadIdx.x >> log_tx) : h;
            const Real *col = xb + lane;
            for (; y + 3 * step < h; y += 4 * step) {  // four loads in flight
                const Real v0 = col[y * row_stride], v1 = col[(y + step) * row_stride],
                           v2 = col[(y + 2 * step) * row_stride], v3 = col[(y + 3 * step) * row_stride];
                a.add((double)v0);
                a.add((double)v1);
                a.add((double)v2);
                a.add((double)v3);
            }
            for (; y < h; y += step) a.add((double)col[y * row_stride]);
        } else {
            for (int64_t y = blockIdx.x; y < h; y += nblk) {
                const Real *row = xb + y * row_stride;
                int64_t i = threadIdx.x;
                for (; i + 3 * 256 < w; i += 4 * 256) {
                    const Real v0 = row[i], v1 = row[i + 256], v2 = row[i + 512], v3 = row[i + 768];
                    a.add((double)v0);
                    a.add((double)v1);
                    a.add((double)v2);
                    a.add((double)v3);
                }
                for (; i < w; i += 256) a.add((double)row[i]);
            }
        }
    }
    const Moments tot = block_merge(a.get(), red);
    if (threadIdx.x == 0) partials[(int64_t)b * nblk + blockIdx.x] = tot;
}

// stats[2b], stats[2b + 1] = mean, population variance of region b
__global__ __launch_bounds__(256) void moments_finish_kernel(const Moments *partials, int nblk, double *stats) {
    __shared__ Moments red[256];
    const int b = blockIdx.x;
    Moments a{0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < nblk; i += 256) a = merge(a, partials[(int64_t)b * nblk + i]);
    const Moments tot = block_merge(a, red);
    if (threadIdx.x == 0) {
        stats[2 * b] = tot.sum / tot.n;
        stats[2 * b + 1] = tot.m2 / tot.n;
    }
}

static int moment_log_tx(int64_t w) {
    int l = 0;
    while (l < 8 && ((int64_t)1 << l) < w) ++l;
    return l;
}
static int moment_blocks(int64_t w, int64_t h, bool run) {
    // at least 16 elements per thread, at most four workgroups per CU
    const int64_t rows = 256 >> moment_log_tx(w), sets = run ? 1024 : (h + rows - 1) / rows;
    const int64_t want = (w * h + 4095) / 4096, most = sets < 1024 ? sets : 1024;
    return (int)(want < 1 ? 1 : want < most ? want : most);
}
size_t moments_scratch_bytes(int64_t w, int64_t h, int nbatch) {
    return (size_t)nbatch * moment_blocks(w, h, true) * sizeof(Moments);
}

hipError_t launch_moments(const void *x, int64_t batch_stride, int64_t w, int64_t h, int64_t row_stride, int nbatch,
                          bool f64, double *stats, void *scratch, hipStream_t stream) {
    const int vec = f64 ? 2 : 4;
    // a full-width region (or a single row) is one contiguous run; 16-byte
    // loads where every batch member starts on one
    const bool run = w == row_stride || h == 1;
    const bool wide = run && (w * h) % vec == 0 && ((uintptr_t)x & 15u) == 0 && batch_stride % vec == 0;
    const int nblk = moment_blocks(w, h, wide), log_tx = moment_log_tx(w);
    Moments *part = static_cast<Moments *>(scratch);
    const int64_t rs = h == 1 ? w : row_stride;
    for (int b0 = 0; b0 < nbatch; b0 += 65535) {
        const int nb = nbatch - b0 < 65535 ? nbatch - b0 : 65535;
        const dim3 grid(nblk, nb);
        Moments *p = part + (int64_t)b0 * nblk;
        const int64_t off = (int64_t)b0 * batch_stride;
        if (f64) {
            const double *xd = static_cast<const double *>(x) + off;
            if (wide)
                hipLaunchKernelGGL((moments_kernel<double, 2>), grid, dim3(256), 0, stream, xd, batch_stride, w, h, rs, log_tx, p);
            else
                hipLaunchKernelGGL((moments_kernel<double, 1>), grid, dim3(256), 0, stream, xd, batch_stride, w, h, rs, log_tx, p);
        } else {
            const float *xf = static_cast<const float *>(x) + off;
            if (wide)
                hipLaunchKernelGGL((moments_kernel<float, 4>), grid, dim3(256), 0, stream, xf, batch_stride, w, h, rs, log_tx, p);
            else
                hipLaunchKernelGGL((moments_kernel<float, 1>), grid, dim3(256), 0, stream, xf, batch_stride, w, h, rs, log_tx, p);
        }
        if (hipError_t e = hipGetLastError()) return e;
        hipLaunchKernelGGL(moments_finish_kernel, dim3(nb), dim3(256), 0, stream, p, nblk, stats + 2 * (size_t)b0);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- light curves
// One workgroup per (pattern, line): sample k of line l lies at
// (x0 + k dx, y0 + k dy) pixels (pixel (ix, iy) at the integer point), wrapped
// onto the periodic pattern; mode 0 takes the nearest pixel, mode 1
// interpolates bilinearly (weights and sum in FP64).  The curve is written
// and its mean and population variance formed in FP64 in a fixed order.
__device__ __forceinline__ int64_t wrap_floor(double v, int N) {
    const int64_t i = (int64_t)floor(v);
    const int64_t r = i % N;
    return r < 0 ? r + N : r;
}

// x0 + k dx with the product and the sum rounded separately (no fused
// multiply-add), the same position a plain evaluation of the formula gives
__device__ __forceinline__ double sample_coord(double x0, int k, double dx) {
#pragma clang fp contract(off)
    return x0 + (double)k * dx;
}

template <typename Real>
__global__ __launch_bounds__(256) void light_curve_kernel(const Real *__restrict__ I, int N, LineSet ls, int n_samples,
                                                          int mode, Real *__restrict__ out, int n_lines_total,
                                                          int line0, double *stats) {
    __shared__ double red[256];
    const int l = blockIdx.x, b = blockIdx.y;
    const Real *img = I + (int64_t)b * N * N;
    Real *c = out + ((int64_t)b * n_lines_total + line0 + l) * n_samples;
    const double x0 = ls.p[l][0], y0 = ls.p[l][1], dx = ls.p[l][2], dy = ls.p[l][3];
    double acc = 0.0;
    for (int k = threadIdx.x; k < n_samples; k += 256) {
        const double x = sample_coord(x0, k, dx), y = sample_coord(y0, k, dy);
        Real v;
        if (mode == 0) {
            v = img[wrap_floor(y + 0.5, N) * N + wrap_floor(x + 0.5, N)];
        } else {
            const double fx = x - floor(x), fy = y - floor(y);
            const int64_t ix = wrap_floor(x, N), iy = wrap_floor(y, N);
            const int64_t jx = ix + 1 == N ? 0 : ix + 1, jy = iy + 1 == N ? 0 : iy + 1;
            v = (Real)((1.0 - fx) * (1.0 - fy) * (double)img[iy * N + ix] + fx * (1.0 - fy) * (double)img[iy * N + jx] +
                       (1.0 - fx) * fy * (double)img[jy * N + ix] + fx * fy * (double)img[jy * N + jx]);
        }
        c[k] = v;
        acc += (double)v;
    }
    const double mean = block_tree_sum(acc, red) / (double)n_samples;
    __syncthreads();
    double acc2 = 0.0;
    for (int k = threadIdx.x; k < n_samples; k += 256) {  // each thread re-reads its own samples
        const double d = (double)c[k] - mean;
        acc2 += d * d;
    }
    const double var = block_tree_sum(acc2, red) / (double)n_samples;
    if (threadIdx.x == 0 && stats) {
        stats[2 * ((int64_t)b * n_lines_total + line0 + l)] = mean;
        stats[2 * ((int64_t)b * n_lines_total + line0 + l) + 1] = var;
    }
}

hipError_t launch_light_curves(const void *I, int N, int nbatch, const double *lines, int n_lines, int n_samples,
                               int mode, bool f64, void *out, double *stats, hipStream_t stream) {
    for (int l0 = 0; l0 < n_lines; l0 += kLinesPerLaunch) {
        const int nl = n_lines - l0 < kLinesPerLaunch ? n_lines - l0 : kLinesPerLaunch;
        LineSet ls{};
        for (int l = 0; l < nl; ++l)
            for (int q = 0; q < 4; ++q) ls.p[l][q] = lines[4 * (l0 + l) + q];
        dim3 grid(nl, nbatch);
        if (f64)
            hipLaunchKernelGGL((light_curve_kernel<double>), grid, dim3(256), 0, stream,
                               static_cast<const double *>(I), N, ls, n_samples, mode, static_cast<double *>(out),
                               n_lines, l0, stats);
        else
            hipLaunchKernelGGL((light_curve_kernel<float>), grid, dim3(256), 0, stream,
                               static_cast<const float *>(I), N, ls, n_samples, mode, static_cast<float *>(out),
                               n_lines, l0, stats);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- structure function
// Ring sums of a power map P [batch][N][N] (either orientation): ring b holds
// the pixels of signed frequency k' (components in [-N/2, N/2)) with
// (2b - 1)^2 <= 4 |k'|^2 < (2b + 1)^2 (|k'| rounds to b).  Bound by the read of
// P: neighbouring threads take neighbouring rings of one row, whose pixels lie
// next to each other (one workgroup per ring, its threads on different rows,
// read every pixel from a line of its own: 231 us for two 4000^2 maps).  A
// workgroup takes 256 rings of kRingRows values of |ky'|, each of them the two
// rows +-ky'; every thread sums its ring in a fixed order, and a second kernel
// adds the row groups in order, so the result is reproducible.  A ring crosses
// most rows in one or two pixels: the first two of every row are loaded before
// any is waited for.
constexpr int kRingRows = 4;

__device__ __forceinline__ int64_t isqrt_floor(int64_t v) {  // floor(sqrt(v)), v >= 0
    int64_t r = (int64_t)sqrt((double)v);
    while (r * r > v) --r;
    while ((r + 1) * (r + 1) <= v) ++r;
    return r;
}
// largest k with 4 k^2 < v, v > 0
__device__ __forceinline__ int ring_edge(int64_t v) { return (int)isqrt_floor((v - 1) / 4); }

template <typename Real>
__global__ __launch_bounds__(256) void ring_part_kernel(const Real *__restrict__ P, int N, double *part, double *count) {
    const int b = blockIdx.x * 256 + (int)threadIdx.x, rows0 = blockIdx.y * kRingRows, bat = blockIdx.z;
    const int h = N / 2;
    if (b > h) return;
    const Real *img = P + (int64_t)bat * N * N;
    const int64_t lo2 = b == 0 ? 0 : (int64_t)(2 * b - 1) * (2 * b - 1), hi2 = (int64_t)(2 * b + 1) * (2 * b + 1);
    int k0[kRingRows], k1[kRingRows];
    double v[kRingRows][2][4];
    // the four pixels (+-kx, +-ky') of row a, 0 for those that do not exist:
    // components lie in [-h, h), and -0 is 0
    auto pixels = [&](int a, int kx, double (&x)[4]) {
        const Real *up = img + (int64_t)(a < h ? a : 0) * N, *down = img + (int64_t)(a > 0 ? N - a : 0) * N;
        const int r = kx < h ? kx : 0, l = kx > 0 ? N - kx : 0;
        const double ur = (double)up[r], dr = (double)down[r], ul = (double)up[l], dl = (double)down[l];
        x[0] = kx < h && a < h ? ur : 0.0;
        x[1] = kx < h && a > 0 ? dr : 0.0;
        x[2] = kx > 0 && a < h ? ul : 0.0;
        x[3] = kx > 0 && a > 0 ? dl : 0.0;
    };
#pragma unroll
    for (int i = 0; i < kRingRows; ++i) {
        const int a = rows0 + i;
        const int64_t t = 4 * (int64_t)a * a;
        const bool in = a <= h && t < hi2;
        // kx >= 0 with lo2 <= 4 kx^2 + t < hi2
        k0[i] = in && lo2 > t ? ring_edge(lo2 - t) + 1 : 0;
        k1[i] = in ? min(ring_edge(hi2 - t), h) : -1;
#pragma unroll
        for (int q = 0; q < 2; ++q) pixels(in ? a : 0, min(k0[i] + q, h), v[i][q]);
    }
    double acc = 0.0;
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < kRingRows; ++i) {
        const int a = rows0 + i, rows = (a < h) + (a > 0);
        for (int kx = k0[i]; kx <= k1[i]; ++kx) {
            double x[4];
            if (kx - k0[i] < 2) {
                const int q = kx - k0[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = q ? v[i][1][e] : v[i][0][e];
            } else {
                pixels(a, kx, x);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) acc += x[e];
            cnt += rows * ((kx < h) + (kx > 0));
        }
    }
    const int64_t o = (int64_t)blockIdx.y * (h + 1) + b;
    part[(int64_t)bat * gridDim.y * (h + 1) + o] = acc;
    if (bat == 0) count[o] = (double)cnt;
}

// S[screen][b]: the sum over the row groups in order, over the number of the
// ring's pixels.  A workgroup takes 32 rings, 8 threads each (the groups that
// can touch ring b end at row b).
__global__ __launch_bounds__(256) void ring_sum_kernel(const double *part, const double *count, int nbins, int groups,
                                                       double *S) {
    __shared__ double red[2][8][32];
    const int l = threadIdx.x % 32, g = threadIdx.x / 32, b = blockIdx.x * 32 + l, bat = blockIdx.y;
    double acc = 0.0, cnt = 0.0;
    if (b < nbins) {
        const double *p = part + (int64_t)bat * groups * nbins + b;
        for (int q = g; q < groups && q * kRingRows <= b + 1; q += 8) {
            acc += p[(int64_t)q * nbins];
            cnt += count[(int64_t)q * nbins + b];
        }
    }
    red[0][g][l] = acc;
    red[1][g][l] = cnt;
    __syncthreads();
    if (g == 0 && b < nbins) {
        for (int q = 1; q < 8; ++q) {
            acc += red[0][q][l];
            cnt += red[1][q][l];
        }
        S[(int64_t)bat * nbins + b] = cnt > 0.0 ? acc / cnt : 0.0;
    }
}

static int ring_groups(int N) { return (N / 2 + 1 + kRingRows - 1) / kRingRows; }
size_t ring_scratch_bytes(int N, int nbatch) { return (size_t)(nbatch + 1) * ring_groups(N) * (N / 2 + 1) * 8; }

hipError_t launch_ring_sums(const void *P, int N, int nbatch, bool f64, double *S, void *scratch, hipStream_t stream) {
    const int nbins = N / 2 + 1, groups = ring_groups(N);
    double *count = static_cast<double *>(scratch), *part = count + (size_t)groups * nbins;
    for (int b0 = 0; b0 < nbatch; b0 += 65535) {
        const int nb = nbatch - b0 < 65535 ? nbatch - b0 : 65535;
        const dim3 grid((nbins + 255) / 256, groups, nb);
        if (f64)
            hipLaunchKernelGGL((ring_part_kernel<double>), grid, dim3(256), 0, stream,
                               static_cast<const double *>(P) + (int64_t)b0 * N * N, N, part, count);
        else
            hipLaunchKernelGGL((ring_part_kernel<float>), grid, dim3(256), 0, stream,
                               static_cast<const float *>(P) + (int64_t)b0 * N * N, N, part, count);
        if (hipError_t e = hipGetLastError()) return e;
        hipLaunchKernelGGL(ring_sum_kernel, dim3((nbins + 31) / 32, nb), dim3(256), 0, stream, part, count, nbins, groups,
                           S + (int64_t)b0 * nbins);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

// J0, the Bessel function of the first kind of order 0, in FP64: its power
// series sum_k (-x^2/4)^k / (k!)^2 below x = 14 (largest term about 1e4, so
// an absolute error near 1e-12), and above it Hankel's asymptotic expansion
// J0 = sqrt(2 / (pi x)) (P cos(x - pi/4) - Q sin(x - pi/4)),
// P = sum_k (-1)^k a_2k / x^2k, Q = sum_k (-1)^k a_(2k+1) / x^(2k+1),
// a_k = prod_{j <= k} (2j - 1)^2 / (k! 8^k), summed while the terms shrink.
// Both sums run over a fixed number of terms with compile-time ratios (a
// loop that divides, or takes the ratios from memory, waits for each): 48 of
// the series, whose later terms vanish beside any sum, and 28 of the
// expansion, up to its smallest term at x = 14 (1.0e-13; 1.5e-14 at 15).
constexpr int kJ0Series = 48, kJ0Hankel = 28;

__device__ double bessel_j0(double x) {
    x = fabs(x);
    if (x < 14.0) {
        const double y = -0.25 * x * x;
        double t = 1.0, sum = 1.0;
#pragma unroll
        for (int k = 1; k <= kJ0Series; ++k) {
            t *= y * (1.0 / ((double)k * (double)k));
            sum += t;
        }
        return sum;
    }
    const double ix = 1.0 / x;
    double P = 1.0, Q = 0.0, term = 1.0;
#pragma unroll
    for (int k = 1; k <= kJ0Hankel; ++k) {
        term *= ix * ((double)((2 * k - 1) * (2 * k - 1)) / (8.0 * k));
        if (k & 1)
            Q += ((k / 2) & 1) ? term : -term;  // k = 1: -a1/x, k = 3: +a3/x^3, ...
        else
            P += ((k / 2) & 1) ? -term : term;  // k = 2: -a2/x^2, k = 4: +a4/x^4, ...
    }
    double sn, cs;
    sincos(x - 0.25 * kPi, &sn, &cs);
    return sqrt(2.0 / (kPi * x)) * (P * cs - Q * sn);
}

// D(r) = 2 sum_{b=1}^{N/2} 2 pi (b/N) S_b (1 - J0(2 pi b r / N)) / N for the
// workgroup's ring spectrum S (pixel units), summed over the block.
__device__ double structure_at(const double *S, int N, double r, double *red) {
    double acc = 0.0;
    for (int b = 1 + (int)threadIdx.x; b <= N / 2; b += 256) {
        const double q = (double)b / N;
        acc += q * S[b] * (1.0 - bessel_j0(2.0 * kPi * q * r));
    }
    __syncthreads();
    const double tot = block_tree_sum(acc, red);
    return 4.0 * kPi * tot / N;
}

// D at one radius per workgroup: D[screen ld_D + r0 + j] for radius j (pixels).
__global__ __launch_bounds__(256) void hankel_kernel(const double *S, int N, RadiusSet rs, double *D, int ld_D, int r0) {
    __shared__ double red[256];
    const int j = blockIdx.x, bat = blockIdx.y;
    const double d = structure_at(S + (int64_t)bat * (N / 2 + 1), N, rs.r[j], red);
    if (threadIdx.x == 0) D[(int64_t)bat * ld_D + r0 + j] = d;
}

// R_diff^rec solves D = 1 by bisection on [1e-3, N/2] to a relative 1e-12 (NaN
// when the root is not bracketed), several levels of it per launch: one
// workgroup for each of the 2^levels - 1 midpoints that these levels can come
// to evaluates D there, and the next launch walks down the tree.  On one
// workgroup per screen the 40-60 evaluations run one after the other (the whole
// call for one 4000^2 screen 503 us, for one of 20000^2 5.91 ms; by launches of
// eight levels 313 us and 4.74 ms).  RootState of a screen: the
// bracket before the launch's levels and D at their midpoints (node 1 the
// first, nodes 2n and 2n + 1 below and above it); two alternate.
constexpr int kRootLevels = 8, kRootNodes = 1 << kRootLevels;
constexpr double kRootLo = 1e-3;
struct RootState {
    double lo, hi;
    double D[kRootNodes];
};

// Levels per launch: a level more doubles the evaluations, so as many as keep
// a launch within kRootGroups workgroups; 0, every screen's bisection on a
// workgroup of its own, where fewer than kRootLeast are left (from 69 screens).
// Screens of 64^2, us per call, eight levels always / on one workgroup / this
// rule: 4 116 / 143 / 106, 32 231 / 148 / 123, 128 614 / 154 / 147,
// 4096 16494 / 930 / 931; of 1000^2: 8 229 / 239 / 205, 64 1098 / 720 / 719.
// (2048 workgroups, 64^2: 32 155, 128 197; 4096: 175 and 215.)
constexpr int kRootGroups = 1024, kRootLeast = 4;
static int root_levels(int nbatch) {
    int levels = kRootLevels;
    while (levels >= kRootLeast && (int64_t)nbatch * ((1 << levels) - 1) > kRootGroups) --levels;
    return levels >= kRootLeast ? levels : 0;
}

__device__ __forceinline__ bool root_found(double lo, double hi) { return !(hi - lo > 1e-12 * hi); }

__device__ __forceinline__ void root_walk(const RootState &s, int nodes, double &lo, double &hi) {
    lo = s.lo;
    hi = s.hi;
    for (int node = 1; node < nodes && !root_found(lo, hi);) {
        const double mid = 0.5 * (lo + hi);
        const bool below = s.D[node] < 1.0;
        (below ? lo : hi) = mid;
        node = 2 * node + below;
    }
}

// ends: D at the two ends of the first bracket, [screen][2]; first: the
// bracket is the whole range.  Nodes 1 .. gridDim.x.
__global__ __launch_bounds__(256) void root_kernel(const double *S, int N, const double *ends, const RootState *from,
                                                   RootState *to, int first) {
    __shared__ double red[256];
    const int node = blockIdx.x + 1, bat = blockIdx.y;
    if (!(ends[2 * bat] < 1.0 && ends[2 * bat + 1] >= 1.0)) return;
    double lo = kRootLo, hi = 0.5 * N;
    if (!first) root_walk(from[bat], (int)gridDim.x + 1, lo, hi);
    if (node == 1 && threadIdx.x == 0) {
        to[bat].lo = lo;
        to[bat].hi = hi;
    }
    // the node's midpoint, down the path that its bits spell
    for (int bit = 30 - __clz(node); bit >= 0; --bit) {
        if (root_found(lo, hi)) return;
        const double mid = 0.5 * (lo + hi);
        ((node >> bit) & 1 ? lo : hi) = mid;
    }
    if (root_found(lo, hi)) return;  // (the walk stops above this node)
    const double d = structure_at(S + (int64_t)bat * (N / 2 + 1), N, 0.5 * (lo + hi), red);
    if (threadIdx.x == 0) to[bat].D[node] = d;
}

__global__ __launch_bounds__(64) void root_finish_kernel(int n, int nodes, const double *ends, const RootState *from,
                                                         double *rdiff) {
    const int bat = blockIdx.x * 64 + threadIdx.x;
    if (bat >= n) return;
    if (!(ends[2 * bat] < 1.0 && ends[2 * bat + 1] >= 1.0)) {
        rdiff[bat] = __longlong_as_double(0x7ff8000000000000LL);
        return;
    }
    double lo, hi;
    root_walk(from[bat], nodes, lo, hi);
    rdiff[bat] = 0.5 * (lo + hi);
}

// The same midpoints and decisions, one screen per workgroup.
__global__ __launch_bounds__(256) void root_serial_kernel(const double *S, int N, const double *ends, double *rdiff) {
    __shared__ double red[256];
    const int bat = blockIdx.x;
    if (!(ends[2 * bat] < 1.0 && ends[2 * bat + 1] >= 1.0)) {
        if (threadIdx.x == 0) rdiff[bat] = __longlong_as_double(0x7ff8000000000000LL);
        return;
    }
    double lo = kRootLo, hi = 0.5 * N;
    for (int it = 0; it < 200 && !root_found(lo, hi); ++it) {  // every thread sees the same lo, hi
        const double mid = 0.5 * (lo + hi);
        (structure_at(S + (int64_t)bat * (N / 2 + 1), N, mid, red) < 1.0 ? lo : hi) = mid;
    }
    if (threadIdx.x == 0) rdiff[bat] = 0.5 * (lo + hi);
}

size_t hankel_scratch_bytes(int nbatch) {
    return (size_t)nbatch * ((root_levels(nbatch) ? 2 * sizeof(RootState) : 0) + 2 * sizeof(double));
}

hipError_t launch_hankel(const double *S, int N, int nbatch, const double *radii, int n_r, double *D, double *rdiff,
                         void *scratch, hipStream_t stream) {
    for (int b0 = 0; b0 < nbatch; b0 += 65535) {
        const int nb = nbatch - b0 < 65535 ? nbatch - b0 : 65535;
        const double *Sb = S + (int64_t)b0 * (N / 2 + 1);
        for (int j0 = 0; j0 < n_r; j0 += kRadiiPerLaunch) {
            const int nr = n_r - j0 < kRadiiPerLaunch ? n_r - j0 : kRadiiPerLaunch;
            RadiusSet rs{};
            for (int j = 0; j < nr; ++j) rs.r[j] = radii[j0 + j];
            hipLaunchKernelGGL(hankel_kernel, dim3(nr, nb), dim3(256), 0, stream, Sb, N, rs, D + (int64_t)b0 * n_r, n_r, j0);
            if (hipError_t e = hipGetLastError()) return e;
        }
        if (!rdiff) continue;
        const int lv = root_levels(nbatch);
        RootState *state = static_cast<RootState *>(scratch);
        double *ends = reinterpret_cast<double *>(state + (lv ? 2 * (size_t)nbatch : 0));
        RadiusSet rs{};
        rs.r[0] = kRootLo;
        rs.r[1] = 0.5 * N;
        hipLaunchKernelGGL(hankel_kernel, dim3(2, nb), dim3(256), 0, stream, Sb, N, rs, ends, 2, 0);
        if (hipError_t e = hipGetLastError()) return e;
        if (!lv) {
            hipLaunchKernelGGL(root_serial_kernel, dim3(nb), dim3(256), 0, stream, Sb, N, ends, rdiff + b0);
            if (hipError_t e = hipGetLastError()) return e;
            continue;
        }
        // the bracket shrinks from N/2 to 1e-12 of a root that is at least
        // 1e-3 pixels: at most log2(N/2 / 1e-15) halvings
        const int levels = (int)std::ceil(std::log2(0.5 * N / (1e-12 * kRootLo)));
        const int rounds = (levels + lv - 1) / lv, nodes = 1 << lv;
        for (int k = 0; k < rounds; ++k) {
            hipLaunchKernelGGL(root_kernel, dim3(nodes - 1, nb), dim3(256), 0, stream, Sb, N, ends,
                               state + (size_t)((k + 1) % 2) * nb, state + (size_t)(k % 2) * nb, k == 0 ? 1 : 0);
            if (hipError_t e = hipGetLastError()) return e;
        }
        hipLaunchKernelGGL(root_finish_kernel, dim3((nb + 63) / 64), dim3(64), 0, stream, nb, nodes, ends,
                           state + (size_t)((rounds - 1) % 2) * nb, rdiff + b0);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

__global__ __launch_bounds__(256) void finalize_kernel(const double *partials, int nblk, double scale, double *out) {
    __shared__ double red[256];
    const int b = blockIdx.x;
    double acc = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) acc += partials[(int64_t)b * nblk + i];
    const double tot = block_tree_sum(acc, red);
    if (threadIdx.x == 0) out[b] = scale * tot;
}

hipError_t launch_finalize_sums(const double *partials, int nblk, int nbatch, double scale, double *out,
                                hipStream_t stream) {
    hipLaunchKernelGGL(finalize_kernel, dim3(nbatch), dim3(256), 0, stream, partials, nblk, scale, out);
    return hipGetLastError();
}

template <typename Real>
__global__ __launch_bounds__(256) void l2_loss_kernel(const Real *__restrict__ I, const Real *__restrict__ It,
                                                      Real *__restrict__ grad, int64_t n, double *partials) {
    __shared__ double red[256];
    const int b = blockIdx.y, nblk = gridDim.x;
    const int64_t off = (int64_t)b * n;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)nblk * 256) {
        const Real d = I[off + i] - It[off + i];
        if (grad) grad[off + i] = (Real)2 * d;
        acc += (double)d * (double)d;
    }
    const double tot = block_tree_sum(acc, red);
    if (threadIdx.x == 0) partials[(int64_t)b * nblk + blockIdx.x] = tot;
}

hipError_t launch_l2_loss(const void *I, const void *It, void *grad, int64_t n_per_batch, int nbatch, int nblk,
                          bool f64, double *partials, hipStream_t stream) {
    dim3 grid(nblk, nbatch);
    if (f64)
        hipLaunchKernelGGL((l2_loss_kernel<double>), grid, dim3(256), 0, stream, static_cast<const double *>(I),
                           static_cast<const double *>(It), static_cast<double *>(grad), n_per_batch, partials);
    else
        hipLaunchKernelGGL((l2_loss_kernel<float>), grid, dim3(256), 0, stream, static_cast<const float *>(I),
                           static_cast<const float *>(It), static_cast<float *>(grad), n_per_batch, partials);
    return hipGetLastError();
}

}  // namespace scint
