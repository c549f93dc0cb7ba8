// HIP kernels of the library outside the sweep and the tall-skinny products
// (pv_tall.hip): fixed-order reductions of the fused dot products, scaling,
// copies, Bloch and random start blocks; and the dispatch of a sweep to its
// stencil family's translation unit (the sweep kernels are in pv_sweep.hpp).
#include "pv_sweep.hpp"

namespace pv {
namespace {

// ------------------------------------------------------------------ reductions

// Sums over the `grid` rows of partials, `pitch` doubles apart, of the first N
// doubles of a row, in a fixed order: lane-strided, an xor tree per wave, then
// the four waves (the result is complete in thread 0).
template <int N>
__device__ __forceinline__ void reduce_rows(const double* __restrict__ q, int grid, int pitch, double (&s)[N]) {
    __shared__ double part[kBlock / 64][N];
#pragma unroll
    for (int k = 0; k < N; ++k) s[k] = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < grid; b += kBlock) {
#pragma unroll
        for (int k = 0; k < N; ++k) s[k] += q[(size_t)b * pitch + k];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        for (int m = 32; m >= 1; m >>= 1) s[k] += __shfl_xor(s[k], m);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][k] = s[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k)
            for (int w = 1; w < kBlock / 64; ++w) s[k] += part[w][k];
    }
    __syncthreads();
}

// One workgroup per block column.  (At 2048 rows and 8 columns: 6.4 us as one
// wave per column.)
__global__ __launch_bounds__(kBlock) void reduce_dots_kernel(const double* __restrict__ partials, int grid, int nb,
                                                             double* __restrict__ dots) {
    double s[4];
    reduce_rows(partials + (size_t)blockIdx.x * 4, grid, nb * 4, s);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) dots[blockIdx.x * 4 + k] = s[k];
}

// Moments of step n = n0 + step, column c (launch_kpm_reduce); the steps after
// the first need mu_0 and mu_1, which with n0 = 0 every workgroup sums for
// itself from step 0's partials.
__device__ __forceinline__ void kpm_reduce(const double* __restrict__ partials, int64_t stride, int grid, int nb,
                                           int width, int c, int n0, int step, double* __restrict__ mu, double invD) {
    const int n = n0 + step;
    double s[2], m[2];
    reduce_rows(partials + step * stride + c * width, grid, nb * width, s);
    if (n0 == 0 && n > 0) reduce_rows(partials + c * width, grid, nb * width, m);
    if (threadIdx.x == 0) {
        for (int k = 0; k < 2; ++k)
            mu[2 * n + k] = n == 0 ? s[k] * invD : 2.0 * s[k] * invD - (n0 == 0 ? m[k] * invD : mu[k]);
    }
}

__global__ __launch_bounds__(kBlock) void kpm_reduce_kernel(const double* __restrict__ partials, int64_t stride,
                                                            int grid, int nb, int width, int n0,
                                                            double* __restrict__ mu, int M, double invD) {
    kpm_reduce(partials, stride, grid, nb, width, blockIdx.y, n0, blockIdx.x, mu + (size_t)blockIdx.y * M, invD);
}

// The same for every instance of a batch: instance and column in blockIdx.x.
__global__ __launch_bounds__(kBlock) void batch_reduce_kernel(const double* __restrict__ partials, int64_t stride,
                                                              const int* __restrict__ inst_block0, int nb, int n0,
                                                              double* __restrict__ mu, int M,
                                                              const double* __restrict__ invD) {
    const int i = blockIdx.x / nb, c = blockIdx.x % nb;
    const int b0 = inst_block0[i], b1 = inst_block0[i + 1];
    kpm_reduce(partials + (size_t)b0 * nb * 2, stride, b1 - b0, nb, 2, c, n0, blockIdx.y, mu + (size_t)blockIdx.x * M,
               invD[i]);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void scale_kernel(int64_t n, const cplx<T>* __restrict__ x,
                                                       double re, double im, cplx<T>* __restrict__ y) {
    const T r = T(re), i = T(im);
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < n; k += (int64_t)gridDim.x * kBlock) {
        const cplx<T> v = x[k];
        y[k] = cplx<T>{r * v.re - i * v.im, r * v.im + i * v.re};
    }
}

// Coefficients of the adjoint source terms of the KPM moments, from their
// cotangent gbar [nb][M] (M = 2N).  With mu_{2k} = 2<w_k,w_k>/D - mu_0 and
// mu_{2k+1} = 2 Re<w_k,w_{k+1}>/D - mu_1, the derivative of L = sum gbar mu
// with respect to w_k is (as a sum of terms coef_j w_{k-1+j}, j = 0, 1, 2)
//   j = 0: 2 gbar_{2k-1}, or for k = 1 ghat_1 = gbar_1 - sum_{n=1}^{N-1} gbar_{2n+1};
//   j = 1: 4 gbar_{2k} (k < N);   j = 2: 2 gbar_{2k+1} (k < N);
// each divided by D.  table[k][j][c] complex (imaginary parts zero), k = 0..N
// (row 0 unused, zero).  One thread per (k, c); ghat_1 summed in order of n.
__global__ __launch_bounds__(kBlock) void kpm_adjoint_table_kernel(const double* __restrict__ gbar, int nb, int M,
                                                                  double invD, double* __restrict__ table) {
    const int N = M / 2;
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= (N + 1) * nb) return;
    const int k = e / nb, c = e % nb;
    const double* gc = gbar + (size_t)c * M;
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
    if (k >= 1) {
        if (k == 1) {
            double ghat1 = gc[1];
            for (int n = 1; n <= N - 1; ++n) ghat1 -= gc[2 * n + 1];
            t0 = ghat1 * invD;
        } else {
            t0 = 2.0 * gc[2 * k - 1] * invD;
        }
        t1 = (k < N ? 4.0 * gc[2 * k] : 0.0) * invD;
        t2 = (k < N ? 2.0 * gc[2 * k + 1] : 0.0) * invD;
    }
    double* row = table + (size_t)k * 3 * nb * 2;
    row[(0 * nb + c) * 2] = t0;
    row[(0 * nb + c) * 2 + 1] = 0.0;
    row[(1 * nb + c) * 2] = t1;
    row[(1 * nb + c) * 2 + 1] = 0.0;
    row[(2 * nb + c) * 2] = t2;
    row[(2 * nb + c) * 2 + 1] = 0.0;
}

// dst[0..n) = 0 for 32-bit words (gradients, zero vectors of the adjoint).
__global__ __launch_bounds__(kBlock) void zero_kernel(uint32_t* __restrict__ dst, int64_t n) {
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < n; k += (int64_t)gridDim.x * kBlock)
        dst[k] = 0u;
}

// Streaming copy: each lane moves 4 x 16 B per iteration with all loads
// issued before the stores; nontemporal on both sides.
__global__ __launch_bounds__(kBlock) void copy_kernel(const u32x4* __restrict__ src,
                                                      u32x4* __restrict__ dst, int64_t n) {
    const int64_t chunk = 4 * (int64_t)kBlock;
    for (int64_t base = blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
        u32x4 r[4];
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i < n) r[k] = __builtin_nontemporal_load(src + i);
        }
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i < n) __builtin_nontemporal_store(r[k], dst + i);
        }
    }
}

// Streaming triad over FP64 pairs: y = x + z, the stream mix of one
// Chebyshev step (two reads, one write) without the stencil.
using f64x2 = double __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(kBlock) void triad_kernel(const f64x2* __restrict__ x, const f64x2* __restrict__ z,
                                                       f64x2* __restrict__ y, int64_t n) {
    const int64_t chunk = 4 * (int64_t)kBlock;
    for (int64_t base = blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
        f64x2 a[4], b[4];
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i < n) {
                a[k] = __builtin_nontemporal_load(x + i);
                b[k] = __builtin_nontemporal_load(z + i);
            }
        }
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i < n) __builtin_nontemporal_store(a[k] + b[k], y + i);
        }
    }
}

// Streaming read: every 16-byte chunk of src is loaded once and folded into
// a per-lane XOR; each wave writes one word (the sink keeps the loads live).
__global__ __launch_bounds__(kBlock) void read_kernel(const u32x4* __restrict__ src, int64_t n,
                                                      uint32_t* __restrict__ sink) {
    const int64_t chunk = 4 * (int64_t)kBlock;
    uint32_t acc = 0;
    for (int64_t base = blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
        u32x4 r[4];
        for (int k = 0; k < 4; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            r[k] = i < n ? __builtin_nontemporal_load(src + i) : u32x4{0u, 0u, 0u, 0u};
        }
        for (int k = 0; k < 4; ++k) acc ^= r[k].x ^ r[k].y ^ r[k].z ^ r[k].w;
    }
    for (int d = 32; d > 0; d >>= 1) acc ^= uint32_t(__shfl_xor(int(acc), d));
    if ((threadIdx.x & 63) == 0) sink[blockIdx.x * (kBlock / 64) + threadIdx.x / 64] = acc;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void column_copy_kernel(const cplx<T>* __restrict__ src, int src_ld,
                                                           int src_col, cplx<T>* __restrict__ dst, int dst_ld,
                                                           int dst_col, int ncols, int64_t n, double re, double im) {
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock) {
        const int64_t r = e / ncols;
        const int c = int(e - r * ncols);
        const cplx<T> v = src[r * src_ld + src_col + c];
        dst[r * dst_ld + dst_col + c] = cplx<T>{T(re * v.re - im * v.im), T(re * v.im + im * v.re)};
    }
}

// Bloch start columns (one element per lane).
template <typename T>
__global__ __launch_bounds__(kBlock) void bloch_kernel(cplx<T>* __restrict__ out, int64_t n, int n_orb, int nb,
                                                     int Lx, int Ly, BlochCols cols, int axis, int64_t index) {
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock) {
        const int c = int(e % nb);
        const int64_t r = e / nb;
        const int o = int(r % n_orb);
        const int64_t s = r / n_orb;
        const int64_t x = s % Lx, y = (s / Lx) % Ly, z = s / ((int64_t)Lx * Ly);
        const int64_t coord = axis == 0 ? x : (axis == 1 ? y : z);
        double re = 0.0, im = 0.0;
        if (o == cols.orb[c] && (axis < 0 || coord == index)) {
            const double ph = cols.k[c][0] * double(x) + cols.k[c][1] * double(y) + cols.k[c][2] * double(z);
            sincos(ph, &im, &re);
        }
        out[e] = cplx<T>{T(re), T(im)};
    }
}

// Random start blocks (one element per lane): element e takes the
// generator's output for index i0 + e; a random phase exp(2 pi i u) from its
// top 53 bits, or the Z4 phase i^k from its top two.
template <typename T, int KIND>
__global__ __launch_bounds__(kBlock) void random_block_kernel(cplx<T>* __restrict__ out, int64_t n, uint64_t seed,
                                                            uint64_t i0) {
    constexpr double kTwoPi = 6.283185307179586;   // the double nearest 2 pi
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n; e += (int64_t)gridDim.x * kBlock) {
        const uint64_t z = splitmix64_at(seed, i0 + uint64_t(e));
        double re, im;
        if constexpr (KIND == 0) {
            const double u = double(z >> 11) * 0x1.0p-53;
            sincos(kTwoPi * u, &im, &re);
        } else {
            const int k = int(z >> 62);
            re = k == 0 ? 1.0 : (k == 2 ? -1.0 : 0.0);
            im = k == 1 ? 1.0 : (k == 3 ? -1.0 : 0.0);
        }
        out[e] = cplx<T>{T(re), T(im)};
    }
}

}  // namespace

static int elementwise_grid(int64_t n);

hipError_t launch_column_copy(int dtype, int64_t rows, int ncols, const void* src, int src_ld, int src_col,
                              void* dst, int dst_ld, int dst_col, double re, double im, hipStream_t s) {
    const int64_t n = rows * ncols;
    const int g = elementwise_grid(n);
    if (dtype == 0)
        hipLaunchKernelGGL(column_copy_kernel<double>, dim3(g), dim3(kBlock), 0, s,
                           static_cast<const cplx<double>*>(src), src_ld, src_col, static_cast<cplx<double>*>(dst),
                           dst_ld, dst_col, ncols, n, re, im);
    else
        hipLaunchKernelGGL(column_copy_kernel<float>, dim3(g), dim3(kBlock), 0, s,
                           static_cast<const cplx<float>*>(src), src_ld, src_col, static_cast<cplx<float>*>(dst),
                           dst_ld, dst_col, ncols, n, re, im);
    return hipGetLastError();
}

hipError_t launch_bloch(int dtype, int64_t n_sites, int n_orb, int nb, int Lx, int Ly, const BlochCols& cols,
                        int axis, int64_t index, void* out, hipStream_t s) {
    const int64_t n = n_sites * n_orb * nb;
    const int g = elementwise_grid(n);
    if (dtype == 0)
        hipLaunchKernelGGL(bloch_kernel<double>, dim3(g), dim3(kBlock), 0, s, static_cast<cplx<double>*>(out), n,
                           n_orb, nb, Lx, Ly, cols, axis, index);
    else
        hipLaunchKernelGGL(bloch_kernel<float>, dim3(g), dim3(kBlock), 0, s, static_cast<cplx<float>*>(out), n,
                           n_orb, nb, Lx, Ly, cols, axis, index);
    return hipGetLastError();
}

hipError_t launch_random_block(int dtype, int kind, int64_t n, uint64_t seed, uint64_t i0, void* out, hipStream_t s) {
    const int g = elementwise_grid(n);
    if (dtype == 0) {
        auto* o = static_cast<cplx<double>*>(out);
        if (kind == 0)
            hipLaunchKernelGGL((random_block_kernel<double, 0>), dim3(g), dim3(kBlock), 0, s, o, n, seed, i0);
        else
            hipLaunchKernelGGL((random_block_kernel<double, 1>), dim3(g), dim3(kBlock), 0, s, o, n, seed, i0);
    } else {
        auto* o = static_cast<cplx<float>*>(out);
        if (kind == 0)
            hipLaunchKernelGGL((random_block_kernel<float, 0>), dim3(g), dim3(kBlock), 0, s, o, n, seed, i0);
        else
            hipLaunchKernelGGL((random_block_kernel<float, 1>), dim3(g), dim3(kBlock), 0, s, o, n, seed, i0);
    }
    return hipGetLastError();
}

int64_t sweep_grid_max(const int64_t L[3], int n_orb, int nb) {
    const int64_t rowel = L[0] * n_orb * nb;
    const int64_t ntiles = (rowel + kBlock - 1) / kBlock * ((L[1] + 7) / 8) * L[2];
    const int tpb = tiles_per_block(ntiles * 8);
    const int64_t direct = 8 * ((ntiles + tpb - 1) / tpb);
    return direct > 8 * 256 ? direct : 8 * 256;   // staged: at most 256 workgroups per XCD part
}

hipError_t launch_sweep(SweepParams& p, int num_cus, hipStream_t s) {
    if ((p.ep & (EP_ACC_ADD | EP_ACC_INIT)) && p.acc_kernel > 0) {
        // series steps: their own launch shape (an extra stream changes the best one)
        SweepParams q = p;
        q.kernel = p.acc_kernel;
        q.st_E = p.acc_E;
        q.st_nt = p.acc_nt;
        q.st_C = p.acc_C;
        q.st_Bm = p.acc_Bm;
        q.st_G8 = p.acc_G8;
        q.acc_kernel = 0;
        const hipError_t e = launch_sweep(q, num_cus, s);
        p.grid = q.grid;
        return e;
    }
    switch (p.family) {
        case FAM_TI: return launch_sweep_ti(p, num_cus, s);
        case FAM_GRAPHENE2: return launch_sweep_graphene2(p, num_cus, s);
        case FAM_GRAPHENE4: return launch_sweep_graphene4(p, num_cus, s);
        case FAM_WEYL: return launch_sweep_weyl(p, num_cus, s);
        default:
            if (p.cg_src) {
                const hipError_t e = launch_codegen(p, num_cus, s);
                if (e != hipErrorNotReady || !p.cg_nocompile) return e;
            }
            return launch_sweep_generic(p, num_cus, s);
    }
}

hipError_t launch_reduce_dots(const double* partials, int grid, int nb, double* dots, hipStream_t s) {
    hipLaunchKernelGGL(reduce_dots_kernel, dim3(nb), dim3(kBlock), 0, s, partials, grid, nb, dots);
    return hipGetLastError();
}

hipError_t launch_kpm_reduce(const double* partials, int64_t stride, int grid, int nb, int width, int n0, int steps,
                             double* mu, int M, double invD, hipStream_t s) {
    hipLaunchKernelGGL(kpm_reduce_kernel, dim3(steps, nb), dim3(kBlock), 0, s, partials, stride, grid, nb, width, n0,
                       mu, M, invD);
    return hipGetLastError();
}

static int elementwise_grid(int64_t n) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return int(g);
}

hipError_t launch_scale_block(int dtype, int64_t n, const void* x, double re, double im, void* y,
                              hipStream_t s) {
    if (dtype == 0)
        hipLaunchKernelGGL(scale_kernel<double>, dim3(elementwise_grid(n)), dim3(kBlock), 0, s, n,
                           static_cast<const cplx<double>*>(x), re, im, static_cast<cplx<double>*>(y));
    else
        hipLaunchKernelGGL(scale_kernel<float>, dim3(elementwise_grid(n)), dim3(kBlock), 0, s, n,
                           static_cast<const cplx<float>*>(x), re, im, static_cast<cplx<float>*>(y));
    return hipGetLastError();
}

hipError_t launch_kpm_adjoint_table(const double* gbar, int nb, int M, double invD, double* table, hipStream_t s) {
    const int n = (M / 2 + 1) * nb;
    hipLaunchKernelGGL(kpm_adjoint_table_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, gbar, nb, M, invD,
                       table);
    return hipGetLastError();
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const int64_t n = int64_t(bytes / 16);
    int64_t g = (n + 4 * kBlock - 1) / (4 * kBlock);
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(copy_kernel, dim3(int(g)), dim3(kBlock), 0, s, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), n);
    return hipGetLastError();
}

hipError_t launch_read(const void* src, size_t bytes, void* sink, hipStream_t s) {
    const int64_t n = int64_t(bytes / 16);
    int64_t g = (n + 4 * kBlock - 1) / (4 * kBlock);
    if (g > STREAM_READ_GROUPS) g = STREAM_READ_GROUPS;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(read_kernel, dim3(int(g)), dim3(kBlock), 0, s, static_cast<const u32x4*>(src), n,
                       static_cast<uint32_t*>(sink));
    return hipGetLastError();
}

hipError_t launch_triad(const void* x, const void* z, void* y, size_t bytes, hipStream_t s) {
    const int64_t n = int64_t(bytes / 16);
    int64_t g = (n + 4 * kBlock - 1) / (4 * kBlock);
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(triad_kernel, dim3(int(g)), dim3(kBlock), 0, s, static_cast<const f64x2*>(x),
                       static_cast<const f64x2*>(z), static_cast<f64x2*>(y), n);
    return hipGetLastError();
}

size_t batch_record_bytes() { return sizeof(KArgs<double, double>); }

hipError_t launch_zero(void* dst, size_t bytes, hipStream_t s) {
    const int64_t n = int64_t(bytes / 4);
    hipLaunchKernelGGL(zero_kernel, dim3(elementwise_grid(n)), dim3(kBlock), 0, s, static_cast<uint32_t*>(dst), n);
    return hipGetLastError();
}

hipError_t batch_fill_record(const SweepParams& p, int staged, void* dst, int* nblocks) {
    switch (p.family) {
        case FAM_TI: return batch_fill_record_ti(p, staged, dst, nblocks);
        case FAM_GRAPHENE2: return batch_fill_record_graphene2(p, staged, dst, nblocks);
        case FAM_GRAPHENE4: return batch_fill_record_graphene4(p, staged, dst, nblocks);
        case FAM_WEYL: return batch_fill_record_weyl(p, staged, dst, nblocks);
        default:
            return p.cg_src ? codegen_batch_fill_record(p, staged, dst, nblocks)
                            : batch_fill_record_generic(p, staged, dst, nblocks);
    }
}

hipError_t launch_batch_sweep(const SweepParams& p, int staged, const void* table, const int* block_inst,
                              const int* inst_block0, int grid, int64_t part_off, hipStream_t s) {
    const void* t = table;
    const int* bi = block_inst;
    const int* i0 = inst_block0;
    switch (p.family) {
        case FAM_TI: return launch_batch_sweep_ti(p, staged, t, bi, i0, grid, part_off, s);
        case FAM_GRAPHENE2: return launch_batch_sweep_graphene2(p, staged, t, bi, i0, grid, part_off, s);
        case FAM_GRAPHENE4: return launch_batch_sweep_graphene4(p, staged, t, bi, i0, grid, part_off, s);
        case FAM_WEYL: return launch_batch_sweep_weyl(p, staged, t, bi, i0, grid, part_off, s);
        default:
            return p.cg_src ? launch_batch_codegen(p, staged, t, bi, i0, grid, part_off, s)
                            : launch_batch_sweep_generic(p, staged, t, bi, i0, grid, part_off, s);
    }
}

hipError_t launch_batch_reduce(const double* partials, int64_t stride, const int* inst_block0, int n_inst, int nb,
                               int n0, int steps, double* mu, int M, const double* invD, hipStream_t s) {
    hipLaunchKernelGGL(batch_reduce_kernel, dim3(n_inst * nb, steps), dim3(kBlock), 0, s, partials, stride,
                       inst_block0, nb, n0, mu, M, invD);
    return hipGetLastError();
}

}  // namespace pv
