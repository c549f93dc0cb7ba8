// Products of tall-skinny blocks on the FP64 matrix cores: G = X^H Y (Gram),
// Y = X Q (rotation), and the same over a search space kept as column blocks
// (Sec. 4.2: orthonormalisation and Rayleigh-Ritz of filter diagonalisation).
//
// Narrow rotations of pv_block_rotate take one thread per entry
// (rotate_by_entry).  Otherwise both are streams of one pass over the blocks: at 32 x 32 columns a row
// costs 1 KiB of reads (180 ps at 5.8 TB/s) and 8192 flops (120 ps at the
// 68 TFLOP/s an FP64 library product reaches), so the target is the memory
// rate, and above 48 columns or so the matrix rate.  v_mfma_f64_16x16x4
// multiplies at the vector units' rate, but one operand register serves 16
// products of it, so operands go from global memory straight to registers:
// no LDS staging and no barrier in either loop.  Measured at 1382400 rows of
// 32 x 32 complex128 columns against vector-unit kernels of one product at a
// time: Gram 959 -> 252 us (5.7 TB/s), accumulating rotation 1515 -> 396 us
// (5.4 TB/s); at 128 x 128 columns the Gram runs at 69 TFLOP/s.
//
// Operand layout of the instruction (lane l): A[i = l % 16][k = l / 16],
// B[k = l / 16][j = l % 16], D[i = 4 r + l / 16][j = l % 16] in register r.
// A lane's 16-byte load of one complex entry is one register of a real and
// one of an imaginary operand; four instructions make a complex tile step.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "pv_kernels.hpp"

namespace pv {
namespace {

using f64x2 = double __attribute__((ext_vector_type(2)));
using f64x4 = double __attribute__((ext_vector_type(4)));
// entries of caller's FP64 matrices, which are aligned as doubles only
using f64x2a = double __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kTallBlock = 256;            // four waves
constexpr int kTile = 16;                  // rows and columns of one matrix instruction
constexpr int kSuper = 64;                 // Gram: most columns of a workgroup's tile, each side
constexpr int kGramRows = 16;              // rows per unit of the Gram grids below

// Columns of a block set: column c of block c >> lg is at base + (c >> lg)
// stride + (c & mask), rows ld elements apart (one plain block: lg = 31).
template <typename T>
struct Cols {
    const T* base;       // interleaved (re, im)
    int64_t stride;      // elements between blocks
    int ld, n, lg;       // row stride, total columns
    __device__ __forceinline__ int64_t at(int c) const {
        return int64_t(c >> lg) * stride + (c & ((1u << lg) - 1u));
    }
};

template <typename T>
__device__ __forceinline__ f64x2 ld_c(const T* base, int64_t e) {
    using V = T __attribute__((ext_vector_type(2)));
    const V v = *reinterpret_cast<const V*>(base + 2 * e);
    return f64x2{double(v.x), double(v.y)};
}

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Partial Gram tiles.  A workgroup owns one tile of at most 64 x 64 columns
// and one group of rows; its four waves split the tile into SX x SY parts of
// (16 WX) x (16 WY) columns and, where there are fewer parts than waves, the
// rows.  A wave takes 8 rows per step (two instructions deep) and loads the
// next step's entries before it multiplies the current ones.  Entries past
// the last column repeat the last column (their products land in entries
// that are not stored); rows past the end are zero on both sides.
// Group g's tile goes to partials[g][nx][ny] (re, im); with hermitian only
// tiles on and above the diagonal are computed.
template <typename T, int WX, int WY>
__global__ __launch_bounds__(kTallBlock, 2) void gram_mfma_kernel(Cols<T> X, Cols<T> Y, int64_t rows, int SX, int SY,
                                                                  int ntx, int nty, int hermitian, int G,
                                                                  double* __restrict__ partials) {
    constexpr int U = 2;   // instruction depths (of four rows) per step
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lc = lane & 15, lr = lane >> 4;
    const int S = SX * SY, RS = 4 / S;
    const int sub = wave % S, rs = wave / S;
    // tile (ti, tj) of the tile list: row-major, tj >= ti only with hermitian
    const int ntiles = hermitian ? ntx * (ntx + 1) / 2 : ntx * nty;
    const int g = blockIdx.x / ntiles;
    int t = blockIdx.x - g * ntiles, ti = 0;
    if (hermitian) {
        while (t >= ntx - ti) {
            t -= ntx - ti;
            ++ti;
        }
        t += ti;
    } else {
        ti = t / nty;
        t -= ti * nty;
    }
    const int i0 = ti * kSuper + (sub / SY) * kTile * WX, j0 = t * kSuper + (sub % SY) * kTile * WY;

    int64_t cx[WX], cy[WY];
#pragma unroll
    for (int w = 0; w < WX; ++w) cx[w] = X.at(min(i0 + w * kTile + lc, X.n - 1)) + int64_t(lr) * X.ld;
#pragma unroll
    for (int w = 0; w < WY; ++w) cy[w] = Y.at(min(j0 + w * kTile + lc, Y.n - 1)) + int64_t(lr) * Y.ld;

    f64x4 re[WX][WY], im[WX][WY];
#pragma unroll
    for (int p = 0; p < WX; ++p)
#pragma unroll
        for (int q = 0; q < WY; ++q) re[p][q] = im[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};

    struct Frag {
        f64x2 x[U][WX], y[U][WY];
    };
    auto load = [&](Frag& f, int64_t r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int w = 0; w < WX; ++w) f.x[u][w] = ld_c(X.base, cx[w] + (r + 4 * u) * X.ld);
#pragma unroll
            for (int w = 0; w < WY; ++w) f.y[u][w] = ld_c(Y.base, cy[w] + (r + 4 * u) * Y.ld);
        }
    };
    auto load_tail = [&](Frag& f, int64_t r) {
        const f64x2 zero{0.0, 0.0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = r + 4 * u + lr < rows;
            // a row that is there for every lane: the last one
            const int64_t q = ok ? r + 4 * u : rows - 1 - lr;
#pragma unroll
            for (int w = 0; w < WX; ++w) {
                const f64x2 v = ld_c(X.base, cx[w] + q * X.ld);
                f.x[u][w] = ok ? v : zero;
            }
#pragma unroll
            for (int w = 0; w < WY; ++w) {
                const f64x2 v = ld_c(Y.base, cy[w] + q * Y.ld);
                f.y[u][w] = ok ? v : zero;
            }
        }
    };
    auto multiply = [&](const Frag& f) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int p = 0; p < WX; ++p) {
                const double xr = f.x[u][p].x, xi = f.x[u][p].y, nxi = -xi;
#pragma unroll
                for (int q = 0; q < WY; ++q) {
                    re[p][q] = mfma(xr, f.y[u][q].x, re[p][q]);
                    im[p][q] = mfma(xr, f.y[u][q].y, im[p][q]);
                }
#pragma unroll
                for (int q = 0; q < WY; ++q) {
                    re[p][q] = mfma(xi, f.y[u][q].y, re[p][q]);
                    im[p][q] = mfma(nxi, f.y[u][q].x, im[p][q]);
                }
            }
    };

    // steps of this wave: k = k0, k0 + dk, ...; the last step of all may be short
    const int64_t nsteps = (rows + 4 * U - 1) / (4 * U), full = rows / (4 * U);
    const int64_t dk = int64_t(G) * RS;
    int64_t k = int64_t(g) * RS + rs;
    Frag A, B;
    if (k < full) load(A, k * 4 * U);
    for (; k + dk < full; k += 2 * dk) {
        load(B, (k + dk) * 4 * U);
        multiply(A);
        // past the end: this wave's own last rows again (not multiplied)
        load(A, (k + 2 * dk < full ? k + 2 * dk : k + dk) * 4 * U);
        multiply(B);
    }
    if (k < full) {
        multiply(A);
        k += dk;
    }
    if (k < nsteps) {
        load_tail(A, k * 4 * U);
        multiply(A);
    }

    // waves that split the rows: fixed-order sum through LDS into row part 0
    extern __shared__ double red[];
    for (int h = 1; h < RS; ++h) {
        double* s = red + (size_t)sub * WX * WY * 8 * 64 + lane;
        if (rs == h) {
#pragma unroll
            for (int p = 0; p < WX; ++p)
#pragma unroll
                for (int q = 0; q < WY; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        s[((p * WY + q) * 8 + v) * 64] = re[p][q][v];
                        s[((p * WY + q) * 8 + 4 + v) * 64] = im[p][q][v];
                    }
        }
        __syncthreads();
        if (rs == 0) {
#pragma unroll
            for (int p = 0; p < WX; ++p)
#pragma unroll
                for (int q = 0; q < WY; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        re[p][q][v] += s[((p * WY + q) * 8 + v) * 64];
                        im[p][q][v] += s[((p * WY + q) * 8 + 4 + v) * 64];
                    }
        }
        __syncthreads();
    }
    if (rs != 0) return;
    f64x2a* out = reinterpret_cast<f64x2a*>(partials) + (size_t)g * X.n * Y.n;
#pragma unroll
    for (int p = 0; p < WX; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + p * kTile + 4 * v + lr;
#pragma unroll
            for (int q = 0; q < WY; ++q) {
                const int j = j0 + q * kTile + lc;
                if (i < X.n && j < Y.n) out[(size_t)i * Y.n + j] = f64x2a{re[p][q][v], im[p][q][v]};
            }
        }
}

// out = sum over the G groups of the partial Gram matrices, in a fixed order:
// 8 threads per entry sum every 8th group, then in order.  With hermitian the
// tiles below the diagonal are the conjugate transposes of those above it.
// (One thread per entry over 512 groups took 123 us at 32 x 32.)
__global__ __launch_bounds__(kTallBlock) void gram_sum_kernel(const f64x2a* __restrict__ partials, int G, int nx,
                                                              int ny, int hermitian, f64x2a* __restrict__ out) {
    constexpr int P = 8, N = kTallBlock / P;
    __shared__ f64x2 s[P][N];
    const int n = nx * ny;
    const int slot = threadIdx.x % N, part = threadIdx.x / N;
    const int e = blockIdx.x * N + slot;
    const int i = e / ny, j = e - i * ny;
    const bool mirror = hermitian && j / kSuper < i / kSuper;
    f64x2 sum{0.0, 0.0};
    if (e < n) {
        const f64x2a* q = partials + (mirror ? j * ny + i : e);
#pragma unroll 8
        for (int g = part; g < G; g += P) sum += q[(size_t)g * n];
    }
    s[part][slot] = sum;
    __syncthreads();
    if (part == 0 && e < n) {
        for (int p = 1; p < P; ++p) sum += s[p][slot];
        if (mirror) sum.y = -sum.y;
        out[e] = sum;
    }
}

// OUT = IN Q (+ OUT): a wave owns 16 rows and 16 WC output columns; a lane's
// operand is X[row l % 16][k = l / 16], so one load covers 64 bytes of 16
// rows and the next one the rest of their cache lines.  The columns of IN go
// by in halves of 16 (four instructions deep), the next half loaded before
// the current one is multiplied.  Columns past the end of IN are zero on both
// sides.  The NW waves of a workgroup are CT column tiles of the same rows (L1
// hits), then further rows.
//
// LQ: the coefficients of the workgroup's columns sit in LDS, zero-padded to
// whole instructions, and the workgroups walk the rows.  At 32 x 32 columns
// (1382400 rows, complex128, accumulating) coefficients that every wave reads
// through L1 cost 409 us, in LDS 393, none read at all 367 (the memory rate).
// Two row tiles per wave would halve those reads but leave two waves per SIMD:
// 522 us.  OUT is stored past the caches (427 -> 409 us).
//
// The four real products of a complex one have sums of their own, joined at
// the end with OUT's old value: sums as long as the number of columns, as
// accurate as complex multiply-adds one after another (one sum for a part,
// twice as long, was off by 1.4 times as much).
template <typename T, int WC, int NW, bool LQ>
__global__ __launch_bounds__(NW * 64, LQ ? 4 : 3) void rotate_mfma_kernel(Cols<T> IN, const double* __restrict__ Q,
                                                                 int64_t rows, int accumulate, int CT, Cols<T> OUT) {
    using V = T __attribute__((ext_vector_type(2)));
    constexpr int KS = 4;   // instructions per half
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lc = lane & 15, lr = lane >> 4;
    const int K = IN.n, N = OUT.n;
    const int jg = int(blockIdx.y) * CT * kTile * WC;   // the workgroup's first column
    const int jw = (wave % CT) * kTile * WC;            // the wave's, from there
    const int64_t nrt = (rows + kTile - 1) / kTile;     // row tiles
    T* const outp = const_cast<T*>(OUT.base);

    extern __shared__ f64x2 lq[];   // [K rounded up to 4][ldq]
    const int ldq = CT * kTile * WC;
    if constexpr (LQ) {
        const int total = (K + 3) / 4 * 4 * ldq;
        for (int e = threadIdx.x; e < total; e += NW * 64) {
            const int k = e / ldq, j = jg + e - k * ldq;
            f64x2 v{0.0, 0.0};
            if (k < K && j < N) v = reinterpret_cast<const f64x2a*>(Q)[(size_t)k * N + j];
            lq[e] = v;
        }
        __syncthreads();
    }
    if (jg + jw >= N) return;
    int64_t oc[WC];
    const f64x2a* qc[WC];
#pragma unroll
    for (int w = 0; w < WC; ++w) {
        const int j = min(jg + jw + w * kTile + lc, N - 1);
        oc[w] = OUT.at(j);
        qc[w] = reinterpret_cast<const f64x2a*>(Q) + j;
    }
    for (int64_t rt = int64_t(blockIdx.x) * (NW / CT) + wave / CT; rt < nrt; rt += int64_t(gridDim.x) * (NW / CT)) {
        const int64_t r0 = rt * kTile;
        const int64_t row = (r0 + lc < rows ? r0 + lc : rows - 1) * IN.ld;
        struct Half {
            f64x2 x[KS];
        };
        auto load = [&](Half& h, int k0) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int k = k0 + 4 * s + lr;
                const bool ok = k < K;
                const f64x2 v = ld_c(IN.base, row + IN.at(ok ? k : K - 1));
                h.x[s] = f64x2{ok ? v.x : 0.0, ok ? v.y : 0.0};
            }
        };
        f64x4 rr[WC], ii[WC], ri[WC], ir[WC];
#pragma unroll
        for (int q = 0; q < WC; ++q) rr[q] = ii[q] = ri[q] = ir[q] = f64x4{0.0, 0.0, 0.0, 0.0};
        auto multiply = [&](const Half& h, int k0) {
            f64x2 b[KS][WC];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int k = k0 + 4 * s + lr;
                const bool ok = k < K;
#pragma unroll
                for (int q = 0; q < WC; ++q) {
                    if constexpr (LQ) {
                        // past the padded rows (not multiplied): any row
                        b[s][q] = lq[(k0 + 4 * s < K ? k : lr) * ldq + jw + q * kTile + lc];
                    } else {
                        const f64x2 v = qc[q][(size_t)(ok ? k : K - 1) * N];
                        b[s][q] = f64x2{ok ? v.x : 0.0, ok ? v.y : 0.0};
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < KS; ++s)
                if (k0 + 4 * s < K) {
#pragma unroll
                    for (int q = 0; q < WC; ++q) {
                        rr[q] = mfma(h.x[s].x, b[s][q].x, rr[q]);
                        ii[q] = mfma(h.x[s].y, b[s][q].y, ii[q]);
                        ri[q] = mfma(h.x[s].x, b[s][q].y, ri[q]);
                        ir[q] = mfma(h.x[s].y, b[s][q].x, ir[q]);
                    }
                }
        };
        Half A, B;
        load(A, 0);
        for (int k0 = 0; k0 < K; k0 += 8 * KS) {
            if (k0 + 4 * KS < K) load(B, k0 + 4 * KS);
            multiply(A, k0);
            if (k0 + 4 * KS < K) {
                if (k0 + 8 * KS < K) load(A, k0 + 8 * KS);
                multiply(B, k0 + 4 * KS);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t r = r0 + 4 * v + lr;
#pragma unroll
            for (int q = 0; q < WC; ++q)
                if (r < rows && jg + jw + q * kTile + lc < N) {
                    f64x2 y{rr[q][v] - ii[q][v], ri[q][v] + ir[q][v]};
                    if (accumulate) y += ld_c(OUT.base, r * OUT.ld + oc[q]);
                    __builtin_nontemporal_store(V{T(y.x), T(y.y)},
                                                reinterpret_cast<V*>(outp + 2 * (r * OUT.ld + oc[q])));
                }
        }
    }
}

// The same for few columns, one thread per entry of Y: bound by latency on
// small blocks and by its reads, which the threads of a row share through L1, on
// large ones (rotate_by_entry has the times).  The four real products have sums
// of their own, as above.
template <typename T>
__global__ __launch_bounds__(kTallBlock) void rotate_entry_kernel(const T* __restrict__ X, const double* __restrict__ Q,
                                                                  int64_t n, int nx, int ny, int accumulate,
                                                                  T* __restrict__ Y) {
    for (int64_t e = blockIdx.x * int64_t(kTallBlock) + threadIdx.x; e < n; e += int64_t(gridDim.x) * kTallBlock) {
        const int64_t r = (e >> 32) == 0 ? int64_t(uint32_t(e) / uint32_t(ny)) : e / ny;
        const int j = int(e - r * ny);
        f64x2 y{0.0, 0.0};
        if (accumulate) y = ld_c(static_cast<const T*>(Y), e);
        double rr = 0.0, ii = 0.0, ri = 0.0, ir = 0.0;
        for (int i = 0; i < nx; ++i) {
            const f64x2 u = ld_c(X, r * nx + i);
            const double qr = Q[(i * ny + j) * 2], qi = Q[(i * ny + j) * 2 + 1];
            rr += u.x * qr;
            ii += u.y * qi;
            ri += u.x * qi;
            ir += u.y * qr;
        }
        using V = T __attribute__((ext_vector_type(2)));
        *reinterpret_cast<V*>(Y + 2 * e) = V{T(y.x + (rr - ii)), T(y.y + (ri + ir))};
    }
}

template <typename T>
Cols<T> cols(const void* base, int64_t stride, int ld, int n, int lg) {
    return Cols<T>{static_cast<const T*>(base), stride, ld, n, lg};
}

int log2_of(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

template <class F>
hipError_t by_type(int dtype, F&& f) {
    return dtype == 0 ? f(double{}) : f(float{});
}

// Tiles of one (16 column) instruction per wave and side where a side has at
// most 16 columns, of two otherwise (a 64-column side is two waves' parts).
hipError_t gram_any(int dtype, int64_t rows, const void* X, const void* Y, int64_t stride, int ldx, int nx, int lgx,
                    int ldy, int ny, int lgy, int hermitian, int G, double* partials, double* out, hipStream_t s) {
    const int wx = nx <= kTile ? 1 : 2, wy = ny <= kTile ? 1 : 2;
    const int SX = nx > 2 * kTile ? 2 : 1, SY = ny > 2 * kTile ? 2 : 1;
    const int ntx = (nx + kSuper - 1) / kSuper, nty = (ny + kSuper - 1) / kSuper;
    const int ntiles = hermitian ? ntx * (ntx + 1) / 2 : ntx * nty;
    const hipError_t e = by_type(dtype, [&](auto tt) -> hipError_t {
        using T = decltype(tt);
        auto go = [&](auto kx, auto ky) {
            constexpr int WX = decltype(kx)::value, WY = decltype(ky)::value;
            const size_t lds = SX * SY < 4 ? size_t(SX * SY) * WX * WY * 8 * 64 * sizeof(double) : 0;
            hipLaunchKernelGGL((gram_mfma_kernel<T, WX, WY>), dim3(unsigned(G) * ntiles), dim3(kTallBlock), lds, s,
                               cols<T>(X, stride, ldx, nx, lgx), cols<T>(Y, stride, ldy, ny, lgy), rows, SX, SY, ntx,
                               nty, hermitian, G, partials);
        };
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        if (wx == 1 && wy == 1) go(I1{}, I1{});
        else if (wx == 1) go(I1{}, I2{});
        else if (wy == 1) go(I2{}, I1{});
        else go(I2{}, I2{});
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gram_sum_kernel, dim3((nx * ny + kTallBlock / 8 - 1) / (kTallBlock / 8)), dim3(kTallBlock), 0, s,
                       reinterpret_cast<const f64x2a*>(partials), G, nx, ny, hermitian, reinterpret_cast<f64x2a*>(out));
    return hipGetLastError();
}

// Coefficients in LDS while those of a workgroup's columns (at most 64) take at
// most 64 KiB, which covers every block of PV_MAX_NB columns: one 16-column
// tile per wave; four waves to a workgroup at up to 32 KiB, eight above, so a
// CU always holds sixteen waves.  Larger search spaces are bound by the matrix
// units and by the coefficient reads: two tiles per wave (128 x 128 columns,
// 1382400 rows: 3.8 ms, against 4.6 with one).
hipError_t rotate_any(int dtype, int64_t rows, const void* IN, int64_t in_stride, int ldi, int K, int lgi,
                      const double* Q, int accumulate, void* OUT, int64_t out_stride, int ldo, int N, int lgo,
                      hipStream_t s) {
    auto column_tiles = [&](int nct) { return nct >= 4 ? 4 : (nct >= 2 ? 2 : 1); };
    const int nct1 = (N + kTile - 1) / kTile;
    const size_t lds = size_t((K + 3) / 4 * 4) * column_tiles(nct1) * kTile * sizeof(f64x2);
    const int64_t rt = (rows + kTile - 1) / kTile;
    return by_type(dtype, [&](auto tt) -> hipError_t {
        using T = decltype(tt);
        auto go = [&](auto kc, auto kn, auto kl) {
            constexpr int WC = decltype(kc)::value, NW = decltype(kn)::value;
            constexpr bool LQ = decltype(kl)::value;
            const int nct = (nct1 + WC - 1) / WC, CT = column_tiles(nct);
            int64_t gx = (rt + NW / CT - 1) / (NW / CT);
            // walking workgroups fill the 256 CUs once
            if (LQ && gx > 4096 / NW) gx = 4096 / NW;
            const dim3 grid(unsigned(gx), unsigned((nct + CT - 1) / CT));
            hipLaunchKernelGGL((rotate_mfma_kernel<T, WC, NW, LQ>), grid, dim3(NW * 64), LQ ? lds : 0, s,
                               cols<T>(IN, in_stride, ldi, K, lgi), Q, rows, accumulate, CT,
                               cols<T>(OUT, out_stride, ldo, N, lgo));
        };
        using std::integral_constant;
        if (lds <= 32768) go(integral_constant<int, 1>{}, integral_constant<int, 4>{}, std::true_type{});
        else if (lds <= 65536) go(integral_constant<int, 1>{}, integral_constant<int, 8>{}, std::true_type{});
        else go(integral_constant<int, 2>{}, integral_constant<int, 4>{}, std::false_type{});
        return hipGetLastError();
    });
}

}  // namespace

// Row groups of a Gram (its partials are one matrix per group): two
// workgroups per CU, at most one per 16 rows.
int gram_grid(int64_t rows, int num_cus) {
    int64_t chunks = (rows + kGramRows - 1) / kGramRows;
    int64_t g = (int64_t)num_cus * 2;
    if (g > chunks) g = chunks;
    if (g < 1) g = 1;
    return int(g);
}

hipError_t launch_gram(int dtype, int64_t rows, int nx, int ny, const void* X, const void* Y, double* partials,
                       int grid, double* G, hipStream_t s) {
    return gram_any(dtype, rows, X, Y, 0, nx, nx, 31, ny, ny, 31, 0, grid, partials, G, s);
}

int block_gram_groups(int64_t rows, int nblk, int num_cus) {
    const int64_t chunks = (rows + kGramRows - 1) / kGramRows;
    int64_t g = (2 * (int64_t)num_cus + nblk - 1) / nblk;
    if (g > chunks) g = chunks;
    if (g < 1) g = 1;
    return int(g);
}

hipError_t launch_block_gram(int dtype, int64_t rows, int bw, int nblk, const void* A, const void* B, int64_t stride,
                             int hermitian, double* partials, int groups, double* G, hipStream_t s) {
    const int ns = bw * nblk, lg = log2_of(bw);
    return gram_any(dtype, rows, A, B, stride, bw, ns, lg, bw, ns, lg, hermitian, groups, partials, G, s);
}

hipError_t launch_rotate(int dtype, int64_t rows, int nx, int ny, const void* X, const double* Q, int accumulate,
                         void* Y, hipStream_t s) {
    if (rotate_by_entry(dtype, rows, nx, ny, accumulate != 0)) {
        const int64_t n = rows * ny, g = (n + kTallBlock - 1) / kTallBlock;
        return by_type(dtype, [&](auto tt) -> hipError_t {
            using T = decltype(tt);
            hipLaunchKernelGGL((rotate_entry_kernel<T>), dim3(unsigned(g < 8192 ? g : 8192)), dim3(kTallBlock), 0, s,
                               static_cast<const T*>(X), Q, n, nx, ny, accumulate, static_cast<T*>(Y));
            return hipGetLastError();
        });
    }
    return rotate_any(dtype, rows, X, 0, nx, nx, 31, Q, accumulate, Y, 0, ny, ny, 31, s);
}

hipError_t launch_block_rotate(int dtype, int64_t rows, int bw, int nin, int nout, const void* IN, int64_t in_stride,
                               const double* Q, void* OUT, int64_t out_stride, hipStream_t s) {
    const int lg = log2_of(bw);
    return rotate_any(dtype, rows, IN, in_stride, bw, nin * bw, lg, Q, 0, OUT, out_stride, bw, nout * bw, lg, s);
}

}  // namespace pv
