// Several Chebyshev steps of a 2D lattice in one pass.
//
// A step alone moves three vectors (five with an accumulator) through memory
// for some 30 operations per element, so on 2D lattices, where a walk along
// y needs no neighbour beside its own columns, TS steps go through one pass:
// level 0 is w_k, level t is w_{k+t}, and row r of level t is computed as soon
// as row r + 1 of level t - 1 is there.  A pass reads w_k, w_{k-1} (and the
// accumulator) and writes w_{k+TS-1}, w_{k+TS} (and the accumulator): four
// (six) vectors for TS steps instead of three (five) for one.
//
// One lane owns one site and column; the wave's 64 lanes are 64 / nb sites of
// an x tile with a halo of TS sites on both sides, computed redundantly, and
// a wave walks its rows alone: the two last rows of every level stay in
// registers, x neighbours come from other lanes, and there is neither LDS nor
// a barrier.  The stencil's coefficients are uniform, so they are scalars.
// Rows are loaded three iterations ahead.  The pass must not write what other
// waves read as halo: its outputs are other buffers than w_k and w_{k-1} (the
// accumulator has no halo and is updated in place).
//
// Measured: a propagation step of 64 terms on graphene 1024 x 1024 (complex128)
// 2000 -> 614 us, 56 us per pass of six steps against 31 us per step.  What
// bounds a pass is the wave's own instructions (one wave per SIMD, 1.4 us per row
// of six levels, of which 33 are computed for 21) more than the 208 MB it moves:
// 55 us with vectors of zeros.  Bounding the registers at 256
// for two waves spills: 12 us per step instead of 8.6 (four steps per pass).
#include "pv_sweep.hpp"

#include <algorithm>
#include <cmath>

namespace pv {
namespace {

constexpr int kPlaneMaxSteps = 6;

// The patterns with the field they have here: per site, per orbital.
struct PlaneGraphene2 : PatGraphene2 {
    static constexpr int VO = 1;
};
struct PlaneGraphene4 : PatGraphene4 {
    static constexpr int VO = 4;
};

template <typename T, typename VT>
struct PlaneArgs {
    const cplx<T>* x;        // w_k
    const cplx<T>* z;        // w_{k-1}; NULL: k = 0
    cplx<T>* y1;             // w_{k+TS-1}, w_{k+TS}; NULL: not stored
    cplx<T>* y2;
    const cplx<T>* acc_in;   // series: NULL with k = 0 (acc = eta[0] w_0 + ...)
    cplx<T>* acc_out;
    const VT* V;             // NULL: no field
    const double* coef;
    double* partials;        // moments: [TS][workgroups][nb][2] (<w,w>, Re <w,w'>)
    int Lx, Ly, px, py;
    int nb, lognb;
    int ntx, C, nyc;         // x tiles, rows per walk, walks per column
    double alpha1, alpha, beta;   // alpha1: of level 1
    int levels;              // levels that count (the last pass may have fewer than TS)
    double eta[2 * (kPlaneMaxSteps + 1)];   // eta[0] of w_0 (k = 0), eta[t] of level t
};

// Value of the lane nb lanes below (UP) or above (any value where there is
// none: such lanes' results reach the halo only); ONE: nb = 1, a data-parallel
// move instead of a permutation.
template <bool UP, bool ONE>
__device__ __forceinline__ int lane_shift(int v, int nb) {
    if constexpr (ONE) return __builtin_amdgcn_mov_dpp(v, UP ? 0x138 : 0x130, 0xf, 0xf, true);
    return UP ? __shfl_up(v, nb) : __shfl_down(v, nb);
}
template <bool UP, bool ONE>
__device__ __forceinline__ float lane_shift(float v, int nb) {
    return __int_as_float(lane_shift<UP, ONE>(__float_as_int(v), nb));
}
template <bool UP, bool ONE>
__device__ __forceinline__ double lane_shift(double v, int nb) {
    return __hiloint2double(lane_shift<UP, ONE>(__double2hiint(v), nb), lane_shift<UP, ONE>(__double2loint(v), nb));
}

// Raw buffers over a whole vector (below 2 GiB): a lane offset of kNone, or any
// offset into a buffer of length 0, loads zeros and stores nothing (2^31 is past
// every length, and neither the words of a chunk nor a row's offset carry it
// round to the start).  So lanes and rows outside the lattice, halo lanes and
// absent operands need no branches, and with no memory operation in a branch the
// compiler waits for exactly the loads that an iteration uses.
constexpr uint32_t kNone = 0x80000000u;
using Rsrc = __amdgpu_buffer_rsrc_t;
struct Row {
    Rsrc r;
    uint32_t at;   // the row's byte offset; 0 in a buffer of length 0, whose range check counts from it
};
struct Buf {
    const void* p;
    uint32_t bytes;
    __device__ __forceinline__ Row row(bool on, uint32_t at) const {
        const uint32_t n = on ? bytes : 0u;
        return Row{__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, int(n), 0x00027000), n ? at : 0u};
    }
};
template <typename X>
__device__ __forceinline__ X buf_ld(const Row& b, uint32_t off) {
    if constexpr (sizeof(X) == 16)
        return __builtin_bit_cast(X, __builtin_amdgcn_raw_buffer_load_b128(b.r, int(off), int(b.at), 0));
    else if constexpr (sizeof(X) == 8)
        return __builtin_bit_cast(X, __builtin_amdgcn_raw_buffer_load_b64(b.r, int(off), int(b.at), 0));
    else
        return __builtin_bit_cast(X, __builtin_amdgcn_raw_buffer_load_b32(b.r, int(off), int(b.at), 0));
}
// (Not past the caches: a wave stores the halves of a site one after the other,
// and lines leave L2 whole.  Stored past them, a graphene 1024 x 1024 pass of
// four steps took 65 us instead of 48.)
template <typename X>
__device__ __forceinline__ void buf_st(const Row& b, uint32_t off, X v) {
    using u32x2 = unsigned int __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(X) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b.r, int(off), int(b.at), 0);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b.r, int(off), int(b.at), 0);
}

template <class P, typename T, typename VT, int TS, bool KPM, bool ONE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1)))
void plane_kernel(PlaneArgs<T, VT> a) {
    constexpr int NO = P::NO;
    struct Site {
        cplx<T> v[NO];
    };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nb = ONE ? 1 : a.nb;
    const int c = lane & (nb - 1), sx = ONE ? lane : lane >> a.lognb;
    const int S = ONE ? 64 : 64 >> a.lognb;
    // workgroup b runs on XCD b % 8, which takes a contiguous eighth of the
    // items; an item is four x tiles of one walk
    const int tiles4 = (a.ntx + 3) / 4;
    const int items = tiles4 * a.nyc;
    const int per = (items + 7) / 8;
    const int item = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
    const int yc = item / tiles4;
    const int tile = (item - yc * tiles4) * 4 + wave;
    const bool live = int(blockIdx.x >> 3) < per && item < items && tile < a.ntx;

    double xx[TS], xy[TS];
#pragma unroll
    for (int t = 0; t < TS; ++t) xx[t] = xy[t] = 0.0;

    if (live) {
        const int y0 = yc * a.C, y1 = min(y0 + a.C, a.Ly);
        const int xt = tile * (S - 2 * TS) - TS;              // site of lane 0
        const int x = xt + sx;
        const bool inside = a.px || (x >= 0 && x < a.Lx);
        const bool owned = sx >= TS && sx < S - TS && x < a.Lx;
        int xm = x % a.Lx;
        if (xm < 0) xm += a.Lx;
        constexpr uint32_t ES = sizeof(cplx<T>);
        const uint32_t rowb = uint32_t(a.Lx) * uint32_t(NO * nb) * ES;   // bytes of a row
        const uint32_t vecb = rowb * uint32_t(a.Ly);
        uint32_t lo[NO], so[NO];                              // byte offsets in a row: loads, stores
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            const uint32_t e = uint32_t((xm * NO + o) * nb + c) * ES;
            lo[o] = inside ? e : kNone;
            so[o] = owned ? e : kNone;
        }
        constexpr int VO = P::VO;                             // field entries per site
        const uint32_t vrowb = uint32_t(a.Lx * VO) * uint32_t(sizeof(VT));
        const uint32_t vo = uint32_t(xm * VO) * uint32_t(sizeof(VT));
        const Buf bx{a.x, vecb}, bz{a.z, a.z ? vecb : 0u}, bi{a.acc_in, a.acc_in ? vecb : 0u}, bo{a.acc_out, vecb},
            b1{a.y1, a.y1 ? vecb : 0u}, b2{a.y2, a.y2 ? vecb : 0u}, bv{a.V, a.V ? vrowb * uint32_t(a.Ly) : 0u};

        // the stencil's off-diagonal entries and its real diagonal, uniform
        T cr[P::NT + 1][NO][NO], ci[P::NT + 1][NO][NO], dg[NO];
#pragma unroll
        for (int t = 0; t <= P::NT; ++t)
#pragma unroll
            for (int o = 0; o < NO; ++o)
#pragma unroll
                for (int q = 0; q < NO; ++q) {
                    cr[t][o][q] = T(a.coef[((t * NO + o) * NO + q) * 2]);
                    ci[t][o][q] = T(a.coef[((t * NO + o) * NO + q) * 2 + 1]);
                }
#pragma unroll
        for (int o = 0; o < NO; ++o) dg[o] = cr[P::NT][o][o] - T(a.beta);

        // what iteration i needs from memory: level 0 of row i; of the row
        // before it (i - dir) the predecessor, the accumulator and the field
        // (zeros where absent)
        struct Rows {
            Site x, z, acc;
            VT V[VO];
        };
        // row i wrapped (periodic) or -1 outside (open); i is at most TS <= Ly outside
        auto wrap = [&](int r) {
            const int w = r < 0 ? r + a.Ly : (r >= a.Ly ? r - a.Ly : r);
            return (r < 0 || r >= a.Ly) && !a.py ? -1 : w;
        };
        int rprev = -1;                                       // row before the next one loaded
        auto load = [&](Rows& R, int i, int dir) {
            const int ri = i >= y0 - TS && i < y1 + TS ? wrap(i) : -1, rp = rprev;
            rprev = ri;
            const uint32_t oi = uint32_t(max(ri, 0)) * rowb, op = uint32_t(max(rp, 0));
            const Row rx = bx.row(ri >= 0, oi), rz = bz.row(rp >= 0, op * rowb), rv = bv.row(rp >= 0, op * vrowb);
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                R.x.v[o] = buf_ld<cplx<T>>(rx, lo[o]);
                R.z.v[o] = buf_ld<cplx<T>>(rz, lo[o]);
            }
            if constexpr (!KPM) {
                const int ra = i - dir;
                const bool own = ra >= y0 && ra < y1;
                const Row rc = bi.row(own, uint32_t(ra) * rowb);
#pragma unroll
                for (int o = 0; o < NO; ++o) R.acc.v[o] = buf_ld<cplx<T>>(rc, so[o]);
            }
#pragma unroll
            for (int o = 0; o < VO; ++o) R.V[o] = buf_ld<VT>(rv, vo + o * uint32_t(sizeof(VT)));
        };

        Site P1[TS], P2[TS];     // the last two rows of level t, P1 the later one
        T Vr[TS][VO];            // field of the rows that levels 1 ... TS reach
        Site A[TS];              // accumulator of the row that level t reached (A[0]: unused)
        const cplx<T> zero{T(0), T(0)};
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int o = 0; o < NO; ++o) P1[t].v[o] = P2[t].v[o] = A[t].v[o] = zero;
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int o = 0; o < VO; ++o) Vr[t][o] = T(0);
        const int in_lane = inside ? -1 : 0;
        auto masked = [&](T v, int m) {
            if constexpr (sizeof(T) == 8) return __longlong_as_double(__double_as_longlong(v) & (int64_t)m);
            else return __int_as_float(__float_as_int(v) & m);
        };

        // Iteration of level-0 row i, walking up (DIR 1) or down (-1) the rows.
        // EDGE: the walk's halo leaves an open lattice, whose outside stays zero
        auto body = [&](const Rows& R, int i, auto edge, auto dir) {
            constexpr bool EDGE = decltype(edge)::value;
            constexpr int DIR = decltype(dir)::value;
#pragma unroll
            for (int t = TS - 1; t > 0; --t)
#pragma unroll
                for (int o = 0; o < VO; ++o) Vr[t][o] = Vr[t - 1][o];
#pragma unroll
            for (int o = 0; o < VO; ++o) Vr[0][o] = T(R.V[o]);
            Site ahead = R.x;    // of level t - 1, the row after the one that level t reaches
            Site carry;          // accumulator of that row before level t
            if constexpr (!KPM) {
                carry = R.acc;
                if (a.acc_in == nullptr) {
                    const T er = T(a.eta[0]), ei = T(a.eta[1]);
#pragma unroll
                    for (int o = 0; o < NO; ++o) {
                        const cplx<T> w = P1[0].v[o];
                        carry.v[o] = cplx<T>{er * w.re - ei * w.im, er * w.im + ei * w.re};
                    }
                }
            }
            Site z = R.z;        // that row of level t - 2
#pragma unroll
            for (int t = 1; t <= TS; ++t) {
                const int r = i - DIR * t;
                const Site behind = P2[t - 1], mid = P1[t - 1];
                Site left, right;
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    left.v[o] = cplx<T>{lane_shift<true, ONE>(mid.v[o].re, nb), lane_shift<true, ONE>(mid.v[o].im, nb)};
                    right.v[o] = cplx<T>{lane_shift<false, ONE>(mid.v[o].re, nb), lane_shift<false, ONE>(mid.v[o].im, nb)};
                }
                const T al = T(t == 1 ? a.alpha1 : a.alpha);
                Site nw;
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    const T d = dg[o] + Vr[t - 1][VO == 1 ? 0 : o];
                    T hr = d * mid.v[o].re;
                    T hi = d * mid.v[o].im;
#pragma unroll
                    for (int tb = 0; tb <= P::NT; ++tb)
#pragma unroll
                        for (int q = 0; q < NO; ++q) {
                            if (tb == P::NT && q == o) continue;
                            const int dx = tb < P::NT ? P::off[tb < P::NT ? tb : 0][0] : 0;
                            const int dy = DIR * (tb < P::NT ? P::off[tb < P::NT ? tb : 0][1] : 0);
                            const Site& src = dy < 0 ? behind : (dy > 0 ? ahead : (dx < 0 ? left : (dx > 0 ? right : mid)));
                            mac<T>(hr, hi, P::code[tb][o][q], cr[tb][o][q], ci[tb][o][q], src.v[q]);
                        }
                    nw.v[o] = cplx<T>{al * hr - z.v[o].re, al * hi - z.v[o].im};
                    if constexpr (EDGE) {
                        const int m = in_lane & (a.py || (r >= 0 && r < a.Ly) ? -1 : 0);
                        nw.v[o] = cplx<T>{masked(nw.v[o].re, m), masked(nw.v[o].im, m)};
                    }
                }
                const bool own = r >= y0 && r < y1;
                if constexpr (KPM) {
#pragma unroll
                    for (int o = 0; o < NO; ++o) {
                        const cplx<T> u = zero_unless(owned && own, mid.v[o]), w = zero_unless(owned && own, nw.v[o]);
                        xx[t - 1] += double(u.re) * double(u.re) + double(u.im) * double(u.im);
                        xy[t - 1] += double(u.re) * double(w.re) + double(u.im) * double(w.im);
                    }
                } else {
                    Site s = carry;
                    if (t <= a.levels) {
                        const T er = T(a.eta[2 * t]), ei = T(a.eta[2 * t + 1]);
#pragma unroll
                        for (int o = 0; o < NO; ++o)
                            s.v[o] = cplx<T>{carry.v[o].re + er * nw.v[o].re - ei * nw.v[o].im,
                                             carry.v[o].im + er * nw.v[o].im + ei * nw.v[o].re};
                    }
                    if (t < TS) {
                        carry = A[t];
                        A[t] = s;
                    } else {
                        const Row ro = bo.row(own, uint32_t(r) * rowb);
#pragma unroll
                        for (int o = 0; o < NO; ++o) buf_st(ro, so[o], s.v[o]);
                    }
                }
                if (t >= TS - 1) {
                    const Row ry = (t == TS ? b2 : b1).row(own, uint32_t(r) * rowb);
#pragma unroll
                    for (int o = 0; o < NO; ++o) buf_st(ry, so[o], nw.v[o]);
                }
                // level t - 1 moves on by a row
                z = behind;
                P2[t - 1] = mid;
                P1[t - 1] = ahead;
                ahead = nw;
            }
        };

        // three rows of loads in flight and three iterations per round, after
        // which the rows of every level are back in their registers
        auto walk = [&](auto edge, auto dir) {
            constexpr int DIR = decltype(dir)::value;
            Rows R0, R1, R2;
            int i = DIR > 0 ? y0 - TS : y1 - 1 + TS;
            int n = y1 - y0 + 2 * TS;
            load(R0, i, DIR);
            load(R1, i + DIR, DIR);
            load(R2, i + 2 * DIR, DIR);
            for (;; i += 3 * DIR, n -= 3) {
                body(R0, i, edge, dir);
                if (n == 1) break;
                load(R0, i + 3 * DIR, DIR);
                body(R1, i + DIR, edge, dir);
                if (n == 2) break;
                load(R1, i + 4 * DIR, DIR);
                body(R2, i + 2 * DIR, edge, dir);
                if (n == 3) break;
                load(R2, i + 5 * DIR, DIR);
            }
        };
        using Up = std::integral_constant<int, 1>;
        using Down = std::integral_constant<int, -1>;
        const bool edge = (!a.px && (xt < 0 || xt + S > a.Lx)) || (!a.py && (y0 < TS || y1 + TS > a.Ly));
        // neighbouring walks meet at their common rows at the same time (both
        // at their start or both at their end), so the second read of the halo
        // rows is an L2 hit
        if (yc & 1) {
            if (edge) walk(std::true_type{}, Down{});
            else walk(std::false_type{}, Down{});
        } else {
            if (edge) walk(std::true_type{}, Up{});
            else walk(std::false_type{}, Up{});
        }
    }

    if constexpr (KPM) {
        // lanes of the same column, then the four waves, in a fixed order
        __shared__ double red[kBlock / 64][TS][2][PV_MAX_NB_K];
#pragma unroll
        for (int t = 0; t < TS; ++t) {
            for (int m = nb; m < 64; m <<= 1) {
                xx[t] += __shfl_xor(xx[t], m);
                xy[t] += __shfl_xor(xy[t], m);
            }
            if (lane < nb) {
                red[wave][t][0][lane] = xx[t];
                red[wave][t][1][lane] = xy[t];
            }
        }
        __syncthreads();
        for (int k = threadIdx.x; k < TS * nb * 2; k += kBlock) {
            const int t = k / (2 * nb), cc = (k >> 1) % nb, h = k & 1;
            double s = 0.0;
            for (int w = 0; w < kBlock / 64; ++w) s += red[w][t][h][cc];
            a.partials[(((size_t)t * gridDim.x + blockIdx.x) * nb + cc) * 2 + h] = s;
        }
    }
}

int log2_of(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

// Tiles and walks of a pass of TS steps: one wave per SIMD of the 256 CUs (a
// wave's registers leave room for no more), so walks as long as 256
// workgroups of four allow.  us per pass of a series, graphene-2 complex128, TS =
// 6: 1024 x 1024 in 21 rows per walk 56 (taken), 16 83, 32 69, 42 83; 2048 x 2048
// in 82 rows 201 (taken), 40 263, 120 251: longer walks leave SIMDs idle, shorter
// ones take two rounds and pay their halos twice.
void plane_shape(const SweepParams& p, int TS, int& ntx, int& C, int& nyc, int& grid) {
    const int S = 64 / p.nb, own = S - 2 * TS;
    ntx = int((p.L[0] + own - 1) / own);
    const int tiles4 = (ntx + 3) / 4;
    int walks = 256 / tiles4;
    if (walks < 1) walks = 1;
    C = int((p.L[1] + walks - 1) / walks);
    nyc = int((p.L[1] + C - 1) / C);
    grid = 8 * ((tiles4 * nyc + 7) / 8);
}

template <class P, typename T, typename VT, int TS, bool KPM, bool ONE>
hipError_t plane_go(const SweepParams& p, const PlanePass& q, hipStream_t s) {
    PlaneArgs<T, VT> a;
    a.x = static_cast<const cplx<T>*>(q.x);
    a.z = static_cast<const cplx<T>*>(q.z);
    a.y1 = static_cast<cplx<T>*>(q.y1);
    a.y2 = static_cast<cplx<T>*>(q.y2);
    a.acc_in = static_cast<const cplx<T>*>(q.acc_in);
    a.acc_out = static_cast<cplx<T>*>(q.acc_out);
    a.V = p.field == 1 ? static_cast<const VT*>(p.V) : nullptr;
    a.coef = p.coef;
    a.partials = q.partials;
    a.Lx = int(p.L[0]);
    a.Ly = int(p.L[1]);
    a.px = p.periodic[0] != 0;
    a.py = p.periodic[1] != 0;
    a.nb = p.nb;
    a.lognb = log2_of(p.nb);
    int grid;
    plane_shape(p, TS, a.ntx, a.C, a.nyc, grid);
    a.alpha1 = q.alpha1;
    a.alpha = q.alpha;
    a.beta = p.beta;
    a.levels = q.levels;
    for (int k = 0; k < 2 * (kPlaneMaxSteps + 1); ++k) a.eta[k] = q.eta && k <= 2 * q.levels + 1 ? q.eta[k] : 0.0;
    hipLaunchKernelGGL((plane_kernel<P, T, VT, TS, KPM, ONE>), dim3(grid), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

// f(pattern, TS, nb == 1) for the instance of (family, dtype, nb) with TS steps.
template <class F>
hipError_t plane_instance(int family, int dtype, int nb, int TS, F&& f) {
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I6 = std::integral_constant<int, 6>;
    if (family == FAM_GRAPHENE2) {
        if (nb == 1 && TS == 6) return f(Tag<PlaneGraphene2>{}, I6{}, std::true_type{});
        if (nb == 1 && TS == 4) return f(Tag<PlaneGraphene2>{}, I4{}, std::true_type{});
        if (TS == 4) return f(Tag<PlaneGraphene2>{}, I4{}, std::false_type{});
    } else if (family == FAM_GRAPHENE4) {
        if (TS != (dtype == 0 ? 3 : 4)) return hipErrorInvalidValue;
        if (dtype == 0)
            return nb == 1 ? f(Tag<PlaneGraphene4>{}, I3{}, std::true_type{})
                           : f(Tag<PlaneGraphene4>{}, I3{}, std::false_type{});
        return nb == 1 ? f(Tag<PlaneGraphene4>{}, I4{}, std::true_type{})
                       : f(Tag<PlaneGraphene4>{}, I4{}, std::false_type{});
    }
    return hipErrorInvalidValue;
}

}  // namespace

namespace {

// Times (us) of `steps` steps as passes of TS steps and as sweeps, fitted to 250
// lattices of 4 KB to 100 MB per vector with 2 to 32 steps each (12% rms both).
// A pass is bound by a wave's instructions per row, one or (where the registers
// allow two) two rounds of workgroups at once, or by its memory; a sweep by its
// launch, its streams, and the 256-number tiles that its rows leave empty.
double plane_time(const SweepParams& p, int TS, int steps, bool kpm, double bytes) {
    const bool g2 = p.family == FAM_GRAPHENE2, c128 = p.dtype == 0;
    int ntx, C, nyc, grid;
    plane_shape(p, TS, ntx, C, nyc, grid);
    const double items = double((ntx + 3) / 4) * nyc, levels = C + 2 * TS;
    // us per row of a wave
    const double row = !g2 ? (c128 ? (kpm ? 1.11 : 1.46) : 1.17)
                           : (c128 ? (TS == 6 ? (kpm ? 0.90 : 1.12) : (kpm ? 0.78 : 0.95)) : (TS == 6 ? 0.83 : 0.79));
    const bool two = g2 && !(c128 && TS == 6);
    const double rounds = two ? std::max(1.0, items / 512) : std::ceil(items / 256);
    const double walk = rounds * (levels + 2.5) * row, mem = (kpm ? 5.8e-7 : 8.1e-7) * bytes * levels / C;
    const int passes = (steps + TS - 1) / TS;
    return passes * (0.9 + std::pow(std::pow(walk, 4) + std::pow(mem, 4), 0.25)) + (kpm ? 3.8 : 0.0);
}
double sweeps_time(const SweepParams& p, int steps, bool kpm, double bytes) {
    const bool c128 = p.dtype == 0, large = bytes >= double(1 << 20) * (c128 ? 16 : 8);   // staged
    const int64_t rowel = p.L[0] * p.n_orb * p.nb, tile = large && !c128 ? 512 : 256;
    const double tiles = double((rowel + tile - 1) / tile * tile) * double(p.L[1]), part = double((p.L[1] + 7) / 8);
    const double streams = (kpm ? 3.0 : 11.0 / 3.0) * (large ? (part + 1.3) / part : 1.0);
    return steps * (4.0 + streams * bytes * 1.23e-7 + tiles * (large ? 2e-6 : 4e-6)) + (kpm ? 7.7 : 0.0);
}

}  // namespace

// Which runs take passes.  Fields generated in the kernel and complex diagonals
// are left out (registers), as are the moments of complex64 vectors (their FP64
// dots keep the sweeps' rounding) and blocks of more than four columns, whose
// halo would be most of a wave.  The others take them where they are estimated
// to be faster: a last pass computes all of its levels, and lattices of few
// sites along x leave most of a wave's lanes and of a workgroup's waves idle.
// Measured (us, passes | sweeps): series of 32 terms, one complex128 column:
// graphene-2 12x10 105 | 134, 512x512 167 | 279, 2000x1500 812 | 1954, 8x20000
// 638 | 808; graphene-4 512x512 383 | 458, 8x20000 1277 | 858; of 4 terms 200x150
// 30 | 21; moments, 8 steps: graphene-4 200x150 40 | 49, 8x20000 with four columns
// 297 | 238.  Four-orbital complex128 series below 4 MiB per vector never gain
// (32 terms, 60x1000 200 | 171, 16x512 with four columns 182 | 164).
int plane_steps(const SweepParams& p, int steps, bool kpm) {
    const bool g2 = p.family == FAM_GRAPHENE2, g4 = p.family == FAM_GRAPHENE4;
    if (!(g2 || g4) || p.nb > 4 || p.kernel != 0 || !p.real_diag || p.field == 2 || steps < 2) return 0;
    if (kpm && p.dtype != 0) return 0;
    if (p.field == 1 && p.pot_mode != (g2 ? 1 : 2)) return 0;
    if (p.L[1] < kPlaneMaxSteps + 2) return 0;
    const double bytes = double(p.L[0]) * double(p.L[1]) * p.n_orb * p.nb * (p.dtype == 0 ? 16 : 8);
    if (bytes >= 2147483648.0) return 0;   // 32-bit offsets of the buffers
    if (g4 && !kpm && p.dtype == 0 && bytes < 4194304.0) return 0;   // the registers of one wave per SIMD
    int ts = g4 && p.dtype == 0 ? 3 : 4;
    if (g2 && p.nb == 1) {
        auto cost = [&](int n) { return ((steps + n - 1) / n) * (n + 2.7); };
        if (cost(6) <= cost(4)) ts = 6;
    }
    return 0.9 * plane_time(p, ts, steps, kpm, bytes) < sweeps_time(p, steps, kpm, bytes) ? ts : 0;
}

int plane_grid(const SweepParams& p, int TS) {
    int ntx, C, nyc, grid;
    plane_shape(p, TS, ntx, C, nyc, grid);
    return grid;
}

hipError_t launch_plane(const SweepParams& p, int TS, const PlanePass& q, hipStream_t s) {
    return plane_instance(p.family, p.dtype, p.nb, TS, [&](auto tp, auto tn, auto one) -> hipError_t {
        using P = typename decltype(tp)::type;
        constexpr int N = decltype(tn)::value;
        constexpr bool ONE = decltype(one)::value;
        if (q.partials) {
            if constexpr (N != 4 || P::NO == 2) {
                if (p.dtype == 0) return plane_go<P, double, double, N, true, ONE>(p, q, s);
            }
            return hipErrorInvalidValue;
        }
        if (p.dtype == 0) {
            if constexpr (N != 4 || P::NO == 2) return plane_go<P, double, double, N, false, ONE>(p, q, s);
            return hipErrorInvalidValue;
        }
        if constexpr (N != 3) {
            return p.vtype == 0 ? plane_go<P, float, double, N, false, ONE>(p, q, s)
                                : plane_go<P, float, float, N, false, ONE>(p, q, s);
        }
        return hipErrorInvalidValue;
    });
}

}  // namespace pv
