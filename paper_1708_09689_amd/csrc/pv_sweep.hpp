#pragma once
// HIP sweep kernels for gfx950 (MI355X) and their launchers, as templates
// over the stencil family: the matrix-free stencil sweep with fused
// Chebyshev epilogues and partial dot products.  Each family is compiled in
// a translation unit of its own (pv_fam_*.hip), so the families build in
// parallel; internal to the library, every includer gets its own copies.
//
// The sweep evaluates, per column c of an nb-wide block (Sec. 3.2, generated
// spMVM listing, with scale_h = alpha, shift_h = beta, scale_z = gamma):
//     y = alpha (H x - beta x) + gamma z
// where H acts matrix-free through the stencil blocks of the lattice
// (Sec. 3.2 DSL: one block per neighbour offset), and optionally
//     acc = etaz z + etax x + eta y   or   acc += ...   (Chebyshev series, Sec. 4)
//     partial sums of <x,x>, <x,y>, <y,y>           (fused dots, Sec. 3.2/3.5)
//
// Work decomposition: one lane owns one element (site s, orbital row o,
// column c) of the output block.  A workgroup of 256 lanes covers 256
// consecutive elements, so every load of a neighbour's entries is a fully
// coalesced wave-wide access of 64 consecutive complex numbers (shifted by
// the neighbour's site offset; entries of other orbitals of the same site
// are a fixed lane-dependent offset within the same cache lines).  Because
// n_orb * nb divides 256, a lane keeps the same (o, c) for the whole launch:
// its row's stencil coefficients live in registers.  Block structure is
// compiled in per family: for every neighbour block and entry kind (real,
// imaginary, complex) the kernel carries "slots" -- the k-th nonzero of that
// kind in the lane's row -- so the TI stencil costs 12 two-FMA complex
// updates per row.  The grid is persistent, sized from the occupancy of the
// instantiation, and XCD-aware: workgroup b runs on XCD b % 8, each XCD takes
// one contiguous eighth of the tiles, and its resident workgroups sweep that
// range together, so the +-y / +-z neighbour rows they read were fetched by
// the same XCD shortly before (same L2).
#include "pv_kernels.hpp"

#ifndef PV_RTC
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <utility>
#endif

namespace pv {
namespace {

template <typename T>
struct alignas(2 * sizeof(T)) cplx {
    T re, im;
};

template <int V>
struct IntC {
    static constexpr int value = V;
};

template <int N, int I = 0, typename F>
__device__ __forceinline__ void sfor(F&& f) {
    if constexpr (I < N) {
        f(IntC<I>{});
        sfor<N, I + 1>(f);
    }
}

constexpr int kBlock = 256;

template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
using u32x4 = unsigned int __attribute__((ext_vector_type(4)));

// Round-up division by a runtime constant (Granlund & Montgomery): exact for
// every 32-bit numerator.
struct FastDiv {
    uint32_t d, m, l;
};

inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f{d, 0u, 0u};
    if (d > 1) {
        uint32_t l = 0;
        while ((1ull << l) < d) ++l;
        f.l = l;
        f.m = uint32_t((((1ull << 32) * ((1ull << l) - d)) / d) + 1);
    }
    return f;
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) {
    if (f.d == 1) return n;
    const uint32_t t = __umulhi(n, f.m);
    return (t + ((n - t) >> 1)) >> (f.l - 1);
}

template <typename T, typename VT>
struct KArgs {
    const cplx<T>* x;
    const cplx<T>* z;
    cplx<T>* y;
    const cplx<T>* acc_in;
    cplx<T>* acc_out;
    const cplx<T>* zsrc;    // z, or x when no column reads z (a valid dummy)
    const cplx<T>* asrc;    // acc_in, or x when not accumulating
    const VT* V;
    int field;              // 0 none, 1 stored array V, 2 counter-based generator
    uint64_t rng_seed;
    double rng_W;
    const cplx<T>* gw0;     // adjoint terms: w_{k-1}, w_k, w_{k+1} (or NULL)
    const cplx<T>* gw1;
    const cplx<T>* gw2;
    const double* gcoef;    // [3][nb] complex coefficients of the gw terms
    double* grad;           // on-site field gradient
    double gx, gy;
    int ggroup;             // lanes per gradient entry: n_orb*nb (site field) or nb (orbital field)
    const double* coef;
    const int* offs;
    const double* colp;
    double* partials;
    int64_t n_elem, ntiles;
    int tpb;
    // traversal: XCD part k (rows y in [Ly k/8, Ly (k+1)/8), all z) is swept
    // in slabs of BY rows, each slab plane by plane, each plane row by row
    const cplx<T>* zero_row;   // rowel zeros: neighbour rows dropped by open BCs read here
    int rowel, ntx, BY;
    FastDiv fd_ntx, fd_slab, fd_pf;
    int Lx, Ly, Lz;
    int px, py, pz;
    int nb, lognb, logsite;
    int n_terms, pot_mode;
    double alpha, beta, gamma;
    double eta_re, eta_im, etax_re, etax_im, etaz_re, etaz_im;
    unsigned ep;
    // staged traversal (staged_kernel): column tiles of one row walked along
    // the outer dimension w; m is the middle dimension (y in 3D, none in 2D)
    int st_site, st_seg, st_nxs;   // elements per site, ring row length, column tiles per row
    int st_Lm, st_Lw, st_pm, st_pw;
    int st_rm, st_rw, st_ywalk;    // rows from one m (w) to the next; 1: w is y and m is z
    int st_C, st_Bm, st_parts;     // planes per walk, strip height, 8 XCD parts or 1
};

template <typename T>
__device__ __forceinline__ void mac(T& ar, T& ai, unsigned char k, T cr, T ci, cplx<T> v) {
    if (k == CR) { ar += cr * v.re; ai += cr * v.im; }
    else if (k == CI) { ar -= ci * v.im; ai += ci * v.re; }
    else if (k == CC) { ar += cr * v.re - ci * v.im; ai += cr * v.im + ci * v.re; }
}

// Counter-based generator of the on-the-fly field (SplitMix64, Steele, Lea
// and Flood 2014): output i + 1 of the stream seeded with `seed`, i.e. the
// mixing function applied to seed + (i + 1) * golden gamma.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// On-site field value at index i (site, or orbital row for per-orbital
// fields): the stored array, or W (u - 1/2) with u the generator's top 53
// bits times 2^-53 -- u - 1/2 is exact, so the value is one rounded product.
template <typename T, typename VT>
__device__ __forceinline__ T field_at(const KArgs<T, VT>& a, int64_t i) {
    if (a.field == 2) {
        const double u = double(splitmix64_at(a.rng_seed, uint64_t(i)) >> 11) * 0x1.0p-53;
        return T(a.rng_W * (u - 0.5));
    }
    return T(a.V[i]);
}

// Slots of a compiled family: for block t (t == NT: off-diagonal part of the
// on-site block) and entry kind, slot k holds the k-th nonzero of that kind
// in each row o (q[o] = its column, -1 if the row has fewer).
template <class P>
struct Slots {
    static constexpr int MAX = MAX_SLOTS_K;
    int n = 0;
    int t[MAX] = {};
    unsigned char kind[MAX] = {};
    signed char q[MAX][4] = {};
    bool same[MAX] = {};   // every row's entry sits in its own orbital (orbital offset 0)
    constexpr Slots() {
        constexpr int NO = P::NO;
        for (int tt = 0; tt <= P::NT; ++tt)
            for (int kd = 1; kd <= 3; ++kd) {
                int K = 0;
                for (int o = 0; o < NO; ++o) {
                    int cnt = 0;
                    for (int qq = 0; qq < NO; ++qq)
                        if (!(tt == P::NT && qq == o) && P::code[tt][o][qq] == kd) ++cnt;
                    if (cnt > K) K = cnt;
                }
                for (int k = 0; k < K; ++k) {
                    t[n] = tt;
                    kind[n] = (unsigned char)kd;
                    for (int o = 0; o < 4; ++o) q[n][o] = -1;
                    for (int o = 0; o < NO; ++o) {
                        int cnt = 0;
                        for (int qq = 0; qq < NO; ++qq)
                            if (!(tt == P::NT && qq == o) && P::code[tt][o][qq] == kd) {
                                if (cnt == k) q[n][o] = (signed char)qq;
                                ++cnt;
                            }
                    }
                    same[n] = true;
                    for (int o = 0; o < NO; ++o)
                        if (q[n][o] >= 0 && q[n][o] != o) same[n] = false;
                    ++n;
                }
            }
    }
};

// Generic family descriptor: NO orbitals, runtime offsets, dense blocks.
// SH (every pattern's SIDE_HALO): the staged kernel loads the side rows with
// the x halo (stencils with hops that have a y and an x step).
template <int NO_, bool SH = false>
struct PatGeneric {
    static constexpr int FAMILY = FAM_GENERIC, NO = NO_, NT = 0, DIM = 3;
    static constexpr bool SIDE_HALO = SH, SIDE_W = false;
    static constexpr int off[1][3] = {{0, 0, 0}};
    static constexpr unsigned char code[1][NO_][NO_] = {};   // no compiled slots
};

template <class P>
constexpr bool side_halo() {
    return P::SIDE_HALO;
}

template <typename T>
__device__ __forceinline__ cplx<T> ld_nt(const cplx<T>* p) {
    const vec2<T> v = __builtin_nontemporal_load(reinterpret_cast<const vec2<T>*>(p));
    return cplx<T>{v.x, v.y};
}

template <typename T>
__device__ __forceinline__ void st_nt(cplx<T>* p, T re, T im) {
    vec2<T> v;
    v.x = re;
    v.y = im;
    __builtin_nontemporal_store(v, reinterpret_cast<vec2<T>*>(p));
}

// Loads at a 32-bit byte offset from a (workgroup-uniform) row pointer.
template <typename T>
__device__ __forceinline__ cplx<T> ld_row(const cplx<T>* row, uint32_t boff) {
    return *reinterpret_cast<const cplx<T>*>(reinterpret_cast<const char*>(row) + boff);
}

template <typename T>
__device__ __forceinline__ cplx<T> ld_row_nt(const cplx<T>* row, uint32_t boff) {
    return ld_nt(reinterpret_cast<const cplx<T>*>(reinterpret_cast<const char*>(row) + boff));
}

// acc += eta v
template <typename T>
__device__ __forceinline__ void add_term(T& ar, T& ai, T er, T ei, T vr, T vi) {
    ar = ar + er * vr - ei * vi;
    ai = ai + er * vi + ei * vr;
}

// Epilogue shared by every family: y = alpha h + gamma z (+ sum_j g_j w_j),
// store / accumulate, FP64 partial dots of (x, y), and the on-site field
// gradient.  zv and av were loaded at the top of the element
// (unconditionally, from a valid address) so that every load of an element
// is in flight at the same time; gamma == 0 selects zero instead of
// gamma * z, so z is never used for such columns.
//
// Adjoint options (Clenshaw-type recurrences for gradients):
//   EP_GTERMS  y += sum_{j=0..2} gcoef[j][c] * gw_j[e]   (complex coefficients;
//              gw_j == NULL skips the term)
//   EP_GRAD    grad[site or row] += gx Re(conj(x) gw_1) + gy Re(conj(y) gw_0),
//              summed over the site's (or row's) lanes with a fixed xor tree
//              and written by one lane, read-modify-write (no atomics)
template <typename T, typename VT>
__device__ __forceinline__ void epilogue_ep(const KArgs<T, VT>& a, const unsigned ep, int64_t e, int64_t gidx,
                                            int glane, cplx<T> xc, cplx<T> zv, cplx<T> av, T hr, T hi, T alT, T gaT,
                                            T er, T ei, int c, double& dxx, double& dxr, double& dxi,
                                            double& dyy) {
    T yr = alT * hr, yi = alT * hi;
    yr += (gaT != T(0)) ? gaT * zv.re : T(0);
    yi += (gaT != T(0)) ? gaT * zv.im : T(0);
    cplx<T> gv[3] = {{T(0), T(0)}, {T(0), T(0)}, {T(0), T(0)}};
    if (ep & (EP_GTERMS | EP_GRAD)) {
        const cplx<T>* gws[3] = {a.gw0, a.gw1, a.gw2};
        for (int j = 0; j < 3; ++j)
            if (gws[j] != nullptr) gv[j] = ld_nt(gws[j] + e);
    }
    if (ep & EP_GTERMS) {
        for (int j = 0; j < 3; ++j) {
            const T cr = T(a.gcoef[(j * a.nb + c) * 2]), ci = T(a.gcoef[(j * a.nb + c) * 2 + 1]);
            yr += cr * gv[j].re - ci * gv[j].im;
            yi += cr * gv[j].im + ci * gv[j].re;
        }
    }
    if (ep & EP_STORE_Y) st_nt(a.y + e, yr, yi);
    if (ep & (EP_ACC_INIT | EP_ACC_ADD)) {
        T ar = (ep & EP_ACC_ADD) ? av.re : T(0), ai = (ep & EP_ACC_ADD) ? av.im : T(0);
        if (ep & EP_ACC_Z) add_term(ar, ai, T(a.etaz_re), T(a.etaz_im), zv.re, zv.im);
        if (ep & EP_ACC_X) add_term(ar, ai, T(a.etax_re), T(a.etax_im), xc.re, xc.im);
        add_term(ar, ai, er, ei, yr, yi);
        st_nt(a.acc_out + e, ar, ai);
    }
    if (ep & (EP_DOTS | EP_MOMENTS)) {
        const double xr = double(xc.re), xi = double(xc.im);
        const double dyr = double(yr), dyi = double(yi);
        dxx += xr * xr + xi * xi;
        dxr += xr * dyr + xi * dyi;
        if (ep & EP_DOTS) {
            dxi += xr * dyi - xi * dyr;
            dyy += dyr * dyr + dyi * dyi;
        }
    }
    if (ep & EP_GRAD) {
        double g = a.gx * (double(xc.re) * double(gv[1].re) + double(xc.im) * double(gv[1].im)) +
                   a.gy * (double(yr) * double(gv[0].re) + double(yi) * double(gv[0].im));
        for (int m = 1; m < a.ggroup; m <<= 1) g += __shfl_xor(g, m);
        if (glane == 0) a.grad[gidx] += g;
    }
}

template <typename T, typename VT>
__device__ __forceinline__ void epilogue(const KArgs<T, VT>& a, int64_t e, int64_t gidx, int glane, cplx<T> xc,
                                         cplx<T> zv, cplx<T> av, T hr, T hi, T alT, T gaT, T er, T ei, int c,
                                         double& dxx, double& dxr, double& dxi, double& dyy) {
    epilogue_ep(a, a.ep, e, gidx, glane, xc, zv, av, hr, hi, alT, gaT, er, ei, c, dxx, dxr, dxi, dyy);
}

template <typename T>
__device__ __forceinline__ cplx<T> zero_unless(bool ok, cplx<T> v) {
    return cplx<T>{ok ? v.re : T(0), ok ? v.im : T(0)};
}

#ifndef PV_SWEEP_WAVES_PER_EU
#define PV_SWEEP_WAVES_PER_EU 1
#endif
#ifndef PV_STAGED_WAVES_PER_EU
#define PV_STAGED_WAVES_PER_EU 2
#endif


// Row (y + dy, z + dz) of row (y, z), wrapped along periodic dimensions;
// false when an open boundary drops it.  Uniform over a tile.
template <typename A>
__device__ __forceinline__ bool neighbour_row(const A& a, int y, int z, int dy, int dz, int& row) {
    int yn = y + dy, zn = z + dz;
    bool ok = true;
    if (dy) {
        const bool lo = yn < 0, hi = yn >= a.Ly;
        ok = ok && (a.py || !(lo || hi));
        yn += lo ? a.Ly : (hi ? -a.Ly : 0);
    }
    if (dz) {
        const bool lo = zn < 0, hi = zn >= a.Lz;
        ok = ok && (a.pz || !(lo || hi));
        zn += lo ? a.Lz : (hi ? -a.Lz : 0);
    }
    row = zn * a.Ly + yn;
    return ok;
}

__device__ __forceinline__ FastDiv make_fastdiv_dev(uint32_t d) {
    FastDiv f{d, 0u, 0u};
    if (d > 1) {
        const uint32_t l = 32u - __clz(d - 1u);
        f.l = l;
        f.m = uint32_t((((1ull << 32) * ((1ull << l) - d)) / d) + 1);
    }
    return f;
}

// Element offset of the x-neighbour (x + dx) inside its row, relative to the
// lane's own element xe; false when an open boundary drops it.
template <typename A>
__device__ __forceinline__ bool x_shift(const A& a, int x, int dx, int& dxe) {
    const int site = 1 << a.logsite;
    if (dx == 0) { dxe = 0; return true; }
    const int xn = x + dx;
    if (xn < 0) { dxe = (a.Lx - 1) * site; return a.px; }
    if (xn >= a.Lx) { dxe = -(a.Lx - 1) * site; return a.px; }
    dxe = dx * site;
    return true;
}

// Per-lane data of a compiled family: for every slot the complex coefficient
// of the lane's row and the element offset of the partner orbital inside the
// site (zero coefficient where the row has fewer entries of that kind).
template <class P, typename T, int NS, int NA>
__device__ __forceinline__ void slot_coefficients(const double* coef, int o, int nb, T (&cre)[NA], T (&cim)[NA],
                                                  int (&dq)[NA]) {
    constexpr int NO = P::NO;
    static constexpr Slots<P> S{};
    sfor<NS>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        int q = S.q[j][0];
        if constexpr (NO > 1) { if (o == 1) q = S.q[j][1]; }
        if constexpr (NO > 2) { if (o == 2) q = S.q[j][2]; if (o == 3) q = S.q[j][3]; }
        if (q >= 0) {
            const double* e = coef + ((S.t[j] * NO + o) * NO + q) * 2;
            cre[j] = T(e[0]);
            cim[j] = T(e[1]);
            dq[j] = (q - o) * nb;
        } else {
            cre[j] = T(0);
            cim[j] = T(0);
            dq[j] = 0;
        }
    });
}

// The work of one workgroup: tiles [t0, t1) of the part of the lattice made of
// rows y in [y0, y0 + ny) (all z), swept slab by slab; partial dots go to
// partials[b_out].
template <class P, typename T, typename VT>
__device__ __forceinline__ void sweep_block(const KArgs<T, VT>& a, int b_out, int y0, int ny, int64_t t0,
                                            int64_t t1) {
    constexpr int NO = P::NO;
    const int tid = threadIdx.x;
    const int nb = a.nb;
    const int c = tid & (nb - 1);
    const int o = (tid >> a.lognb) & (NO - 1);

    double al = a.alpha, be = a.beta, ga = a.gamma;
    if (a.colp != nullptr) {
        al = a.colp[3 * c];
        be = a.colp[3 * c + 1];
        ga = a.colp[3 * c + 2];
    }
    const T alT = T(al), beT = T(be), gaT = T(ga);
    const T er = T(a.eta_re), ei = T(a.eta_im);

    // diagonal of the on-site block for this lane's row
    const int nt_onsite = (P::FAMILY != FAM_GENERIC) ? P::NT : a.n_terms;
    const T dgr = T(a.coef[(((size_t)nt_onsite * NO + o) * NO + o) * 2]);
    const T dgi = T(a.coef[(((size_t)nt_onsite * NO + o) * NO + o) * 2 + 1]);

    double dxx = 0.0, dxr = 0.0, dxi = 0.0, dyy = 0.0;

    // per-lane slot data of compiled families
    static constexpr Slots<P> S{};
    constexpr int NS = (P::FAMILY != FAM_GENERIC) ? S.n : 0;
    T cre[NS > 0 ? NS : 1], cim[NS > 0 ? NS : 1];
    int dq[NS > 0 ? NS : 1];
    slot_coefficients<P, T, NS>(a.coef, o, nb, cre, cim, dq);

    // generic stencils: the nonzero entries of every block row (row starts,
    // columns, values; the host packs them after the offsets and the dense
    // blocks), staged in LDS once per workgroup
    constexpr int GMAX = (PV_MAX_TERMS_K + 1) * NO * NO;
    __shared__ int g_ptr[P::FAMILY == FAM_GENERIC ? (PV_MAX_TERMS_K + 1) * NO + 1 : 1];
    __shared__ int g_col[P::FAMILY == FAM_GENERIC ? GMAX : 1];
    __shared__ cplx<T> g_val[P::FAMILY == FAM_GENERIC ? GMAX : 1];
    if constexpr (P::FAMILY == FAM_GENERIC) {
        const int nptr = (a.n_terms + 1) * NO + 1;
        const int* gp = a.offs + 3 * a.n_terms;
        const int nnz = gp[nptr - 1];
        const double* gv = a.coef + (size_t)(a.n_terms + 1) * NO * NO * 2;
        for (int i = tid; i < nptr; i += kBlock) g_ptr[i] = gp[i];
        for (int i = tid; i < nnz; i += kBlock) {
            g_col[i] = gp[nptr + i];
            g_val[i] = cplx<T>{T(gv[2 * i]), T(gv[2 * i + 1])};
        }
        __syncthreads();
    }

    constexpr uint32_t ES = sizeof(cplx<T>);
    for (int64_t t = t0; t < t1; ++t) {
        // tile -> (row, x-tile): uniform over the workgroup.  Part k is swept
        // in slabs of BY rows; a slab plane by plane (z), a plane row by row.
        const uint32_t tt32 = uint32_t(t);
        const uint32_t slab_tiles = uint32_t(a.ntx) * uint32_t(a.BY) * uint32_t(a.Lz);
        const uint32_t yb = fdiv(tt32, a.fd_slab);
        const uint32_t rr = tt32 - yb * slab_tiles;
        const int by = min(a.BY, ny - int(yb) * a.BY);
        const uint32_t ptiles = uint32_t(a.ntx) * uint32_t(by);
        const uint32_t zz = (by == a.BY) ? fdiv(rr, a.fd_pf) : fdiv(rr, make_fastdiv_dev(ptiles));
        const uint32_t r2 = rr - zz * ptiles;
        const uint32_t yy = fdiv(r2, a.fd_ntx);
        const int xt = int(r2 - yy * uint32_t(a.ntx));
        const int y = y0 + int(yb) * a.BY + int(yy);
        const int z = int(zz);
        const int row = z * a.Ly + y;
        const int xe = xt * kBlock + tid;           // element inside the row
        if (xe >= a.rowel) continue;                // ragged end of the row
        const int x = xe >> a.logsite;
        const int64_t rb = (int64_t)row * a.rowel;
        const uint32_t off0 = uint32_t(xe) * ES;    // byte offset inside a row
        const cplx<T>* xrow = a.x + rb;
        const cplx<T> xc = ld_row(xrow, off0);
        const cplx<T> zv = ld_row_nt(a.zsrc + rb, off0);
        cplx<T> av{T(0), T(0)};
        if (a.ep & EP_ACC_ADD) av = ld_row_nt(a.acc_in + rb, off0);
        T vs = T(0);
        if (a.field != 0) {
            const int64_t vs0 = (int64_t)row * a.Lx * (a.pot_mode == 1 ? 1 : NO);
            vs = field_at(a, a.pot_mode == 1 ? vs0 + x : vs0 + x * NO + o);
        }
        T hr, hi;
        const T d = dgr - beT + vs;
        hr = d * xc.re - dgi * xc.im;
        hi = d * xc.im + dgi * xc.re;
        if constexpr (P::FAMILY != FAM_GENERIC) {
            cplx<T> nv[NS > 0 ? NS : 1];
            bool okt[P::NT > 0 ? P::NT : 1];
            sfor<P::NT>([&](auto tt) {
                constexpr int tb = decltype(tt)::value;
                constexpr int dy = P::off[tb][1], dz = P::off[tb][2];
                const cplx<T>* prow = xrow;
                if constexpr (dy != 0 || dz != 0) {
                    int nrow;
                    const bool rok = neighbour_row(a, y, z, dy, dz, nrow);
                    prow = rok ? a.x + (int64_t)nrow * a.rowel : a.zero_row;
                }
                int dxe;
                okt[tb] = x_shift(a, x, P::off[tb][0], dxe);
                sfor<NS>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    if constexpr (S.t[j] == tb) nv[j] = ld_row(prow, uint32_t(xe + dxe + dq[j]) * ES);
                });
            });
            sfor<NS>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                if constexpr (S.t[j] == P::NT) nv[j] = ld_row(xrow, uint32_t(xe + dq[j]) * ES);
            });
            sfor<NS>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                if constexpr (S.t[j] < P::NT && P::off[S.t[j] < P::NT ? S.t[j] : 0][0] != 0) {
                    // x neighbour: lane-dependent open boundary
                    if (!a.px) nv[j] = zero_unless(okt[S.t[j]], nv[j]);
                }
                mac<T>(hr, hi, S.kind[j], cre[j], cim[j], nv[j]);
            });
        } else {
            // nonzero entries only; the loads of a term are issued together
            const int own = xe - o * nb;            // orbital-0 element of this site and column
            for (int tb = 0; tb < a.n_terms; ++tb) {
                const int dy = a.offs[3 * tb + 1], dz = a.offs[3 * tb + 2];
                int nrow;
                const bool rok = neighbour_row(a, y, z, dy, dz, nrow);
                const cplx<T>* prow = rok ? a.x + (int64_t)nrow * a.rowel : a.zero_row;
                int dxe;
                const bool ok = x_shift(a, x, a.offs[3 * tb], dxe);
                const int e0 = g_ptr[tb * NO + o], ne = g_ptr[tb * NO + o + 1] - e0;
                cplx<T> v[NO];
#pragma unroll
                for (int k = 0; k < NO; ++k)
                    if (k < ne) v[k] = ld_row(prow, uint32_t(own + dxe + g_col[e0 + k] * nb) * ES);
#pragma unroll
                for (int k = 0; k < NO; ++k)
                    if (k < ne) mac<T>(hr, hi, CC, g_val[e0 + k].re, g_val[e0 + k].im, zero_unless(ok, v[k]));
            }
            const int e0 = g_ptr[a.n_terms * NO + o], e1 = g_ptr[a.n_terms * NO + o + 1];
            for (int e = e0; e < e1; ++e)
                mac<T>(hr, hi, CC, g_val[e].re, g_val[e].im, ld_row(xrow, uint32_t(own + g_col[e] * nb) * ES));
        }
        const int64_t site = (int64_t)row * a.Lx + x;
        const int64_t gidx = a.ggroup == nb ? site * NO + o : site;
        epilogue(a, rb + xe, gidx, tid & (a.ggroup - 1), xc, zv, av, hr, hi, alT, gaT, er, ei, c, dxx, dxr, dxi, dyy);
    }

    if (a.ep & (EP_DOTS | EP_MOMENTS)) {
        // lanes with the same column: lane = (site * NO + o) * nb + c inside the wave
        const int ndot = (a.ep & EP_DOTS) ? 4 : 2;
        for (int m = nb; m < 64; m <<= 1) {
            dxx += __shfl_xor(dxx, m);
            dxr += __shfl_xor(dxr, m);
        }
        if (ndot == 4) {
            for (int m = nb; m < 64; m <<= 1) {
                dxi += __shfl_xor(dxi, m);
                dyy += __shfl_xor(dyy, m);
            }
        }
        __shared__ double red[kBlock / 64][PV_MAX_NB_K][4];
        const int wave = tid >> 6, lane = tid & 63;
        if (lane < nb) {
            red[wave][lane][0] = dxx;
            red[wave][lane][1] = dxr;
            red[wave][lane][2] = dxi;
            red[wave][lane][3] = dyy;
        }
        __syncthreads();
        if (tid < nb * ndot) {
            const int cc = ndot == 4 ? tid >> 2 : tid >> 1, k = tid & (ndot - 1);
            double sum = 0.0;
            for (int w = 0; w < kBlock / 64; ++w) sum += red[w][cc][k];
            a.partials[((size_t)b_out * nb + cc) * ndot + k] = sum;
        }
    }
}

// One sweep over a whole lattice.  Workgroup b runs on XCD b % 8 (the
// hardware deals workgroups out round-robin); XCD k owns the rows y in
// [Ly k/8, Ly (k+1)/8) for every z and its workgroups sweep them slab by slab,
// so the +-y and +-z neighbour rows a tile reads were fetched into the same L2
// shortly before.
template <class P, typename T, typename VT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(PV_SWEEP_WAVES_PER_EU)))
void sweep_kernel(KArgs<T, VT> a) {
    const int b = blockIdx.x;
    const int k = b & 7;
    const int y0 = int((int64_t)a.Ly * k / 8);
    const int ny = int((int64_t)a.Ly * (k + 1) / 8) - y0;
    const int64_t ntl = (int64_t)a.ntx * ny * a.Lz;
    const int64_t t0 = (int64_t)(b >> 3) * a.tpb;
    const int64_t t1 = min(t0 + a.tpb, ntl);
    sweep_block<P, T, VT>(a, b, y0, ny, t0, t1);
}

// One sweep over a batch of independent lattices of the same family in a
// single launch: workgroup b serves instance block_inst[b], whose argument
// record (geometry, buffers, scale and shift) is table[instance]; each
// instance's workgroups are consecutive and cover its tiles in order.
// part_off: doubles from the records' partials to this step's.
template <class P, typename T, typename VT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(PV_SWEEP_WAVES_PER_EU)))
void batch_sweep_kernel(const KArgs<T, VT>* __restrict__ table, const int* __restrict__ block_inst,
                        const int* __restrict__ inst_block0, int64_t part_off) {
    const int b = blockIdx.x;
    const int i = __builtin_amdgcn_readfirstlane(block_inst[b]);
    const int lb = b - __builtin_amdgcn_readfirstlane(inst_block0[i]);
    KArgs<T, VT> a = table[i];
    a.partials += part_off;
    const int64_t ntl = (int64_t)a.ntx * a.Ly * a.Lz;
    const int64_t t0 = (int64_t)lb * a.tpb;
    const int64_t t1 = min(t0 + a.tpb, ntl);
    sweep_block<P, T, VT>(a, b, 0, a.Ly, t0, t1);
}

// ---------------------------------------------------------------------------
// Staged sweep.  A workgroup owns a column tile of TW consecutive elements of
// the rows (m, w) -- w the outer lattice index (z in 3D, y in 2D), m the
// middle one (y in 3D, none in 2D) -- and walks w.  The rows (m, w-1),
// (m, w), (m, w+1), each with one site of x halo on both sides, live in a
// three-slot LDS ring, so a walk fetches every element of its rows once; the
// rows (m -+ 1, w) of 3D lattices, the tile's z (and acc_in) elements and its
// field values are staged per step.  Every global load is a 16-byte chunk
// per lane.  Loads run two steps ahead: step s issues the rows of step s + 2
// into one of two register sets while it computes from LDS, then hands the
// other set (issued one step earlier) to LDS behind a barrier that waits for
// LDS operations only, so loads and y stores stay in flight across steps.
//
// Walks are items of an XCD part (8 parts: split along m when the lattice has
// at least 8 middle rows, along w otherwise).  Items are numbered walk chunk
// first, then strips of st_Bm middle rows, then x tile, then m; the G
// workgroups of a part take items j, j + G, ... so the workgroups resident on
// one XCD walk a compact block of neighbouring columns side by side and read
// each other's rows (m -+ 1, w) and x halos from the same L2.
// ---------------------------------------------------------------------------
// The kernel's elements are 16-byte chunks wherever the layout allows: one
// complex128 number (W = 1), or the complex64 numbers of two neighbouring
// columns (W = 2, blocks of at least two columns), with half as many "columns"
// nb / W.  A lane's LDS read of a neighbour is then 16 bytes, the coefficients
// serve both columns, and z and acc go from memory to the lane that uses them
// without LDS (ZR).  Blocks of one complex64 column, and the run-time epilogue,
// have 8-byte elements, two to a chunk.  E counts complex numbers per lane, EL
// elements.  Measured on TI, complex64, against one column per element (half
// as many LDS instructions and row addresses; four numbers per lane no longer
// spill): step 256x256x64 nb 4 376 -> 352 us (E = 4: 326 -> 293), 64^3 nb 32,
// E = 4, 154 -> 140; plain 240x240x6 nb 32 242 -> 209.  complex128 without the
// LDS copies of z and acc: unchanged within 1%.
template <typename T, int W>
struct alignas(W * sizeof(cplx<T>)) Elem {
    cplx<T> v[W];
};

template <typename T, int E, int NT, int W>
struct Staged {
    static constexpr int NTH = NT;                           // lanes per workgroup
    static constexpr int EL = E / W;
    static constexpr int LW = W == 2 ? 1 : 0;
    static constexpr int ES = int(sizeof(Elem<T, W>));
    static constexpr int CE = 16 / ES;                       // elements per 16-byte chunk
    static constexpr bool ZR = CE == 1;
    static constexpr int TW = NT * EL;                       // elements per column tile
    static constexpr int TCH = TW / (CE * NT);               // chunks per lane of a row without halo
    static constexpr int RCH = (TW + 2 * STAGED_MAX_SITE / W + CE * NT - 1) / (CE * NT);  // with halo
    static_assert(E % W == 0 && W * sizeof(cplx<T>) <= 16, "whole elements per lane, at most a chunk each");
    static_assert(TW % (CE * NT) == 0, "a tile must be whole chunks per lane");
    static_assert(NT % 64 == 0 && NT <= 1024, "whole waves");
};

// Barrier for LDS hand-offs only: waits for this wave's LDS operations, not
// for its global loads and stores, so prefetches and y stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // gfx9 encoding: lgkmcnt(0), vmcnt and expcnt unlimited
    __builtin_amdgcn_s_barrier();
}

template <typename T>
__device__ __forceinline__ u32x4 ld_chunk(const void* base, uint32_t boff) {
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + boff);
}

// (of a vector that is aligned as its numbers are)
template <typename T>
__device__ __forceinline__ u32x4 ld_chunk_nt(const void* base, uint32_t boff) {
    using V = unsigned int __attribute__((ext_vector_type(4), aligned(sizeof(cplx<T>))));
    return __builtin_nontemporal_load(reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + boff));
}

// One step's worth of rows in flight: ring row with halo, z and acc_in
// chunks, field values.  (The side rows of 3D lattices, mostly L2 hits, are
// loaded one step ahead into a single set of their own.)
template <class P, typename T, typename VT, int E, int NT, int W>
struct StagedSet {
    using S = Staged<T, E, NT, W>;
    u32x4 ring[S::RCH];
    u32x4 z[S::TCH];
    VT v[S::EL];      // stored field entries (converted when handed to LDS)
    int64_t vrow;     // first field entry of the set's row
};

// Side rows hold the tile, or for stencils with hops that have a y and an x
// step (P::SIDE_HALO) the tile with the one-site x halo of ring rows.  They
// are the rows (m -+ 1, w), and for stencils with hops that have a y and a z
// step (P::SIDE_W) also (m -+ 1, w -+ 1): side row idx(dm, dw).
template <class P, typename T, int E, int NT, int W>
struct StagedSide {
    using S = Staged<T, E, NT, W>;
    static constexpr int NTR = P::DIM == 3 ? (P::SIDE_W ? 6 : 2) : 0;
    __host__ __device__ static constexpr int idx(int dm, int dw) {
        return (dm < 0 ? 0 : 1) + (P::SIDE_W ? 2 * (dw + 1) : 0);
    }
    static constexpr bool HALO = side_halo<P>();
    static constexpr int SCH = HALO ? S::RCH : S::TCH;                  // chunks per lane
    static constexpr int SLEN = HALO ? S::RCH * NT * S::CE : S::TW;     // LDS elements per row
    u32x4 side[NTR > 0 ? NTR : 1][SCH];
    u32x4 acc[S::TCH];
    u32x4 gw[3][S::TCH];   // adjoint steps: the three source vectors
    double grad[S::EL];    // and the gradient entries
};

// Stencils whose rows differ along one axis at a time: the kernel can walk along
// z with side rows y -+ 1, or along y with side rows z -+ 1.
template <class P>
__host__ __device__ constexpr bool walks_either() {
    if (P::FAMILY != FAM_TI && P::FAMILY != FAM_WEYL) return false;
    for (int t = 0; t < P::NT; ++t)
        if ((P::off[t][0] != 0) + (P::off[t][1] != 0) + (P::off[t][2] != 0) != 1) return false;
    return true;
}

// ZL: the step reads z (every epilogue but the plain sweep with gamma = 0)
template <class P, typename T, typename VT, int E, bool ACC, int NT, int W, bool ZL = true, bool ADJ = false>
struct StagedCtx {
    using S = Staged<T, E, NT, W>;
    using El = Elem<T, W>;
    using Set = StagedSet<P, T, VT, E, NT, W>;
    using Side = StagedSide<P, T, E, NT, W>;
    static constexpr int NTR = Side::NTR, EL = S::EL;
    const KArgs<T, VT>& a;
    El* ring;        // [3][seg]
    El* tra;         // [NTR][Side::SLEN]
    El* zl;          // [TW] (without ZR)
    El* al;          // [TW] (ACC only, without ZR)
    T* vl;           // [EL S::NTH]
    int tid, nch, m, wb;
    int rowel, site;   // elements per row, per site
    // per walk: byte offsets inside a row of this lane's ring chunks (x
    // wrapped; open boundaries are applied when computing), row chunks and
    // field entries (clamped into the row)
    uint32_t roff[S::RCH] = {};
    uint32_t soff[S::TCH] = {};
    uint32_t voff[EL] = {};
    uint32_t goff[EL] = {};   // adjoint steps: gradient entries inside a row
    int vshift = 0;  // element -> field entry: log2 of elements per site or per orbital row

    __device__ __forceinline__ int64_t row_of(int mm, int ww) const {
        return P::DIM == 3 ? (int64_t)ww * a.st_rw + (int64_t)mm * a.st_rm : (int64_t)ww;
    }
    // Row (mm, ww) after wrapping periodic dimensions; -1 when an open
    // boundary drops it.  Integer selects (no boolean state across blocks),
    // so the row arithmetic stays in scalar registers.
    __device__ __forceinline__ int64_t row_idx(int mm, int ww) const {
        const int Lw = a.st_Lw, Lm = a.st_Lm;
        const int wout = int(ww < 0) | int(ww >= Lw);
        const int mout = int(mm < 0) | int(mm >= Lm);
        const int dead = (wout & (a.st_pw ^ 1)) | (mout & (a.st_pm ^ 1));
        ww += ww < 0 ? Lw : 0;
        ww -= ww >= Lw ? Lw : 0;
        if (ww >= Lw) ww %= Lw;   // w + 3 on a lattice of few planes
        mm += mm < 0 ? Lm : 0;
        mm -= mm >= Lm ? Lm : 0;
        return dead ? int64_t(-1) : row_of(mm, ww);
    }
    __device__ __forceinline__ const cplx<T>* row_ptr(int mm, int ww) const {
        const int64_t r = row_idx(mm, ww);
        return r >= 0 ? a.x + r * a.rowel : a.zero_row;
    }
    __device__ __forceinline__ void setup(int xe0) {
        // chunks past the ring row (tile + halo) repeat its last chunk: every
        // lane loads and stores every chunk without branches, and the
        // repeated addresses add no traffic
#pragma unroll
        for (int k = 0; k < S::RCH; ++k) {
            const int q = tid + k * S::NTH;
            int g = xe0 - site + (q < nch ? q : nch - 1) * S::CE;
            if (g < 0) g += rowel;
            if (g >= rowel) g %= rowel;
            roff[k] = uint32_t(g) * S::ES;
        }
#pragma unroll
        for (int k = 0; k < S::TCH; ++k) {
            const int g = xe0 + (tid + k * S::NTH) * S::CE;
            soff[k] = uint32_t(g < rowel ? g : rowel - S::CE) * S::ES;
        }
        // field entries of the tile: one per site (site field) or per orbital
        // row, clamped into the lattice row
        const int vlen = a.pot_mode == 1 ? a.Lx : a.Lx * P::NO;
#pragma unroll
        for (int k = 0; k < EL; ++k) {
            int r = (xe0 >> vshift) + tid + k * S::NTH;
            if (r >= vlen) r = vlen - 1;
            voff[k] = uint32_t(r);
        }
        if constexpr (ADJ) {
#pragma unroll
            for (int k = 0; k < EL; ++k) {
                int g = xe0 + tid + k * S::NTH;
                if (g >= rowel) g = rowel - 1;
                goff[k] = uint32_t(g) >> __builtin_ctz(a.ggroup);   // a power of two
            }
        }
    }
    __device__ __forceinline__ double* grad_row(int64_t row) const {
        return a.grad + row * (a.rowel >> __builtin_ctz(a.ggroup));
    }
    // Issue the loads of ring row (m, w_ring) and of the per-step rows of
    // outer index w_row (clamped to the walk) into the set.  Every load is
    // unconditional (branch-free code lets the compiler wait for exactly
    // the loads a hand-over needs, keeping the next step's loads in flight).
    __device__ __forceinline__ void issue(Set& st, int w_ring, int w_row) const {
        const cplx<T>* rp = row_ptr(m, w_ring);
#pragma unroll
        for (int k = 0; k < S::RCH; ++k) st.ring[k] = ld_chunk<T>(rp, roff[k]);
        const int wr = w_row < wb ? w_row : wb - 1;
        const int64_t rw = row_of(m, wr);
        const cplx<T>* zr = a.zsrc + rw * a.rowel;
        if constexpr (ZL) {
#pragma unroll
            for (int k = 0; k < S::TCH; ++k) st.z[k] = ld_chunk_nt<T>(zr, soff[k]);
        }
        // stored field entries (a row of the zero row's bytes when the field
        // is absent or generated; those values are not used)
        st.vrow = rw * a.Lx * (a.pot_mode == 1 ? 1 : P::NO);
        const VT* vp = a.field == 1 ? a.V + st.vrow : reinterpret_cast<const VT*>(a.zero_row);
#pragma unroll
        for (int k = 0; k < EL; ++k) st.v[k] = vp[voff[k]];
    }
    // Side rows (m -+ 1, w_row) (and (m -+ 1, w_row -+ 1) for SIDE_W),
    // w_row clamped to the walk (3D lattices).
    __device__ __forceinline__ void issue_side(Side& sd, int w_row) const {
        if constexpr (ACC) {
            const int wr = w_row < wb ? w_row : wb - 1;
            const cplx<T>* ar = a.asrc + row_of(m, wr) * a.rowel;
#pragma unroll
            for (int k = 0; k < S::TCH; ++k) sd.acc[k] = ld_chunk_nt<T>(ar, soff[k]);
        }
        if constexpr (ADJ) {
            const int64_t rw = row_of(m, w_row < wb ? w_row : wb - 1);
#pragma unroll
            for (int k = 0; k < S::TCH; ++k) {
                sd.gw[0][k] = ld_chunk_nt<T>(a.gw0 + rw * a.rowel, soff[k]);
                sd.gw[1][k] = ld_chunk_nt<T>(a.gw1 + rw * a.rowel, soff[k]);
                sd.gw[2][k] = ld_chunk_nt<T>(a.gw2 + rw * a.rowel, soff[k]);
            }
            const double* gr = grad_row(rw);
#pragma unroll
            for (int k = 0; k < EL; ++k) sd.grad[k] = gr[goff[k]];
        }
        if constexpr (NTR > 0) {
            const int wr = w_row < wb ? w_row : wb - 1;
#pragma unroll
            for (int h = 0; h < NTR; ++h) {
                const cplx<T>* sp = row_ptr(m + ((h & 1) ? 1 : -1), wr + (P::SIDE_W ? (h >> 1) - 1 : 0));
                if constexpr (Side::HALO) {
#pragma unroll
                    for (int k = 0; k < Side::SCH; ++k) sd.side[h][k] = ld_chunk<T>(sp, roff[k]);
                } else {
#pragma unroll
                    for (int k = 0; k < Side::SCH; ++k) sd.side[h][k] = ld_chunk<T>(sp, soff[k]);
                }
            }
        }
    }
    __device__ __forceinline__ void commit_side(const Side& sd) const {
        if constexpr (ACC && !S::ZR) {
            u32x4* da = reinterpret_cast<u32x4*>(al);
#pragma unroll
            for (int k = 0; k < S::TCH; ++k) da[tid + k * S::NTH] = sd.acc[k];
        }
        if constexpr (NTR > 0) {
#pragma unroll
            for (int h = 0; h < NTR; ++h) {
                u32x4* ds = reinterpret_cast<u32x4*>(tra + h * Side::SLEN);
#pragma unroll
                for (int k = 0; k < Side::SCH; ++k) ds[tid + k * S::NTH] = sd.side[h][k];
            }
        }
    }
    // Hand a set to LDS: ring row into slot, per-step rows into their buffers.
    __device__ __forceinline__ void commit(const Set& st, int slot) const {
        u32x4* d = reinterpret_cast<u32x4*>(ring + slot * a.st_seg);
#pragma unroll
        for (int k = 0; k < S::RCH; ++k) d[tid + k * S::NTH] = st.ring[k];
        if constexpr (ZL && !S::ZR) {
            u32x4* dz = reinterpret_cast<u32x4*>(zl);
#pragma unroll
            for (int k = 0; k < S::TCH; ++k) dz[tid + k * S::NTH] = st.z[k];
        }
        if (a.field == 2) {
            // only the entries the tile reads (TW >> vshift: one per site or
            // orbital row) are generated, not one per lane and element
            const int nent = S::TW >> vshift;
#pragma unroll
            for (int k = 0; k < EL; ++k) {
                const int q = tid + k * S::NTH;
                if (q < nent) vl[q] = field_at(a, st.vrow + voff[k]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < EL; ++k) vl[tid + k * S::NTH] = T(st.v[k]);
        }
    }
    // Ring row (m, ww) alone, and its hand-over to a slot (start of a walk: all
    // of its loads are in flight before the first wait).
    __device__ __forceinline__ void ring_load(u32x4 (&r)[S::RCH], int ww) const {
        const cplx<T>* rp = row_ptr(m, ww);
#pragma unroll
        for (int k = 0; k < S::RCH; ++k) r[k] = ld_chunk<T>(rp, roff[k]);
    }
    __device__ __forceinline__ void ring_store(const u32x4 (&r)[S::RCH], int slot) const {
        u32x4* d = reinterpret_cast<u32x4*>(ring + slot * a.st_seg);
#pragma unroll
        for (int k = 0; k < S::RCH; ++k) d[tid + k * S::NTH] = r[k];
    }
};

// LDS of a staged workgroup: three ring rows with halo (slots padded to
// whole chunks per lane), the side rows of 3D lattices, z (and acc_in) of
// the tile without ZR, and the field of its orbital rows (padded to EL per
// lane).
template <typename T, int E, int NT, int W>
__host__ __device__ constexpr int staged_seg() {
    return Staged<T, E, NT, W>::RCH * NT * Staged<T, E, NT, W>::CE;
}
template <class P, typename T, int E, int NT, int W>
__host__ __device__ constexpr size_t staged_table_offset(bool acc) {
    using S = Staged<T, E, NT, W>;
    using Side = StagedSide<P, T, E, NT, W>;
    return (size_t(3 * staged_seg<T, E, NT, W>() + Side::NTR * Side::SLEN +
                   (S::ZR ? 0 : 1 + (acc ? 1 : 0)) * S::TW) * S::ES +
            size_t(S::EL * NT) * sizeof(T) + 15) / 16 * 16;
}
// Generic stencils also keep their block entries in LDS: values, then
// offsets, row starts and columns.
template <class P>
struct StagedTable {
    static constexpr int GMAX = (PV_MAX_TERMS_K + 1) * P::NO * P::NO;
    static constexpr int NPTR = (PV_MAX_TERMS_K + 1) * P::NO + 1;
    static constexpr int NINT = 3 * PV_MAX_TERMS_K + NPTR + GMAX;
};
template <class P, typename T, int E, int NT, int W>
__host__ __device__ constexpr size_t staged_lds_bytes_for(bool acc) {
    return staged_table_offset<P, T, E, NT, W>(acc) +
           (P::FAMILY == FAM_GENERIC
                ? StagedTable<P>::GMAX * sizeof(cplx<T>) + StagedTable<P>::NINT * sizeof(int)
                : 0);
}

// Epilogue of the specialised kernels (uniform alpha, beta, gamma): the
// operations of epilogue_ep, with whole elements loaded and stored.
template <unsigned EPM, typename T, typename VT, int W>
__device__ __forceinline__ void staged_epilogue(const KArgs<T, VT>& a, int64_t e, const Elem<T, W>& x,
                                                const Elem<T, W>& z, const Elem<T, W>& acc, const Elem<T, W>& h, T alT,
                                                T gaT, T er, T ei, double (&dxx)[W], double (&dxr)[W],
                                                double (&dxi)[W], double (&dyy)[W]) {
    using V = T __attribute__((ext_vector_type(2 * W), aligned(sizeof(cplx<T>))));
    V yo, ao;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        T yr = alT * h.v[q].re, yi = alT * h.v[q].im;
        yr += (gaT != T(0)) ? gaT * z.v[q].re : T(0);
        yi += (gaT != T(0)) ? gaT * z.v[q].im : T(0);
        yo[2 * q] = yr;
        yo[2 * q + 1] = yi;
        if constexpr ((EPM & EP_ACC_ADD) != 0u) {
            T ar = acc.v[q].re, ai = acc.v[q].im;
            if constexpr ((EPM & EP_ACC_Z) != 0u)
                add_term(ar, ai, T(a.etaz_re), T(a.etaz_im), z.v[q].re, z.v[q].im);
            if constexpr ((EPM & EP_ACC_X) != 0u)
                add_term(ar, ai, T(a.etax_re), T(a.etax_im), x.v[q].re, x.v[q].im);
            add_term(ar, ai, er, ei, yr, yi);
            ao[2 * q] = ar;
            ao[2 * q + 1] = ai;
        }
        if constexpr ((EPM & (EP_DOTS | EP_MOMENTS)) != 0u) {
            const double xr = double(x.v[q].re), xi = double(x.v[q].im);
            const double dyr = double(yr), dyi = double(yi);
            dxx[q] += xr * xr + xi * xi;
            dxr[q] += xr * dyr + xi * dyi;
            if constexpr ((EPM & EP_DOTS) != 0u) {
                dxi[q] += xr * dyi - xi * dyr;
                dyy[q] += dyr * dyr + dyi * dyi;
            }
        }
    }
    if constexpr ((EPM & EP_STORE_Y) != 0u) __builtin_nontemporal_store(yo, reinterpret_cast<V*>(a.y + e));
    if constexpr ((EPM & EP_ACC_ADD) != 0u) __builtin_nontemporal_store(ao, reinterpret_cast<V*>(a.acc_out + e));
}

template <class P, typename T, typename VT, int E, unsigned EPM, int NT, int W>
__device__ __forceinline__ void staged_block(const KArgs<T, VT>& a, int b_out, int part, int jb, int G) {
    using S = Staged<T, E, NT, W>;
    using El = Elem<T, W>;
    constexpr bool ADJ = EPM == EP_ADJOINT;
    static_assert((EPM != 0u && !ADJ) || W == 1, "these epilogues have elements of one column");
    constexpr int EL = S::EL;
    constexpr bool ACC = EPM == 0u || (EPM & EP_ACC_ADD) != 0u;
    constexpr bool ZL = (EPM & EP_NO_Z) == 0u;
    using Ctx = StagedCtx<P, T, VT, E, ACC, NT, W, ZL, ADJ>;
    static_assert(!ADJ || S::ZR, "adjoint steps take their vectors from registers");
    using Set = typename Ctx::Set;
    constexpr int NO = P::NO;
    constexpr int NTR = Ctx::NTR;
    constexpr bool GEN = P::FAMILY == FAM_GENERIC;
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned ep = EPM ? EPM : a.ep;
    const int tid = threadIdx.x;
    // in elements of W columns
    const int nb = a.nb >> S::LW, lognb = a.lognb - S::LW, logsite = a.logsite - S::LW;
    const int c = tid & (nb - 1);
    const int o = (tid >> lognb) & (NO - 1);
    const int site = a.st_site >> S::LW, rowel = a.rowel >> S::LW;

    // per-column alpha, beta, gamma only in the run-time epilogue (the
    // specialised ones are launched with uniform values)
    double al = a.alpha, be = a.beta, ga = a.gamma;
    if (EPM == 0u && a.colp != nullptr) {
        al = a.colp[3 * c];
        be = a.colp[3 * c + 1];
        ga = a.colp[3 * c + 2];
    }
    const T alT = T(al), beT = T(be), gaT = T(ga);
    const T er = T(a.eta_re), ei = T(a.eta_im);
    const int nt_on = GEN ? a.n_terms : P::NT;   // index of the on-site block
    const T dgr = T(a.coef[(((size_t)nt_on * NO + o) * NO + o) * 2]);
    const T dgi = T(a.coef[(((size_t)nt_on * NO + o) * NO + o) * 2 + 1]);
    static constexpr Slots<P> SL{};
    constexpr int NS = SL.n;
    T cre[NS > 0 ? NS : 1], cim[NS > 0 ? NS : 1];
    int dq[NS > 0 ? NS : 1];
    slot_coefficients<P, T, NS>(a.coef, o, nb, cre, cim, dq);
    double dxx[W] = {}, dxr[W] = {}, dxi[W] = {}, dyy[W] = {};
    T gcr[3] = {}, gci[3] = {};   // coefficients of the adjoint source terms
    if constexpr (ADJ) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            gcr[j] = T(a.gcoef[(j * a.nb + c) * 2]);
            gci[j] = T(a.gcoef[(j * a.nb + c) * 2 + 1]);
        }
    }

    // generic stencils: offsets and the nonzero entries of every block row
    // (packed by the host after the offsets and the dense blocks) in LDS
    using Tab = StagedTable<P>;
    cplx<T>* g_val = reinterpret_cast<cplx<T>*>(smem + staged_table_offset<P, T, E, NT, W>(ACC));
    int* g_off = reinterpret_cast<int*>(g_val + Tab::GMAX);
    int* g_ptr = g_off + 3 * PV_MAX_TERMS_K;
    int* g_col = g_ptr + Tab::NPTR;
    if constexpr (GEN) {
        const int nptr = (a.n_terms + 1) * NO + 1;
        const int* gp = a.offs + 3 * a.n_terms;
        const int nnz = gp[nptr - 1];
        const double* gv = a.coef + (size_t)(a.n_terms + 1) * NO * NO * 2;
        for (int i = tid; i < 3 * a.n_terms; i += NT) g_off[i] = a.offs[i];
        for (int i = tid; i < nptr; i += NT) g_ptr[i] = gp[i];
        for (int i = tid; i < nnz; i += NT) {
            g_col[i] = gp[nptr + i];
            g_val[i] = cplx<T>{T(gv[2 * i]), T(gv[2 * i + 1])};
        }
        __syncthreads();
    }

    Ctx cx{a, reinterpret_cast<El*>(smem), nullptr, nullptr, nullptr, nullptr, tid, (S::TW + 2 * site) / S::CE, 0, 0,
           rowel, site};
    cx.vshift = a.pot_mode == 1 ? logsite : lognb;
    cx.tra = cx.ring + 3 * a.st_seg;
    cx.zl = cx.tra + NTR * Ctx::Side::SLEN;
    cx.al = cx.zl + (S::ZR ? 0 : S::TW);
    cx.vl = reinterpret_cast<T*>(cx.al + (ACC && !S::ZR ? S::TW : 0));

    // this part's ranges of m and w
    int m0 = 0, m1 = a.st_Lm, wA = 0, wB = a.st_Lw;
    if (a.st_parts == 8) {
        if (a.st_Lm >= 8) {
            m0 = a.st_Lm * part / 8;
            m1 = a.st_Lm * (part + 1) / 8;
        } else {
            wA = a.st_Lw * part / 8;
            wB = a.st_Lw * (part + 1) / 8;
        }
    }
    const int nm = m1 - m0, nW = wB - wA;
    const int nwc = nW > 0 ? (nW + a.st_C - 1) / a.st_C : 0;
    const int bms = min(a.st_Bm, nm);
    const int per_wc = nm * a.st_nxs;
    const int items = nwc * per_wc;

    for (int j = jb; j < items; j += G) {
        const int wc = j / per_wc;
        const int rem = j - wc * per_wc;
        const int ms = (rem / (bms * a.st_nxs)) * bms;
        const int bm = min(bms, nm - ms);
        const int r2 = rem - ms * a.st_nxs;
        const int xs = r2 / bm;
        cx.m = m0 + ms + (r2 - xs * bm);
        const int xe0 = xs * S::TW;
        cx.setup(xe0);
        const int wa = wA + wc * a.st_C;
        const int wb = min(wa + a.st_C, wB);
        cx.wb = wb;
        const int nsteps = wb - wa;

        // prologue: ring rows wa - 1, wa into slots 0, 1; set A = ring row
        // wa + 1 and the rows of step 0, handed over now; set B = ring row
        // wa + 2 and the rows of step 1, left in flight
        Set A, B;
        typename Ctx::Side SD;
        {
            u32x4 r0[S::RCH], r1[S::RCH];
            cx.ring_load(r0, wa - 1);
            cx.ring_load(r1, wa);
            cx.issue_side(SD, wa);
            cx.issue(A, wa + 1, wa);
            cx.ring_store(r0, 0);
            cx.ring_store(r1, 1);
        }
        cx.commit(A, 2);
        cx.commit_side(SD);
        El zc[EL], ac[EL];   // z and acc of the step at hand (ZR)
        El gc[3][EL];        // and what an adjoint step reads
        double gradc[EL];
        auto take = [&](const Set& st) {
            if constexpr (S::ZR) {
#pragma unroll
                for (int k = 0; k < EL; ++k) {
                    if constexpr (ZL) zc[k] = __builtin_bit_cast(El, st.z[k]);
                    if constexpr (ACC) ac[k] = __builtin_bit_cast(El, SD.acc[k]);
                    if constexpr (ADJ) {
                        for (int j = 0; j < 3; ++j) gc[j][k] = __builtin_bit_cast(El, SD.gw[j][k]);
                        gradc[k] = SD.grad[k];
                    }
                }
            }
        };
        take(A);
        cx.issue(B, wa + 2, wa + 1);
        lds_barrier();

        // step s (outer index wa + s): issue the side rows of step s + 1 and
        // `nx` for step s + 2, compute from LDS, hand `cur` (issued for step
        // s + 1) and the side rows over, store.  Issue and hand-over run on
        // every step; past the walk they fetch rows read two steps earlier
        // (cache hits) and fill buffers nobody reads.
        auto step = [&](int s, Set& nx, const Set& cur) {
            const int w = wa + s;
            cx.issue_side(SD, w + 1);
            cx.issue(nx, s + 2 < nsteps ? w + 3 : w + 1, w + 2);
            const El* rm = cx.ring + (s % 3) * a.st_seg + site;
            const El* r0 = cx.ring + ((s + 1) % 3) * a.st_seg + site;
            const El* rp = cx.ring + ((s + 2) % 3) * a.st_seg + site;
            // the rows y -+ 1 and z -+ 1 of a stencil that walks along either axis
            const El* ylo = a.st_ywalk ? rm : cx.tra;
            const El* yhi = a.st_ywalk ? rp : cx.tra + Ctx::Side::SLEN;
            const El* zlo = a.st_ywalk ? cx.tra : rm;
            const El* zhi = a.st_ywalk ? cx.tra + Ctx::Side::SLEN : rp;
            const int64_t rowi = cx.row_of(cx.m, w);
            const int64_t rb = rowi * a.rowel;
            El hv[EL], xs_[EL], zv[EL], av[EL], gv[3][EL];
            double gradv[EL];
#pragma unroll
            for (int k = 0; k < EL; ++k) {
                const int l = tid + k * NT;
                const int xe = xe0 + l;
                const int x = xe >> logsite;
                const bool xlo = a.px || x > 0, xhi = a.px || x < a.Lx - 1;
                const El xc = r0[l];
                const T vs = a.field != 0 ? cx.vl[l >> cx.vshift] : T(0);
                const T d = dgr - beT + vs;
                T hr[W], hi[W];
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    hr[q] = d * xc.v[q].re - dgi * xc.v[q].im;
                    hi[q] = d * xc.v[q].im + dgi * xc.v[q].re;
                }
                if constexpr (GEN) {
                    // runtime terms: rows (m, w + dw) from the ring with the x
                    // halo, rows (m -+ 1, w) from the side rows (with the x halo
                    // in the instance for hops with a y and an x step; the host
                    // admits no offset with both a y and a z step)
                    for (int tb = 0; tb < a.n_terms; ++tb) {
                        const int dx = g_off[3 * tb], dm = g_off[3 * tb + 1], dw = g_off[3 * tb + 2];
                        // side rows start at the tile (no halo) or one site before it
                        constexpr int side0 = Ctx::Side::HALO ? 1 : 0;
                        const El* rw = (dm != 0 ? cx.tra + (dm < 0 ? 0 : Ctx::Side::SLEN) + side0 * site
                                                : (dw < 0 ? rm : (dw > 0 ? rp : r0))) + l + dx * site;
                        const bool ok = dx < 0 ? xlo : (dx > 0 ? xhi : true);
                        const int e0 = g_ptr[tb * NO + o], e1 = g_ptr[tb * NO + o + 1];
                        for (int e = e0; e < e1; ++e) {
                            const El v = rw[(g_col[e] - o) * nb];
#pragma unroll
                            for (int q = 0; q < W; ++q)
                                mac<T>(hr[q], hi[q], CC, g_val[e].re, g_val[e].im, zero_unless(ok, v.v[q]));
                        }
                    }
                    const int e0 = g_ptr[a.n_terms * NO + o], e1 = g_ptr[a.n_terms * NO + o + 1];
                    for (int e = e0; e < e1; ++e) {
                        const El v = r0[l + (g_col[e] - o) * nb];
#pragma unroll
                        for (int q = 0; q < W; ++q) mac<T>(hr[q], hi[q], CC, g_val[e].re, g_val[e].im, v.v[q]);
                    }
                } else {
                    sfor<NS>([&](auto jj) {
                        constexpr int jx = decltype(jj)::value;
                        constexpr int t = SL.t[jx];
                        const int dqj = SL.same[jx] ? 0 : dq[jx];   // constant 0 for own-orbital slots
                        El v;
                        constexpr int tt = t < P::NT ? t : 0;
                        constexpr int dx = t < P::NT ? P::off[tt][0] : 0;
                        if constexpr (t == P::NT) {
                            v = r0[l + dqj];
                        } else if constexpr (walks_either<P>()) {
                            constexpr int dy = P::off[tt][1], dz = P::off[tt][2];
                            if constexpr (dx != 0) v = r0[l + dx * site + dqj];
                            else if constexpr (dy != 0) v = (dy < 0 ? ylo : yhi)[l + dqj];
                            else v = (dz < 0 ? zlo : zhi)[l + dqj];
                        } else {
                            constexpr int dm = P::DIM == 3 ? P::off[tt][1] : 0;
                            constexpr int dw = P::DIM == 3 ? P::off[tt][2] : P::off[tt][1];
                            if constexpr (dm == 0) {
                                const El* rw = dw < 0 ? rm : (dw > 0 ? rp : r0);
                                v = rw[l + dx * site + dqj];
                            } else {
                                // side rows start at the tile, or one site
                                // before it in the instance with the halo
                                constexpr bool HALO = Ctx::Side::HALO;
                                static_assert(dw == 0 || P::SIDE_W, "side rows at w -+ 1 need SIDE_W");
                                static_assert(dx == 0 || HALO, "x steps on side rows need their halo");
                                constexpr int h = Ctx::Side::idx(dm, dw);
                                v = cx.tra[h * Ctx::Side::SLEN + (HALO ? site : 0) + l + dx * site + dqj];
                            }
                        }
#pragma unroll
                        for (int q = 0; q < W; ++q) {
                            cplx<T> u = v.v[q];
                            if constexpr (dx < 0) u = zero_unless(xlo, u);
                            if constexpr (dx > 0) u = zero_unless(xhi, u);
                            mac<T>(hr[q], hi[q], SL.kind[jx], cre[jx], cim[jx], u);
                        }
                    });
                }
                xs_[k] = xc;
#pragma unroll
                for (int q = 0; q < W; ++q) hv[k].v[q] = cplx<T>{hr[q], hi[q]};
                if constexpr (ZL) zv[k] = S::ZR ? zc[k] : cx.zl[l];
                else zv[k] = El{};
                if constexpr (ACC) av[k] = S::ZR ? ac[k] : cx.al[l];
                else av[k] = El{};
                if constexpr (ADJ) {
                    for (int j = 0; j < 3; ++j) gv[j][k] = gc[j][k];
                    gradv[k] = gradc[k];
                }
            }
            lds_barrier();
            cx.commit(cur, (s + 3) % 3);
            cx.commit_side(SD);
            take(cur);
#pragma unroll
            for (int k = 0; k < EL; ++k) {
                const int xe = xe0 + tid + k * NT;
                if (xe < rowel) {
                    if constexpr (EPM == 0u) {
                        const int64_t st = rowi * a.Lx + (xe >> logsite);
                        const int64_t gidx = a.ggroup == a.nb ? st * NO + o : st;
                        epilogue_ep(a, ep, rb + xe, gidx, tid & (a.ggroup - 1), xs_[k].v[0], zv[k].v[0], av[k].v[0],
                                    hv[k].v[0].re, hv[k].v[0].im, alT, gaT, er, ei, c, dxx[0], dxr[0],
                                    dxi[0], dyy[0]);
                    } else if constexpr (ADJ) {
                        // the operations of epilogue_ep
                        const cplx<T> xc = xs_[k].v[0], zc1 = zv[k].v[0];
                        T yr = alT * hv[k].v[0].re, yi = alT * hv[k].v[0].im;
                        yr += (gaT != T(0)) ? gaT * zc1.re : T(0);
                        yi += (gaT != T(0)) ? gaT * zc1.im : T(0);
#pragma unroll
                        for (int j = 0; j < 3; ++j) {
                            const cplx<T> g = gv[j][k].v[0];
                            yr += gcr[j] * g.re - gci[j] * g.im;
                            yi += gcr[j] * g.im + gci[j] * g.re;
                        }
                        st_nt(a.y + rb + xe, yr, yi);
                        const cplx<T> g0 = gv[0][k].v[0], g1 = gv[1][k].v[0];
                        double g = a.gx * (double(xc.re) * double(g1.re) + double(xc.im) * double(g1.im)) +
                                   a.gy * (double(yr) * double(g0.re) + double(yi) * double(g0.im));
                        for (int mm = 1; mm < a.ggroup; mm <<= 1) g += __shfl_xor(g, mm);
                        if ((tid & (a.ggroup - 1)) == 0)
                            cx.grad_row(rowi)[cx.goff[k]] = gradv[k] + g;
                    } else {
                        staged_epilogue<EPM>(a, rb + (int64_t(xe) << S::LW), xs_[k], zv[k], av[k], hv[k], alT, gaT, er,
                                             ei, dxx, dxr, dxi, dyy);
                    }
                }
            }
            lds_barrier();
        };
        int s = 0;
        for (; s + 1 < nsteps; s += 2) {
            step(s, A, B);
            step(s + 1, B, A);
        }
        if (s < nsteps) step(s, A, B);
    }

    if (ep & (EP_DOTS | EP_MOMENTS)) {
        const int ndot = (ep & EP_DOTS) ? 4 : 2;
#pragma unroll
        for (int q = 0; q < W; ++q)
            for (int mm = nb; mm < 64; mm <<= 1) {
                dxx[q] += __shfl_xor(dxx[q], mm);
                dxr[q] += __shfl_xor(dxr[q], mm);
                if (ndot == 4) {
                    dxi[q] += __shfl_xor(dxi[q], mm);
                    dyy[q] += __shfl_xor(dyy[q], mm);
                }
            }
        __syncthreads();
        double* red = reinterpret_cast<double*>(smem);   // the ring is free after the last barrier
        const int wave = tid >> 6, lane = tid & 63;
        if (lane < nb) {
#pragma unroll
            for (int q = 0; q < W; ++q) {
                double* r = red + (wave * PV_MAX_NB_K + lane * W + q) * 4;
                r[0] = dxx[q];
                r[1] = dxr[q];
                r[2] = dxi[q];
                r[3] = dyy[q];
            }
        }
        __syncthreads();
        if (tid < a.nb * ndot) {
            const int cc = ndot == 4 ? tid >> 2 : tid >> 1, q = tid & (ndot - 1);
            double sum = 0.0;
            for (int wv = 0; wv < NT / 64; ++wv) sum += red[(wv * PV_MAX_NB_K + cc) * 4 + q];
            a.partials[((size_t)b_out * a.nb + cc) * ndot + q] = sum;
        }
    }
}

// Staged sweep over a batch of lattices in one launch: instance i owns the
// workgroups [inst_block0[i], inst_block0[i+1]), a multiple of 8 starting at
// a multiple of 8, split into its 8 XCD parts like a single-lattice launch.
template <class P, typename T, typename VT, int E, unsigned EPM, int NT, int W>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(PV_STAGED_WAVES_PER_EU)))
void batch_staged_kernel(const KArgs<T, VT>* __restrict__ table, const int* __restrict__ block_inst,
                         const int* __restrict__ inst_block0, int64_t part_off) {
    const int b = blockIdx.x;
    const int i = __builtin_amdgcn_readfirstlane(block_inst[b]);
    const int b0 = __builtin_amdgcn_readfirstlane(inst_block0[i]);
    const int b1 = __builtin_amdgcn_readfirstlane(inst_block0[i + 1]);
    KArgs<T, VT> a = table[i];
    a.partials += part_off;
    const int lb = b - b0;
    staged_block<P, T, VT, E, EPM, NT, W>(a, b, lb & 7, lb >> 3, (b1 - b0) >> 3);
}

// NT lanes per workgroup (256, or 512 for twice the tile length: half the
// relative x halo, one workgroup per CU at the larger shapes)
template <class P, typename T, typename VT, int E, unsigned EPM, int NT, int W>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(PV_STAGED_WAVES_PER_EU)))
void staged_kernel(KArgs<T, VT> a) {
    const bool p8 = a.st_parts == 8;
    const int b = blockIdx.x, g = gridDim.x;
    staged_block<P, T, VT, E, EPM, NT, W>(a, b, p8 ? (b & 7) : 0, p8 ? (b >> 3) : b, p8 ? (g >> 3) : g);
}

#ifndef PV_RTC
// Tiles per workgroup: enough workgroups to keep every CU busy for several
// rounds (>= 32 per CU), at most 64 tiles each (fewer workgroups also means
// fewer partial dot products to reduce).  PV_TILES_PER_BLOCK overrides it
// for tuning runs.
int tiles_per_block(int64_t ntiles) {
    static const int forced = [] {
        const char* e = getenv("PV_TILES_PER_BLOCK");
        return e ? atoi(e) : -1;
    }();
    if (forced > 0) return forced;
    int64_t tpb = ntiles / (256 * 32);
    if (tpb < 1) tpb = 1;
    if (tpb > 64) tpb = 64;
    return int(tpb);
}

template <class P, typename T, typename VT>
int occupancy_blocks() {
    static const int cached = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_kernel<P, T, VT>, kBlock, 0) != hipSuccess || n < 1)
            n = 1;
        return n;
    }();
    return cached;
}

// Kernel arguments from the launch description.  whole_part: one part
// covering the lattice (used by batched launches) instead of 8 XCD parts.
template <class P, typename T, typename VT>
void make_kargs(const SweepParams& p, bool whole_part, KArgs<T, VT>& a) {
    a.x = static_cast<const cplx<T>*>(p.x);
    a.z = static_cast<const cplx<T>*>(p.z);
    a.y = static_cast<cplx<T>*>(p.y);
    a.acc_in = static_cast<const cplx<T>*>(p.acc_in);
    a.acc_out = static_cast<cplx<T>*>(p.acc_out);
    a.zsrc = a.z ? a.z : a.x;
    a.asrc = ((p.ep & EP_ACC_ADD) && a.acc_in) ? a.acc_in : a.x;
    a.V = static_cast<const VT*>(p.V);
    a.field = p.field;
    a.rng_seed = p.rng_seed;
    a.rng_W = p.rng_W;
    a.gw0 = static_cast<const cplx<T>*>(p.gw[0]);
    a.gw1 = static_cast<const cplx<T>*>(p.gw[1]);
    a.gw2 = static_cast<const cplx<T>*>(p.gw[2]);
    a.gcoef = p.gcoef;
    a.grad = p.grad;
    a.gx = p.gx;
    a.gy = p.gy;
    a.ggroup = (p.grad_mode == 2) ? p.nb : P::NO * p.nb;
    a.coef = p.coef;
    a.offs = p.offs;
    a.colp = p.colp;
    a.partials = p.partials;
    a.Lx = int(p.L[0]);
    a.Ly = int(p.L[1]);
    a.Lz = int(p.L[2]);
    a.px = p.periodic[0] != 0;
    a.py = p.periodic[1] != 0;
    a.pz = p.periodic[2] != 0;
    a.nb = p.nb;
    int lg = 0;
    while ((1 << lg) < p.nb) ++lg;
    a.lognb = lg;
    int lo = 0;
    while ((1 << lo) < P::NO) ++lo;
    a.logsite = lg + lo;
    a.n_elem = p.L[0] * p.L[1] * p.L[2] * P::NO * p.nb;
    a.rowel = int(p.L[0] * P::NO * p.nb);
    a.ntx = (a.rowel + kBlock - 1) / kBlock;
    a.fd_ntx = make_fastdiv(uint32_t(a.ntx));
    a.BY = p.slab_rows;
    a.fd_slab = make_fastdiv(uint32_t(a.ntx) * uint32_t(a.BY) * uint32_t(p.L[2]));
    a.fd_pf = make_fastdiv(uint32_t(a.ntx) * uint32_t(a.BY));
    a.zero_row = static_cast<const cplx<T>*>(p.zero_row);
    a.ntiles = int64_t(a.ntx) * ((p.L[1] + 7) / 8) * p.L[2];   // tiles of the largest XCD part
    a.n_terms = p.n_terms;
    a.pot_mode = p.pot_mode;
    a.alpha = p.alpha;
    a.beta = p.beta;
    a.gamma = p.gamma;
    a.eta_re = p.eta_re;
    a.eta_im = p.eta_im;
    a.etax_re = p.etax_re;
    a.etax_im = p.etax_im;
    a.etaz_re = p.etaz_re;
    a.etaz_im = p.etaz_im;
    a.ep = p.ep;
    {
        // a requested count below the default would need more partial-dot
        // rows than a workspace holds: raise it to the default
        const int dflt = tiles_per_block(a.ntiles * 8);
        a.tpb = p.tpb > dflt ? p.tpb : dflt;
    }
    if (whole_part) {
        a.BY = int(p.L[1]);
        a.fd_slab = make_fastdiv(uint32_t(a.ntx) * uint32_t(p.L[1]) * uint32_t(p.L[2]));
        a.fd_pf = make_fastdiv(uint32_t(a.ntx) * uint32_t(p.L[1]));
        a.ntiles = int64_t(a.ntx) * p.L[1] * p.L[2];
        a.tpb = p.tpb > 0 ? p.tpb : tiles_per_block(a.ntiles);
    }
}

int env_int(const char* name, int dflt) {
    const char* e = getenv(name);
    return e ? atoi(e) : dflt;
}

// LDS of a staged kernel instance (independent of nb: tiles are elements)
template <class P, typename T, int E, unsigned EPM, int NT, int W>
size_t staged_lds_bytes() {
    return staged_lds_bytes_for<P, T, E, NT, W>(EPM == 0u || (EPM & EP_ACC_ADD) != 0u);
}

// Walks of a staged launch: which axis they follow and how many planes each.
// One eighth of the lattice (the largest XCD part, split along m when there are
// 8 middle rows, else along w) is nm rows m by nW planes; in nwc chunks of C
// planes it is `items` walks over G8 workgroups.  A walk costs its planes and
// about two more to fill the ring, and a last round of walks that leaves
// workgroups idle costs about three tenths of what it would if they did not
// leave their bandwidth to the others (one tenth with four workgroups on each
// of an XCD's 32 CUs).
struct StagedWalk {
    int nm = 0, nW = 0, C = 1, items = 1, along_y = 0;
    double cost = 0.0;
    StagedWalk(int Lm, int Lw, int nxs, int y) : along_y(y) {
        const bool split_m = Lm >= 8;
        nm = split_m ? (Lm + 7) / 8 : Lm;
        nW = split_m ? Lw : (Lw + 7) / 8;
        chunk(nW, nxs, 1);
    }
    // last: what the last round costs of a whole one
    double planes(int G8, double last) const {
        const int rounds = (items + G8 - 1) / G8;
        return ((1.0 - last) * std::max(1.0, double(items) / G8) + last * rounds) * (C + 2);
    }
    void chunk(int c, int nxs, int G8) {
        C = c < nW ? c : nW;
        if (C < 1) C = 1;
        items = nW < 1 ? 1 : ((nW + C - 1) / C) * nm * nxs;
        cost = planes(G8, G8 > 96 ? 0.1 : 0.3);
    }
};

// The walks of a launch that asks for none: along w in as few chunks as give
// every workgroup one, or, where that costs 8% less, in up to 8 chunks that
// fill the last round, or (built-in 3D stencils, fewer than 8 planes z) along
// y.  us per sweep, before | after:
//   TI c128 240x240x6 nb 32   step 522 | 447   plain 402 | 346   series 790 | 703   (along y)
//   TI c128 240x240x6 nb 2    step 37.6 | 33.6   plain 30.1 | 27.4   series 50.2 | 45.6   (along y)
//   TI c64 57x83x46 nb 8      step 56.8 | 43.0   plain 45.3 | 33.3   series 66.3 | 62.1   (5, 5, 2 chunks)
// Along y with 8 planes or more the parts are single rows m, whose side rows
// other XCDs load: 96x96x8 nb 16 step 54.0 | 58.0 at best.  Below 2^21 numbers
// and with more than two workgroups per CU a round is not filled by more chunks:
// TI c128 36x166x43 nb 2 plain 31.7 in three, 37.6 in four; 131x89x30 nb 1 24.0
// in three, 25.3 in five.
// nxs: column tiles per row.
template <class P>
StagedWalk staged_walk(const SweepParams& p, int nxs, int G8, bool full_walk) {
    const int Ly = int(p.L[1]), Lz = int(p.L[2]);
    StagedWalk k(P::DIM == 3 ? Ly : 1, P::DIM == 3 ? Lz : Ly, nxs, 0);
    if (p.st_C > 0 || full_walk) {
        k.chunk(full_walk && p.st_C <= 0 ? k.nW : p.st_C, nxs, 1);
        return k;
    }
    auto fill = [&](const StagedWalk& from, int least, StagedWalk& best) {
        for (int nwc = 1; nwc <= 8; ++nwc) {
            StagedWalk t = from;
            t.chunk((t.nW + nwc - 1) / nwc, nxs, G8);
            if (t.C >= least && t.cost < best.cost) best = t;
        }
    };
    const int cols = k.nm * nxs, n0 = std::max(1, std::min((G8 + cols - 1) / cols, k.nW));
    k.chunk((k.nW + n0 - 1) / n0, nxs, G8);
    if (p.st_Bm <= 0 && p.st_G8 <= 0) {
        const StagedWalk k0 = k;
        k.cost *= 0.92;
        const bool more = G8 <= 64 || p.L[0] * Ly * Lz * P::NO * p.nb >= (int64_t(1) << 21);
        fill(k0, more ? 1 : k0.C, k);
        if (walks_either<P>() && Lz < 8) fill(StagedWalk(Lz, Ly, nxs, 1), 1, k);
    }
    return k;
}

template <class P, typename T, typename VT, int E, int NT, int W>
int staged_setup(const SweepParams& p, int G8, bool full_walk, KArgs<T, VT>& a) {
    constexpr int TW = NT * E;   // complex numbers of a column tile
    a.st_site = P::NO * p.nb;
    a.st_seg = staged_seg<T, E, NT, W>();   // ring slot; its first elements hold the tile and two sites
    a.st_nxs = (a.rowel + TW - 1) / TW;
    const StagedWalk k = staged_walk<P>(p, a.st_nxs, G8, full_walk);
    a.st_ywalk = k.along_y;
    a.st_C = k.C;
    if (P::DIM != 3) {
        a.st_Lm = 1; a.st_Lw = a.Ly; a.st_pm = 0; a.st_pw = a.py;
        a.st_rm = 0; a.st_rw = 1;
    } else if (a.st_ywalk) {
        a.st_Lm = a.Lz; a.st_Lw = a.Ly; a.st_pm = a.pz; a.st_pw = a.py;
        a.st_rm = a.Ly; a.st_rw = 1;
    } else {
        a.st_Lm = a.Ly; a.st_Lw = a.Lz; a.st_pm = a.py; a.st_pw = a.pz;
        a.st_rm = 1; a.st_rw = a.Ly;
    }
    if (G8 > k.items) G8 = k.items;
    int bx = int(std::lround(std::sqrt(double(G8) * a.st_site / TW)));
    if (bx > a.st_nxs) bx = a.st_nxs;
    if (bx < 1) bx = 1;
    a.st_Bm = p.st_Bm > 0 ? p.st_Bm : (G8 / bx > 1 ? G8 / bx : 1);
    a.st_parts = 8;
    return G8;
}

template <class P, typename T, typename VT, int E, unsigned EPM, int NT, int W>
hipError_t launch_staged_w(SweepParams& p, int num_cus, hipStream_t s) {
    KArgs<T, VT> a;
    make_kargs<P, T, VT>(p, false, a);
    // LDS size and workgroups resident per CU: fixed per kernel instance,
    // set up once (thread-safe initialisation of the local static)
    static const std::pair<hipError_t, int> occ_res = [] {
        const size_t bytes = staged_lds_bytes<P, T, E, EPM, NT, W>();
        if (bytes > 65536) {
            const hipError_t e = hipFuncSetAttribute(
                reinterpret_cast<const void*>(&staged_kernel<P, T, VT, E, EPM, NT, W>),
                hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
            if (e != hipSuccess) return std::make_pair(e, 0);
        }
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, staged_kernel<P, T, VT, E, EPM, NT, W>, NT, bytes) !=
                hipSuccess || n < 1)
            n = 1;
        return std::make_pair(hipSuccess, n);
    }();
    if (occ_res.first != hipSuccess) return occ_res.first;
    const int occ = occ_res.second;
    const size_t lds = staged_lds_bytes<P, T, E, EPM, NT, W>();
    int G8 = p.st_G8 > 0 ? p.st_G8 : (num_cus >= 8 ? num_cus / 8 : 1) * occ;
    if (G8 > 256) G8 = 256;
    G8 = staged_setup<P, T, VT, E, NT, W>(p, G8, false, a);
    p.grid = 8 * G8;
    hipLaunchKernelGGL((staged_kernel<P, T, VT, E, EPM, NT, W>), dim3(p.grid), dim3(NT), lds, s, a);
    return hipGetLastError();
}

// Whether a block's vectors can be taken as 16-byte elements of two complex64
// columns: whole pairs of columns, and everything the epilogue touches aligned
// (x is checked with every staged launch).
template <typename T>
bool paired(const SweepParams& p) {
    if (sizeof(T) != 4 || p.nb < 2) return false;
    const uintptr_t all = reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.z) |
                          reinterpret_cast<uintptr_t>(p.y) |
                          ((p.ep & EP_ACC_ADD) ? reinterpret_cast<uintptr_t>(p.acc_in) |
                                                     reinterpret_cast<uintptr_t>(p.acc_out) : 0);
    return (all & 15) == 0;
}

template <class P, typename T, typename VT, int E, unsigned EPM, int NT = kBlock>
hipError_t launch_staged(SweepParams& p, int num_cus, hipStream_t s) {
    if constexpr (sizeof(T) == 4 && EPM != 0u) {
        if (paired<T>(p)) return launch_staged_w<P, T, VT, E, EPM, NT, 2>(p, num_cus, s);
    }
    return launch_staged_w<P, T, VT, E, EPM, NT, 1>(p, num_cus, s);
}

// Whether a launch is the adjoint step of a gradient with everything that the
// staged kernel reads a step ahead: all three sources, in 16-byte elements.
// Bound by its 6 vector streams; the direct kernel also re-reads its neighbours
// through the caches: TI 64^3 nb 8 182 us per step, staged 140 (5.7 TB/s).
template <class P, typename T>
bool staged_adjoint(const SweepParams& p) {
    if (sizeof(T) != 8 || P::FAMILY == FAM_GENERIC || p.ep != EP_ADJOINT || p.colp != nullptr || !p.z) return false;
    const uintptr_t all = reinterpret_cast<uintptr_t>(p.gw[0]) | reinterpret_cast<uintptr_t>(p.gw[1]) |
                          reinterpret_cast<uintptr_t>(p.gw[2]) | reinterpret_cast<uintptr_t>(p.z);
    return p.gw[0] && p.gw[1] && p.gw[2] && (all & 15) == 0;
}

// Epilogue specialisations of the staged kernel: the Chebyshev step with
// fused dots (KPM), the series step (propagation, filters), the plain sweep
// or Chebyshev step without dots (with gamma = 0: no z stream at all), and
// every other combination with the flags read at run time.
template <class P, typename T, typename VT, int E>
hipError_t launch_staged_ep(SweepParams& p, int nt, int num_cus, hipStream_t s) {
    constexpr unsigned KPM = EP_STORE_Y | EP_MOMENTS, DOTS = EP_STORE_Y | EP_DOTS, SERIES = EP_SERIES,
                       PLAIN = EP_STORE_Y;
    if (p.colp == nullptr) {
        if constexpr (P::FAMILY != FAM_GENERIC) {
            if (nt == 512) {
                if (p.ep == KPM) return launch_staged<P, T, VT, E, KPM, 512>(p, num_cus, s);
                if (p.ep == DOTS) return launch_staged<P, T, VT, E, DOTS, 512>(p, num_cus, s);
                if (p.ep == SERIES) return launch_staged<P, T, VT, E, SERIES, 512>(p, num_cus, s);
                if (p.ep == PLAIN)
                    return p.gamma == 0.0 ? launch_staged<P, T, VT, E, PLAIN | EP_NO_Z, 512>(p, num_cus, s)
                                          : launch_staged<P, T, VT, E, PLAIN, 512>(p, num_cus, s);
            }
        }
        if (p.ep == KPM) return launch_staged<P, T, VT, E, KPM>(p, num_cus, s);
        if (p.ep == DOTS) return launch_staged<P, T, VT, E, DOTS>(p, num_cus, s);
        if (p.ep == SERIES) return launch_staged<P, T, VT, E, SERIES>(p, num_cus, s);
        if (p.ep == PLAIN)
            return p.gamma == 0.0 ? launch_staged<P, T, VT, E, PLAIN | EP_NO_Z>(p, num_cus, s)
                                  : launch_staged<P, T, VT, E, PLAIN>(p, num_cus, s);
    }
    if constexpr (sizeof(T) == 8 && E == 2) {
        // the run-time epilogue at two complex128 elements per lane needs more
        // than 256 VGPRs: one element per lane, default walk and workgroups
        SweepParams q = p;
        q.st_C = q.st_Bm = q.st_G8 = 0;
        const hipError_t e = launch_staged<P, T, VT, 1, 0u>(q, num_cus, s);
        p.grid = q.grid;
        return e;
    } else {
        return launch_staged<P, T, VT, E, 0u>(p, num_cus, s);
    }
}

// Epilogues the staged kernel takes by default: plain sweeps, the Chebyshev
// step with dots and the series steps; adjoint steps with all three sources
// where adjoint_default says so, other adjoint epilogues take the direct kernel,
// which issues their loads together with the neighbour loads.
// Small blocks (below 2^20 elements, cache resident) are launch-latency
// bound, where the direct kernel's single pass beats the staged walks.
bool large_block(const SweepParams& p) {
    return p.L[0] * p.L[1] * p.L[2] * p.n_orb * p.nb >= (int64_t(1) << 20);
}
bool staged_default(const SweepParams& p) { return (p.ep & (EP_GTERMS | EP_GRAD)) == 0 && large_block(p); }

// Adjoint steps with all three sources that are staged by default: on large
// blocks whose rows fill enough of the 256-number tiles (empty lanes load what
// the direct kernel does not).  Gradients of 32 moments, all direct | adjoint
// steps staged (us), with the fill of the tiles: TI 12x100x100 nb 4 (0.75)
// 1567 | 1259, 17x300x60 nb 4 (0.53) 3773 | 3525, 3x300x300 nb 8 (0.38) 7739 |
// 9125, 6x191x115 nb 2 (0.19) 1706 | 1926; in 2D, without side rows, graphene-2
// 30x20000 nb 1 (0.23) 1086 | 1034, 8x80000 nb 1 (0.06) 2828 | 2919.  Weyl steps
// stay direct unless asked for: their few neighbours cost little there, and
// ragged rows more here (direct | staged: 64^3 nb 16 4272 | 4194, 100x90x40
// nb 2 1182 | 1099, nb 8 3478 | 3759, nb 32 13203 | 13327).
template <class P>
bool adjoint_default(const SweepParams& p) {
    if (P::FAMILY == FAM_WEYL || !large_block(p)) return false;
    const int64_t rowel = p.L[0] * P::NO * p.nb, tiles = (rowel + kBlock - 1) / kBlock * kBlock;
    return P::DIM == 3 ? 2 * rowel >= tiles : 5 * rowel >= tiles;
}

// Elements per lane of a staged launch that asks for none: one for complex128,
// two for complex64 (one 16-byte chunk per lane and row either way).
// staged_tile says where the built-in families take more.
int staged_elems(const SweepParams& p) {
    static const int env_e = env_int("PV_STAGED_E", 0);
    if (p.st_E > 0) return p.st_E;
    if (env_e > 0) return env_e;
    return p.dtype == 0 ? 1 : 2;
}

// Tile of a staged launch of a built-in family that asks for no elements per
// lane and no workgroup size.  Longer tiles re-read less x halo (two sites per
// tile) and have more loads in flight, but fill ragged rows worse and make
// fewer walks, so each candidate's time is estimated as its walks' planes
// (StagedWalk) times the numbers of its tiles, padding included, times a weight:
// the ratio of times at equal work, with the share of a full round that the
// last one costs (512 lanes leave one workgroup per CU, which nothing
// balances).  Fitted to 454 launches on random and listed lattices of 2^22 to
// 2^27 numbers, each with all three tiles: the chosen one is 0.6% from the best
// on average, and more than 5% slower than the short one in 5 (at most 7%).
// us per sweep: short | 2x | 2x with 512 lanes, * the choice:
//   TI c128 256x256x64 nb 4      step 619 | 611 | 584*    plain 503 | 472 | 444*
//   TI c128 264x256x64 nb 4      step 662 | 663* | 699    plain 522 | 502* | 543
//   TI c128 64^3 nb 32           step 326 | 304 | 292*    plain 267 | 241 | 224*
//   TI c128 72x64x64 nb 32       step 379 | 376* | 413    plain 309 | 299* | 324
//   TI c128 64^3 nb 8            step 83 | 71* | 73       plain 62 | 54* | 58
//   TI c128 17x300x60 nb 16      step 210* | 235 | 342    plain 184* | 194 | 296
//   TI c64 256x256x64 nb 4       step 320 | 275* | 288    plain 267 | 226* | 234
//   TI c64 65^3 nb 8             step 61* | 73 | 91       plain 50* | 61 | 79
//   Weyl c128 130x130x60 nb 4    step 96* | 102 | 136     plain 72* | 87 | 122
//   graphene 512x512 c128 nb 32  step 276 at 512 lanes, 330 short
// The accumulating series step carries two more streams and keeps the short tile
// in 3D: at twice the registers per lane it loses (TI c128 64^3 nb 8 113 | 129).
struct StagedTile {
    int e, nt;
};
template <class P, typename T>
StagedTile staged_tile(const SweepParams& p, int num_cus) {
    static const int env_e = env_int("PV_STAGED_E", 0);
    const int e0 = staged_elems(p);
    const StagedTile t0{e0, p.st_nt == 512 ? 512 : kBlock};
    if (P::FAMILY == FAM_GENERIC || p.st_E > 0 || p.st_nt > 0 || env_e > 0 || p.colp != nullptr) return t0;
    const int64_t n = p.L[0] * p.L[1] * p.L[2] * P::NO * p.nb;
    const bool series = p.ep == EP_SERIES;
    const bool step = p.ep == (EP_STORE_Y | EP_DOTS) || p.ep == (EP_STORE_Y | EP_MOMENTS);
    if (n < (int64_t(1) << 22) || !(series || step || p.ep == EP_STORE_Y) || (series && P::DIM == 3)) return t0;
    const int rowel = int(p.L[0]) * P::NO * p.nb;
    auto time = [&](StagedTile t, double weight, double last) {
        const int TW = t.nt * t.e, nxs = (rowel + TW - 1) / TW;
        int G8 = p.st_G8 > 0 ? p.st_G8 : (num_cus >= 8 ? num_cus / 8 : 1) * (t.nt == kBlock ? 2 : 1);
        if (G8 > 256) G8 = 256;
        return weight * staged_walk<P>(p, nxs, G8, false).planes(G8, last) * G8 * TW;
    };
    StagedTile best = t0;
    double t_best = time(t0, 1.0, 0.2);
    auto consider = [&](int nt, double weight, double last) {
        const StagedTile t{2 * e0, nt};
        const double tt = time(t, weight, last);
        if (tt < t_best) {
            t_best = tt;
            best = t;
        }
    };
    const bool c128 = sizeof(T) == 8;
    if (P::DIM == 2) {
        consider(512, c128 ? 0.80 : 0.88, 0.9);
    } else if (!c128) {
        consider(kBlock, 0.82, 0.9);
    } else if (n >= (int64_t(1) << 24)) {   // vectors of 256 MiB: halo re-reads miss the last-level cache
        consider(kBlock, 0.92, 0.3);
        consider(512, 0.90, 0.9);
    } else {
        consider(kBlock, 0.80, 0.5);
    }
    return best;
}

template <class X>
struct Tag {
    using type = X;
};

// Sweep kernel of a launch: the staged kernel for compiled families, and for
// generic 3D stencils with no offset that has both a y and a z step, when
// the block is 16-byte aligned (its chunk loads); else the direct kernel.
// p.kernel (or PV_SWEEP) 1 forces direct, 2 staged; p.st_E (or PV_STAGED_E)
// selects the elements per lane.
enum class Route { DIRECT, STAGED, STAGED_ADJOINT };
template <class P, typename T>
Route sweep_route(const SweepParams& p) {
    static const int env_kernel = env_int("PV_SWEEP", 0);
    const int kind = p.kernel > 0 ? p.kernel : env_kernel;
    const bool aligned = ((reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.zero_row)) & 15) == 0;
    // generic stencils default to staged only on 3D lattices (walks along z)
    const bool can = P::FAMILY != FAM_GENERIC || p.generic_stageable;
    const bool adjoint = staged_adjoint<P, T>(p);
    const bool dflt = (staged_default(p) || (adjoint && adjoint_default<P>(p))) &&
                      (P::FAMILY != FAM_GENERIC || p.L[2] > 1);
    // a site must be whole 16-byte chunks: ring rows start one site
    // before the tile and wrap by whole chunks (complex64 with
    // n_orb * nb = 1 is half a chunk per site: direct kernel)
    const bool whole = (P::NO * p.nb * int(sizeof(cplx<T>))) % 16 == 0;
    if (!can || !aligned || !whole || P::NO * p.nb > STAGED_MAX_SITE || kind == 1 || (kind == 0 && !dflt))
        return Route::DIRECT;
    return adjoint ? Route::STAGED_ADJOINT : Route::STAGED;
}

template <class P, typename T, typename VT>
hipError_t launch_typed(SweepParams& p, int num_cus, hipStream_t s) {
    const Route route = sweep_route<P, T>(p);
    if constexpr (sizeof(T) == 8 && P::FAMILY != FAM_GENERIC) {
        // one number per lane whatever the shape says: the six vectors of a
        // second one do not fit the registers (a longer tile's walk and
        // workgroups are not this one's)
        if (route == Route::STAGED_ADJOINT) {
            SweepParams q = p;
            if (staged_elems(p) != 1) q.st_C = q.st_Bm = q.st_G8 = 0;
            const hipError_t e = launch_staged<P, T, VT, 1, EP_ADJOINT>(q, num_cus, s);
            p.grid = q.grid;
            return e;
        }
    }
    if (route != Route::DIRECT) {
        const auto [e, nt] = staged_tile<P, T>(p, num_cus);
        auto staged = [&, e = e, nt = nt](auto pt) -> hipError_t {
            using Q = typename decltype(pt)::type;
            if constexpr (sizeof(T) == 8)
                return e == 2 ? launch_staged_ep<Q, T, VT, 2>(p, nt, num_cus, s)
                              : launch_staged_ep<Q, T, VT, 1>(p, nt, num_cus, s);
            else
                return e == 4 ? launch_staged_ep<Q, T, VT, 4>(p, nt, num_cus, s)
                              : launch_staged_ep<Q, T, VT, 2>(p, nt, num_cus, s);
        };
        if constexpr (P::FAMILY == FAM_GENERIC) {
            if (p.generic_side_halo) return staged(Tag<PatGeneric<P::NO, true>>{});
        }
        return staged(Tag<P>{});
    }
    KArgs<T, VT> a;
    make_kargs<P, T, VT>(p, false, a);
    p.grid = int(8 * ((a.ntiles + a.tpb - 1) / a.tpb));
    hipLaunchKernelGGL((sweep_kernel<P, T, VT>), dim3(p.grid), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

template <class P>
hipError_t launch_family(SweepParams& p, int num_cus, hipStream_t s) {
    if (p.dtype == 0) {
        if (p.vtype != 0) return hipErrorInvalidValue;
        return launch_typed<P, double, double>(p, num_cus, s);
    }
    if (p.vtype == 0) return launch_typed<P, float, double>(p, num_cus, s);
    return launch_typed<P, float, float>(p, num_cus, s);
}


// Calls f(Tag<T>, Tag<VT>) for the vector and field types of a launch.
template <class F>
hipError_t dispatch_types(int dtype, int vtype, F&& f) {
    if (dtype == 0) {
        if (vtype != 0) return hipErrorInvalidValue;
        return f(Tag<double>{}, Tag<double>{});
    }
    if (vtype == 0) return f(Tag<float>{}, Tag<double>{});
    return f(Tag<float>{}, Tag<float>{});
}

// Calls f(IntC<E>, IntC<NT>, IntC<W>) for a batched staged launch: elements per
// lane, lanes and columns per element (two for complex64 blocks of at least two
// columns: a batch's vectors are 16-byte aligned).
template <typename T, class F>
void batch_shape(const SweepParams& p, F&& f) {
    constexpr int E0 = sizeof(T) == 8 ? 1 : 2, E1 = 2 * E0;
    const bool e1 = staged_elems(p) == E1, w512 = p.st_nt == 512;
    auto lanes = [&](auto ke) {
        auto go = [&](auto kn) {
            if constexpr (sizeof(T) == 4) {
                if (p.nb >= 2) {
                    f(ke, kn, IntC<2>{});
                    return;
                }
            }
            f(ke, kn, IntC<1>{});
        };
        if (w512) go(IntC<512>{});
        else go(IntC<kBlock>{});
    };
    if (e1) lanes(IntC<E1>{});
    else lanes(IntC<E0>{});
}

// Argument record of one instance of a batched sweep and its workgroup count.
template <class P>
hipError_t batch_fill_record_fam(const SweepParams& p, int staged, void* dst, int* nblocks) {
    return dispatch_types(p.dtype, p.vtype, [&](auto tt, auto tv) -> hipError_t {
        using T = typename decltype(tt)::type;
        using VT = typename decltype(tv)::type;
        static_assert(sizeof(KArgs<T, VT>) == sizeof(KArgs<double, double>), "record sizes differ");
        KArgs<T, VT> a;
        if constexpr (P::FAMILY != FAM_GENERIC) {
            if (staged) {
                if (P::NO * p.nb > STAGED_MAX_SITE || (P::NO * p.nb * int(sizeof(cplx<T>))) % 16 != 0)
                    return hipErrorInvalidValue;
                make_kargs<P, T, VT>(p, false, a);
                int G8 = 0;
                batch_shape<T>(p, [&](auto ke, auto kn, auto kw) {
                    G8 = staged_setup<P, T, VT, decltype(ke)::value, decltype(kn)::value, decltype(kw)::value>(
                        p, 1 << 30, true, a);
                });
                std::memcpy(dst, &a, sizeof(a));
                *nblocks = 8 * G8;
                return hipSuccess;
            }
        }
        make_kargs<P, T, VT>(p, true, a);
        std::memcpy(dst, &a, sizeof(a));
        *nblocks = int((a.ntiles + a.tpb - 1) / a.tpb);
        return hipSuccess;
    });
}

// One step of a batched sweep: every instance's workgroups in one launch.
template <class P>
hipError_t launch_batch_sweep_fam(const SweepParams& p, int staged, const void* table, const int* block_inst,
                                  const int* inst_block0, int grid, int64_t part_off, hipStream_t s) {
    return dispatch_types(p.dtype, p.vtype, [&](auto tt, auto tv) -> hipError_t {
        using T = typename decltype(tt)::type;
        using VT = typename decltype(tv)::type;
        if constexpr (P::FAMILY != FAM_GENERIC) {
            if (staged) {
                constexpr unsigned KPM = EP_STORE_Y | EP_MOMENTS;
                if (p.ep != KPM) return hipErrorInvalidValue;
                hipError_t e = hipSuccess;
                batch_shape<T>(p, [&](auto ke, auto kn, auto kw) {
                    constexpr int E = decltype(ke)::value, NT = decltype(kn)::value, W = decltype(kw)::value;
                    const size_t lds = staged_lds_bytes<P, T, E, KPM, NT, W>();
                    if (lds > 65536) {
                        e = hipFuncSetAttribute(
                            reinterpret_cast<const void*>(&batch_staged_kernel<P, T, VT, E, KPM, NT, W>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
                        if (e != hipSuccess) return;
                    }
                    hipLaunchKernelGGL((batch_staged_kernel<P, T, VT, E, KPM, NT, W>), dim3(grid), dim3(NT), lds, s,
                                       static_cast<const KArgs<T, VT>*>(table), block_inst, inst_block0, part_off);
                    e = hipGetLastError();
                });
                return e;
            }
        }
        hipLaunchKernelGGL((batch_sweep_kernel<P, T, VT>), dim3(grid), dim3(kBlock), 0, s,
                           static_cast<const KArgs<T, VT>*>(table), block_inst, inst_block0, part_off);
        return hipGetLastError();
    });
}

#endif  // PV_RTC
}  // namespace

#ifndef PV_RTC
// One translation unit per family (pv_fam_*.hip) defines these.
#define PV_FAMILY_ENTRY_POINTS(name)                                                                          \
    hipError_t launch_sweep_##name(SweepParams& p, int num_cus, hipStream_t s);                              \
    hipError_t batch_fill_record_##name(const SweepParams& p, int staged, void* dst, int* nblocks);          \
    hipError_t launch_batch_sweep_##name(const SweepParams& p, int staged, const void* table,                \
                                         const int* block_inst, const int* inst_block0, int grid, int64_t part_off, \
                                         hipStream_t s);
PV_FAMILY_ENTRY_POINTS(ti)
PV_FAMILY_ENTRY_POINTS(graphene2)
PV_FAMILY_ENTRY_POINTS(graphene4)
PV_FAMILY_ENTRY_POINTS(weyl)
PV_FAMILY_ENTRY_POINTS(generic)
#undef PV_FAMILY_ENTRY_POINTS
#endif

}  // namespace pv
