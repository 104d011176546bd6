// fd_stencil.h -- gfx950 stencil kernels for the leapfrog acoustic update.
//
// One launch performs one time step of
//     u^{n+1} = 2 u^n - u^{n-1} + c * Lh u^n + sources,   c = (v dt / h)^2,
// where Lh = h^2 L is the radius-R star stencil applied on every axis (the xy
// stencil form of Sec. 1 of Medina, St-Cyr and Warburton, extended to z with
// the same radius and spacing).  For R <= 4 the forward evaluates it in
// difference form,
//     Lh u = sum_axes sum_l w_l [ (u_{+l} - u) + (u_{-l} - u) ],
// algebraically the centre-weight form, which keeps FP32 rounding of smooth
// fields small and costs nothing there (the kernel is bandwidth-bound).  For
// R > 4 the vector work of that form limits the kernel, so it uses the
// centre-weight form of the paper, ndim w_0 u + sum_axes sum_l w_l (u_{+l} + u_{-l}),
// two operations per neighbour pair instead of four.
//
// Design (a star stencil is not a dense contraction, so no MFMA):
//  - A workgroup owns a BX x BY tile of the xy plane and marches a chunk of z
//    planes.  Each thread owns VEC consecutive x points (one 16-byte vector) in
//    EY rows and keeps u^n of its column at planes z-R..z+R in registers (the
//    z "register queue"); the plane z with an R-wide x/y halo is staged in LDS
//    (double buffered, one barrier per plane) for the x and y neighbours.
//  - Global traffic is x-contiguous 16-byte vectors: u^n once per point (plus
//    the halo), u^{n-1} and c streamed with nontemporal loads, u^{n+1} written
//    with nontemporal stores.  Every load of the next plane is issued one plane
//    ahead of its use, and without a branch (see plane_buf).
//  - Receivers are fused: a CSR event list over (x, y) columns, sorted by z, gives
//    each thread the next plane where one of its columns has an event, and the events
//    there when it starts.  One or two sources travel in the shot descriptor, more of
//    them in the event list.  The descriptor itself is a launch argument.
//  - Workgroup ids are remapped so that a contiguous run of tiles lands on one
//    XCD (workgroups are dealt round-robin to the 8 XCDs), which keeps halo
//    re-reads inside that XCD's L2.
//
// Field layout (padded): element (x, y, z) of the interior sits at
// off0 + z * pxy + y * px + x; at least R zero ghost cells surround the
// interior on every face (the zero solution outside the domain, Sec. 1) and
// rows/planes carry alignment padding so that every tile load is in bounds.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "fd_types.h"

#pragma clang fp contract(off)

namespace fdw {

// ------------------------------------------------------------------ weights

constexpr unsigned __int128 gcd_u128(unsigned __int128 a, unsigned __int128 b)
{
    while (b != 0) {
        const unsigned __int128 t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// Exact central weight of the radius-r second-derivative stencil:
// w_l = 2 (-1)^{l+1} (r!)^2 / (l^2 (r-l)! (r+l)!) = 2 (-1)^{l+1} [r!/(r-l)!] / (l^2 [(r+l)!/r!]).
// The fraction is reduced in 128-bit integers; for r <= 12 its reduced numerator and
// denominator are below 2^53, so the one division is correctly rounded.
constexpr double stencil_weight(int r, int l)
{
    unsigned __int128 num = 2, den = (unsigned __int128)(l * l);
    for (int i = r - l + 1; i <= r; ++i) num *= (unsigned)i;
    for (int i = r + 1; i <= r + l; ++i) den *= (unsigned)i;
    const unsigned __int128 g = gcd_u128(num, den);
    num /= g;
    den /= g;
    const double w = (double)(uint64_t)num / (double)(uint64_t)den;
    return (l % 2 == 1) ? w : -w;
}

template <int R>
struct StencilWeights {
    double w[R + 1];
    constexpr StencilWeights() : w()
    {
        double s = 0.0;
        for (int l = 1; l <= R; ++l) {
            w[l] = stencil_weight(R, l);
            s += w[l];
        }
        w[0] = -2.0 * s;
    }
};

// ------------------------------------------------------------------ x vectors

// N consecutive x points of one row, moved with one load or store instruction.  The
// kernels use 16-byte vectors (4 floats, 2 doubles) unless a tile asks for 8-byte ones.
template <typename T, int N>
struct VecT {
    typedef T t __attribute__((ext_vector_type(N)));
};
template <typename T>
struct V16 {
    static constexpr int N = 16 / (int)sizeof(T);
};

template <typename T, int N>
__device__ __forceinline__ void vld(T (&d)[N], const T *p)
{
    typename VecT<T, N>::t v = *reinterpret_cast<const typename VecT<T, N>::t *>(p);
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = v[i];
}

template <typename T, int N>
__device__ __forceinline__ void vld_nt(T (&d)[N], const T *p)
{
    typename VecT<T, N>::t v = __builtin_nontemporal_load(reinterpret_cast<const typename VecT<T, N>::t *>(p));
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = v[i];
}

template <typename T, int N>
__device__ __forceinline__ void vst(T *p, const T (&s)[N])
{
    typename VecT<T, N>::t v;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s[i];
    *reinterpret_cast<typename VecT<T, N>::t *>(p) = v;
}

template <typename T, int N>
__device__ __forceinline__ void vst_nt(T *p, const T (&s)[N])
{
    typename VecT<T, N>::t v;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s[i];
    __builtin_nontemporal_store(v, reinterpret_cast<typename VecT<T, N>::t *>(p));
}

template <typename T, int N>
__device__ __forceinline__ void vzero(T (&d)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = T(0);
}

// A whole number kept in the register of a floating one.
template <typename T>
__device__ __forceinline__ T bits_of(int i)
{
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, (int64_t)i);
    else
        return __builtin_bit_cast(T, i);
}
__device__ __forceinline__ int bits_to_int(float x) { return __builtin_bit_cast(int, x); }
__device__ __forceinline__ int bits_to_int(double x) { return (int)__builtin_bit_cast(int64_t, x); }

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of
// logical tile ids so that neighbouring tiles share an L2.  Bijective for any G.
__device__ __forceinline__ int xcd_remap(int b, int G)
{
    constexpr int NX = 8;
    const int q = G / NX, rem = G % NX;
    const int xcd = b % NX, idx = b / NX;
    return (xcd < rem) ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
}

// Calls f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): the index is a
// compile-time constant inside f whatever the loop unroller decides.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ int lower_bound_z(const Event *ev, int lo, int hi, int z)
{
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (ev[mid].z < z)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// ------------------------------------------------------------------ tile configuration

// Elements of LDS to declare for a kernel that uses `used`, so that no more than `waves` waves
// per SIMD (0: no limit) fit on a compute unit, in workgroups of nt threads.  A compute unit
// hands out its 160 KB in 128 units of 1280 bytes.
template <typename T>
constexpr int lds_limited(int used, int waves, int nt)
{
    const int least = waves ? (128 / (waves * 256 / nt + 1) + 1) * 1280 / (int)sizeof(T) : 0;
    return used > least ? used : least;
}

template <typename T, int R_, int NDIM_, int TXN_, int TYN_, int EY_, int VEC_ = V16<T>::N, int OCC_ = 0,
          bool LEAN_ = (OCC_ > 0), int HOFF_ = -1>
struct TileCfg {
    typedef T type;
    // OCC > 0: the forward kernel is built for OCC waves per SIMD (the compiler keeps to
    // the matching register budget).  LEAN: it keeps one set of prefetch registers instead
    // of two.  HOFF: planes the halo is fetched ahead of its use, through a ring of HOFF + 2
    // LDS planes (R for R <= 4, one less in the 4-wave builds, whose ring is smaller; 0 for
    // larger radii, whose ring would need too much LDS, and where the tile asks for it)
    static constexpr int OCC = OCC_;
    static constexpr int R = R_;
    static constexpr int NDIM = NDIM_;
    static constexpr int TXN = TXN_;                       // threads along x
    static constexpr int TYN = (NDIM_ == 3) ? TYN_ : 1;    // threads along y
    static constexpr int EY = (NDIM_ == 3) ? EY_ : 1;      // rows per thread
    static constexpr int VEC = VEC_;                       // x points per thread (one vector)
    static constexpr int NT = TXN * TYN;
    static constexpr int BX = TXN * VEC;
    static constexpr int BY = TYN * EY;
    static constexpr int LPAD = (R + VEC - 1) / VEC * VEC; // x halo rounded to vectors
    static constexpr int LW = BX + 2 * LPAD;               // LDS row length
    static constexpr int HY = (NDIM == 3) ? R : 0;         // y halo rows
    static constexpr int GZ = R;                           // ghost planes
    static constexpr int LH = BY + 2 * HY;
    static constexpr int LDS = LW * LH;                    // elements per LDS plane
    static constexpr int NXV = 2 * LPAD / VEC + 1;         // vectors read per row for x neighbours
    static constexpr int NHY = 2 * HY * TXN;               // y-halo vectors per plane
    static constexpr int NHS = LPAD / VEC;                 // x-halo vectors per side per row
    static constexpr int NHX = 2 * BY * NHS;
    static constexpr int NH = NHY + NHX;
    static constexpr int HPT = (NH + NT - 1) / NT;         // halo vectors per thread
    static constexpr int YR = EY + 2 * HY;                 // rows a thread touches along y
    static constexpr bool LEAN = LEAN_;
    static constexpr int HOFF = HOFF_ >= 0 ? HOFF_ : (R <= 4) ? (OCC_ >= 4 ? R - 1 : R) : 0;
    static constexpr int NB = HOFF + 2;
    // Waves per SIMD that the forward kernel may hold (0: what its registers allow).  With one
    // more the chunks of the larger grids get shorter or the compute unit streams more rows at
    // once: 512^3 r = 4 388 us against 352, 320^3 r = 6 109 against 94, 201x119x333 r = 5 31.2
    // against 27.5, 512^3 r = 3 damped 378 against 369 (where no limit stands, both measure
    // the same or the registers allow no more).
    static constexpr int max_waves(bool damp)
    {
        if (NDIM < 3 || OCC > 0 || VEC * (int)sizeof(T) < 16) return 0;
        if (NT == 512 && R == 3 && damp) return 2;
        if (NT == 512 && sizeof(T) == 4) return R == 4 ? 2 : R == 1 ? 4 : 0;
        if (NT == 256 && R == 5 && sizeof(T) == 8 && damp) return 2;
        return (NT == 128 && R == 5) || (NT == 256 && R == 6) ? 2 : 0;
    }
    static constexpr int lds_fwd(bool damp) { return lds_limited<T>(NB * LDS, max_waves(damp), NT); }
    static_assert(256 % BX == 0 && 64 % BY == 0, "tile must divide the layout alignment");
};

// ------------------------------------------------------------------ plane access

// One plane of a padded field as a raw buffer: a uniform base and a 32-bit byte offset per
// lane.  A lane whose offset is kOffGrid, and every lane when `on` is false, is out of the
// buffer's range: its load returns zero and its store is dropped, both without memory
// traffic.  So the plane loop masks lanes and the last plane without a branch, which keeps
// the number of loads in flight the same on every path: with branches around the loads the
// compiler has to assume the path that issued fewest and waits for the loads it has just
// issued.  (A plane holds less than 2 GiB, so kOffGrid is outside every plane.)
constexpr uint32_t kOffGrid = 0x80000000u;
constexpr int kNontemporal = 2;  // cache policy bit of the buffer instructions

// Cache policy of the loads of fields that a step reads point by point (u^{n-1}, c, ...):
// CACHED where a step's fields stay in the last-level cache until the next step reads them
// again, nontemporal otherwise (the host decides, cache_keeps()).
template <bool CACHED>
constexpr int kPointLoads = CACHED ? 0 : kNontemporal;

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_buf(const T *base, int64_t pxy, int zp, bool on = true)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base + (int64_t)zp * pxy), 0,
                                             on ? (int)(pxy * (int64_t)sizeof(T)) : 0, 0x00027000);
}

// A pointer read from memory, known to be to device memory: a flat access may be to LDS as
// well, so any of them in a rare branch makes the plane loop wait for all loads and all of
// LDS where the branch joins (a batch of one 400^3 shot: 237 us per step against 200).
template <typename P>
__device__ __forceinline__ P *as_global(P *p)
{
    return (P *)(__attribute__((address_space(1))) P *)(uintptr_t)p;
}

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int AUX, typename T, int N>
__device__ __forceinline__ void bld(T (&d)[N], __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    typename VecT<T, N>::t v;
    if constexpr (N * sizeof(T) == 16)
        v = __builtin_bit_cast(typename VecT<T, N>::t, (i32x4)__builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX));
    else
        v = __builtin_bit_cast(typename VecT<T, N>::t, (i32x2)__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX));
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = v[i];
}

template <typename T>
__device__ __forceinline__ T bld1(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, (i32x2)__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else
        return __builtin_bit_cast(T, (int)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

template <int AUX, typename T, int N>
__device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, uint32_t off, const T (&s)[N])
{
    typename VecT<T, N>::t v;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s[i];
    if constexpr (N * sizeof(T) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), r, off, 0, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, v), r, off, 0, AUX);
}

// Per-thread geometry of one tile, shared by the forward and adjoint kernels.  Offsets are
// bytes within a plane, or kOffGrid for a vector that no point of the grid needs.
template <class C>
struct TileGeom {
    int lx, ly, gx, gy, x0, y0, z0, z1;
    uint32_t obl[C::EY];     // row e, inside the grid or its R-wide ghost ring (the field the stencil reads)
    uint32_t obr[C::EY];     // row e, inside the grid (point-wise operands, results)
    bool rin[C::EY];         // row e lies inside the grid
    uint32_t hob[C::HPT];    // halo vector k
    int hl[C::HPT];          // halo vector k: LDS offset
    bool hval;               // the last halo vector exists (the others always do)

    template <class Desc>
    __device__ __forceinline__ void init(const Desc &s, int tx, int ty, int cz, int zch, int tid)
    {
        typedef typename C::type T;
        lx = (tid % C::TXN) * C::VEC;
        ly = (tid / C::TXN) * C::EY;
        x0 = tx * C::BX;
        y0 = ty * C::BY;
        gx = x0 + lx;
        gy = y0 + ly;
        z0 = cz * zch;
        z1 = min(z0 + zch, s.nz);
        const int px = (int)s.px;  // a row is shorter than a plane, which is under 2 GiB
        const int base = (int)(s.off0 - (int64_t)C::GZ * s.pxy);  // interior (0, 0) within its plane
#pragma unroll
        for (int e = 0; e < C::EY; ++e) {
            rin[e] = (gx < s.nx) && (gy + e < s.ny);
            const bool lin = (gx < s.nx + C::R) && (gy + e < s.ny + C::HY);
            const uint32_t ob = (uint32_t)(base + (gy + e) * px + gx) * (uint32_t)sizeof(T);
            obl[e] = lin ? ob : kOffGrid;
            obr[e] = rin[e] ? ob : kOffGrid;
        }
        hval = tid + (C::HPT - 1) * C::NT < C::NH;
#pragma unroll
        for (int k = 0; k < C::HPT; ++k) {
            const int hv = tid + k * C::NT;
            int ry = 0, cx = 0;
            if (hv < C::NHY) {
                const int ri = hv / C::TXN;
                cx = (hv % C::TXN) * C::VEC;
                ry = (ri < C::HY) ? ri - C::HY : C::BY + (ri - C::HY);
            } else if (hv < C::NH) {
                const int hx = hv - C::NHY;
                ry = hx / (2 * C::NHS);
                const int si = hx % (2 * C::NHS);
                cx = (si < C::NHS) ? -C::LPAD + si * C::VEC : C::BX + (si - C::NHS) * C::VEC;
            }
            const bool need = hv < C::NH && x0 + cx < s.nx + C::R && y0 + ry < s.ny + C::HY;
            hob[k] = need ? (uint32_t)(base + (y0 + ry) * px + (x0 + cx)) * (uint32_t)sizeof(T) : kOffGrid;
            hl[k] = (ry + C::HY) * C::LW + (cx + C::LPAD);
        }
    }
    __device__ __forceinline__ bool has(int k) const { return k + 1 < C::HPT || hval; }
};

// ------------------------------------------------------------------ sources and receivers

// Column bounds of this thread's events, loaded before the fields so that the look-ups that
// depend on them overlap with those loads.
template <class C>
struct EventBounds {
    int p[C::EY][C::VEC + 1];
    bool any;  // uniform: the chunk holds planes with events

    template <class Desc>
    __device__ __forceinline__ void load(const Desc &s, const TileGeom<C> &g)
    {
        any = s.ev_ptr && s.ev_zlo < g.z1 && s.ev_zhi >= g.z0;
        if (!any) return;
#pragma unroll
        for (int e = 0; e < C::EY; ++e) {
            const int row = min(g.gy + e, s.ny - 1) * s.nx;
#pragma unroll
            for (int v = 0; v <= C::VEC; ++v) p[e][v] = s.ev_ptr[row + min(g.gx + v, s.nx)];
        }
    }
};

// The next plane z at which this thread's columns have an event.  While no column has more
// than one event left, the usual case of receivers, `code` holds the event of each column
// at that plane (kNoEvent: none) and the plane needs no look-up when it comes.  Otherwise
// (`look`) it holds the place in the list of each column's next event (kNoEvent: none left),
// which is read when its plane comes.  That waits for all loads of the next plane, but once a
// plane: a search from the column's bounds, as many times as the list is deep, had a column of
// receivers cost 64^3 r = 4 8.2 us per step instead of 6.3, 256^3 103 instead of 67.
constexpr int kNoEvent = -0x7fffffff - 1;

// Waits for this wave's loads (vmcnt 0).  At the end of a branch that has waited for all but
// some lanes' loads, it keeps the compiler from waiting for those in the plane loop, and so
// for the fields' loads with them.
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }

template <class C>
struct EventNext {
    int z, code[C::EY][C::VEC];
    bool look;

    template <class Desc>
    __device__ __forceinline__ void first(const Desc &s, const TileGeom<C> &g, const EventBounds<C> &b)
    {
        z = 0x7fffffff;
        look = false;
        int ez[C::EY][C::VEC], first_z[C::EY][C::VEC];
#pragma unroll
        for (int e = 0; e < C::EY; ++e)
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) code[e][v] = kNoEvent;
        bool mine = false;
#pragma unroll
        for (int e = 0; e < C::EY; ++e)
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) mine = mine || (g.rin[e] && b.p[e][v] < b.p[e][v + 1]);
        if (!b.any || !mine) return;
        // the first event of each column (of the list, where it has none)
#pragma unroll
        for (int e = 0; e < C::EY; ++e)
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) {
                const Event *ev = s.ev + (b.p[e][v] < b.p[e][v + 1] ? b.p[e][v] : 0);
                ez[e][v] = first_z[e][v] = ev->z;
                code[e][v] = ev->code;
            }
#pragma unroll
        for (int e = 0; e < C::EY; ++e)
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) {
                const int n = g.rin[e] ? b.p[e][v + 1] - b.p[e][v] : 0;
                const bool one = n == 1 && ez[e][v] >= g.z0;
                look = look || n > 1;
                code[e][v] = one ? code[e][v] : kNoEvent;
                ez[e][v] = one ? ez[e][v] : 0x7fffffff;
                z = min(z, ez[e][v]);
            }
        // events of one thread on several planes, too, are looked up
#pragma unroll
        for (int e = 0; e < C::EY; ++e)
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) look = look || (code[e][v] != kNoEvent && ez[e][v] != z);
        if (look) seek(s, g, b, first_z);
        loads_done();
    }

    // the first event of each column from plane z0 on
    template <class Desc>
    __device__ __forceinline__ void seek(const Desc &s, const TileGeom<C> &g, const EventBounds<C> &b,
                                         const int (&first_z)[C::EY][C::VEC])
    {
        z = 0x7fffffff;
        static_for<C::EY * C::VEC>([&](auto slot) __attribute__((always_inline)) {
            constexpr int e = decltype(slot)::value / C::VEC, v = decltype(slot)::value % C::VEC;
            const int lo = b.p[e][v], hi = g.rin[e] ? b.p[e][v + 1] : lo;
            int at = lo, at_z = lo < hi ? first_z[e][v] : 0x7fffffff;
            // receivers of a column are mostly on consecutive planes, a few planes with more
            // events than one among them: two steps of that length, then a search
            for (int i = 0; i < 2 && at_z < g.z0; ++i) {
                const int to = min(at + (g.z0 - at_z), hi);
                const int before = s.ev[to - 1].z, to_z = s.ev[min(to, hi - 1)].z;
                if (before >= g.z0) break;
                at = to;
                at_z = to < hi ? to_z : 0x7fffffff;
            }
            if (at_z < g.z0) {
                at = lower_bound_z(s.ev, at + 1, hi, g.z0);
                at_z = at < hi ? s.ev[at].z : 0x7fffffff;
            }
            code[e][v] = at < hi ? at : kNoEvent;
            z = min(z, at_z);
        });
    }
};

// Runs f(code, row, lane) over the events of this thread's columns at plane z in list order
// (row and lane are compile-time constants) and moves the columns' places in `at` past them;
// returns the next plane with an event.  (The entry behind the list's last is workspace, too.)
template <class C, class Desc, class F>
__device__ __forceinline__ int look_events(const Desc &s, const TileGeom<C> &g, int (&at)[C::EY][C::VEC], int z, F &&f)
{
    int nxt = 0x7fffffff;
    static_for<C::EY * C::VEC>([&](auto slot) __attribute__((always_inline)) {
        constexpr int e = decltype(slot)::value / C::VEC, v = decltype(slot)::value % C::VEC;
        int p = at[e][v];
        if (p == kNoEvent) return;
        const int hi = s.ev_ptr[(g.gy + e) * s.nx + g.gx + v + 1];
        Event ev = s.ev[p], next = s.ev[p + 1];
        while (ev.z == z) {
            f(ev.code, std::integral_constant<int, e>{}, std::integral_constant<int, v>{});
            if (++p == hi) break;
            ev = next;
            if (ev.z == z) next = s.ev[p + 1];
        }
        at[e][v] = p < hi ? p : kNoEvent;
        if (p < hi) nxt = min(nxt, ev.z);
    });
    loads_done();
    return nxt;
}

// ------------------------------------------------------------------ forward step

// Address of byte offset `ob` inside plane zp of a padded field (plane pitch pxy elements).
template <typename T>
__device__ __forceinline__ const T *plane_at(const T *base, int64_t pxy, int zp, uint32_t ob)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base + (int64_t)zp * pxy) + ob);
}
template <typename T>
__device__ __forceinline__ T *plane_at(T *base, int64_t pxy, int zp, uint32_t ob)
{
    return reinterpret_cast<T *>(reinterpret_cast<char *>(base + (int64_t)zp * pxy) + ob);
}

// One leapfrog step over this workgroup's tile and z chunk.
//
// The z register queue has P = 2R+2 slots: planes z-R .. z+R of the current plane
// z plus one slot receiving plane z+R+1 while z is computed; it shifts by one slot
// per plane.  (Unrolling the plane loop by P to rotate the queue instead removes the
// register moves but multiplies the code size, and measured slower on gfx950.)
//
// Halo timing: the x/y halo of a plane is interior data of the neighbouring tiles.
// With HOFF = R the halo of plane z+R+1 is fetched in the same iteration in which
// the neighbours fetch that plane as their queue tail, so the requests meet in L2,
// and it waits in a ring of NB = R+2 LDS plane buffers until the plane becomes the
// centre.  (Fetching it only when it is needed comes R planes later, by which time
// the XCD has streamed several MB and the lines have left its 4 MB L2.)  Plane p
// lives in buffer p mod NB: when iteration z writes the halo of plane z+R its buffer
// was last read by iteration z-2, and every thread passed the barrier of z-1.
//
// The plane loop is unrolled by 2 (static_for) so that the u^{n-1}, c and halo
// prefetch registers alternate between two sets by parity.
//
// What bounds it: HBM for large grids, the latency of a plane's loads, LDS and arithmetic for
// small ones.  Measured per step, with branches around the loads and the descriptor, event
// list and sponge factors read through memory one after another, and as it is here:
// 512^3 r = 4 383 -> 352 us (5.60 -> 6.10 TB/s of 16 B/pt; the three-workgroup tile would
// take 414: loads no longer waited for keep more places in memory open at once, so the
// one-workgroup 128x16 tile is the one to use), 256^3 56 -> 44, 384^3 r = 8 202 -> 171,
// 256^3 FP64 93 -> 85, 64^3 6.6 -> 5.3, 97x161x203 r = 2 with sponge 25.5 -> 13.0, 2-D
// 1203x801 r = 8 with sponge 12.5 -> 6.8 (of 256^3 1.5, of 64^3 0.2 and of the ragged grid
// 2.0 us are the cached loads and short chunks).  A launch that returns at once takes 2.3 us.
//
// DAMP: the sponge's per-axis factors are in s.damp (a null s.damp counts as all ones, for
// batches that mix damped and undamped shots); G = gx gy gz scales both time levels.
template <class C, bool DAMP, int LD>
__device__ __forceinline__ void fwd_tile(const ShotDesc &s, const typename C::type *__restrict__ cur,
                                         const typename C::type *prev, typename C::type *out,
                                         int64_t step, bool record, int tx, int ty, int cz,
                                         typename C::type *lds)
{
    typedef typename C::type T;
    constexpr int R = C::R, VEC = C::VEC, EY = C::EY, HPT = C::HPT, HY = C::HY;
    constexpr int HOFF = C::HOFF, NB = C::NB;
    constexpr StencilWeights<R> W{};
    const T *__restrict__ cc = static_cast<const T *>(s.c);
    const int64_t pxy = s.pxy;

    TileGeom<C> g;
    g.init(s, tx, ty, cz, s.zch, threadIdx.x);
    if (g.z0 >= g.z1) return;

    EventBounds<C> evb;
    evb.load(s, g);

    // the sample of a source inside this tile and chunk (at most kInlineSources, in s.isrc)
    int srcz[kInlineSources];
    T srcv[kInlineSources];
#pragma unroll
    for (int i = 0; i < kInlineSources; ++i) {
        const InlineSource &is = s.isrc[i];
        srcz[i] = -1;
        srcv[i] = T(0);
        if (i < s.nisrc && is.z >= g.z0 && is.z < g.z1 && is.x >= g.x0 && is.x < g.x0 + C::BX && is.y >= g.y0 &&
            is.y < g.y0 + C::BY && step < is.nsamp) {
            srcz[i] = is.z;
            srcv[i] = T(is.scale) * static_cast<const T *>(is.wav)[step];
        }
    }

    // LEAN: one register set for the u^{n-1}, c and halo prefetches (the next plane's
    // values are loaded into it once the current plane is done with it) instead of two
    constexpr bool LEAN = C::LEAN;
    constexpr int NSET = LEAN ? 1 : 2;
    constexpr int P = 2 * R + 2;
    T q[P][EY][VEC];
    T pv[NSET][EY][VEC], cv[NSET][EY][VEC], hv[NSET][HPT][VEC];

    // prologue: planes z0-R .. z0+R into slots 0 .. 2R; u^{n-1} and c of plane z0 into
    // set 0; halos of planes z0 .. z0+HOFF-1 into their LDS buffers and the halo of plane
    // z0+HOFF into set 0.  Every load is issued before the first one is waited for.
    T hp[HOFF > 0 ? HOFF : 1][HPT][VEC];
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) {
        const auto b = plane_buf(cur, pxy, g.z0 + k);
#pragma unroll
        for (int e = 0; e < EY; ++e) bld<0>(q[k][e], b, g.obl[e]);
    }
#pragma unroll
    for (int j = 0; j < HOFF; ++j) {
        const auto b = plane_buf(cur, pxy, g.z0 + j + R, g.z0 + j < g.z1);
#pragma unroll
        for (int k = 0; k < HPT; ++k) bld<0>(hp[j][k], b, g.hob[k]);
    }
    {
        const auto bp = plane_buf(prev, pxy, g.z0 + R), bc = plane_buf(cc, pxy, g.z0 + R);
#pragma unroll
        for (int e = 0; e < EY; ++e) {
            bld<LD>(pv[0][e], bp, g.obr[e]);
            bld<LD>(cv[0][e], bc, g.obr[e]);
        }
        const auto bh = plane_buf(cur, pxy, g.z0 + HOFF + R, g.z0 + HOFF < g.z1);
#pragma unroll
        for (int k = 0; k < HPT; ++k) bld<0>(hv[0][k], bh, g.hob[k]);
    }

    // absorbing sponge: G = gx gy gz scales both time levels (1 outside the sponge)
    T gxy[EY][VEC], gz[NSET];
    const bool damped = DAMP && s.damp;
    const auto bd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(s.damp), 0, damped ? (s.nx + s.ny + s.nz) * (int)sizeof(T) : 0, 0x00027000);
    auto load_gz = [&](int z) { return bld1<T>(bd, (uint32_t)(s.nx + s.ny + z) * (uint32_t)sizeof(T)); };
    if constexpr (DAMP) {
        T gx[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) gx[v] = bld1<T>(bd, (uint32_t)(g.gx + v) * (uint32_t)sizeof(T));
#pragma unroll
        for (int e = 0; e < EY; ++e) {
            const T gy = bld1<T>(bd, (uint32_t)(s.nx + g.gy + e) * (uint32_t)sizeof(T));
#pragma unroll
            for (int v = 0; v < VEC; ++v) gxy[e][v] = damped ? gx[v] * gy : T(1);
        }
        gz[0] = load_gz(g.z0);
    }

    EventNext<C> nev;
    nev.first(s, g, evb);
    int bz = g.z0 % NB;              // LDS buffer of plane z
    int bh = (g.z0 + HOFF) % NB;     // LDS buffer of plane z + HOFF
#pragma unroll
    for (int j = 0; j < HOFF; ++j) {
        T *L = lds + ((g.z0 + j) % NB) * C::LDS;
#pragma unroll
        for (int k = 0; k < HPT; ++k)
            if (g.has(k)) vst(L + g.hl[k], hp[j][k]);
    }
    const int64_t row = step - s.rec_base;
    T *const trow = record && row >= 0 && row < s.rec_cap ? static_cast<T *>(s.traces) + row * s.nrec : nullptr;

    for (int zb = g.z0; zb < g.z1; zb += NSET) {
        static_for<NSET>([&](auto st_) __attribute__((always_inline)) {
            constexpr int st = decltype(st_)::value;
            constexpr int cs = LEAN ? 0 : (st & 1), ns = LEAN ? 0 : (cs ^ 1);
            constexpr int tail = 2 * R + 1;  // slot receiving plane z+R+1
            constexpr int ctr = R;                // slot of plane z
            const int z = zb + st;
            if (z >= g.z1) return;
            const bool more = z + 1 < g.z1;
            {
                const auto bt = plane_buf(cur, pxy, z + 1 + 2 * R, more);
#pragma unroll
                for (int e = 0; e < EY; ++e) bld<0>(q[tail][e], bt, g.obl[e]);
            }
            if constexpr (!LEAN) {
                const auto bp = plane_buf(prev, pxy, z + 1 + R, more), bc = plane_buf(cc, pxy, z + 1 + R, more);
#pragma unroll
                for (int e = 0; e < EY; ++e) {
                    bld<LD>(pv[ns][e], bp, g.obr[e]);
                    bld<LD>(cv[ns][e], bc, g.obr[e]);
                }
                const auto bh2 = plane_buf(cur, pxy, z + 1 + HOFF + R, z + 1 + HOFF < g.z1);
#pragma unroll
                for (int k = 0; k < HPT; ++k) bld<0>(hv[ns][k], bh2, g.hob[k]);
            }
            if constexpr (DAMP && !LEAN) gz[ns] = load_gz(z + 1);

            // stage plane z's interior (from the queue) and plane z+HOFF's halo in LDS
            T *L = lds + bz * C::LDS;
#pragma unroll
            for (int e = 0; e < EY; ++e) vst(L + (g.ly + e + HY) * C::LW + C::LPAD + g.lx, q[ctr][e]);
            {
                T *LH = lds + bh * C::LDS;
#pragma unroll
                for (int k = 0; k < HPT; ++k)
                    if (g.has(k)) vst(LH + g.hl[k], hv[cs][k]);
            }
            if constexpr (LEAN) {  // the next halo, into the registers just staged
                const auto bh2 = plane_buf(cur, pxy, z + 1 + HOFF + R, z + 1 + HOFF < g.z1);
#pragma unroll
                for (int k = 0; k < HPT; ++k) bld<0>(hv[0][k], bh2, g.hob[k]);
            }
            __syncthreads();

            // y neighbour rows: yr[k] is row ly - HY + k at this thread's x vector
            T yr[C::YR][VEC];
#pragma unroll
            for (int k = 0; k < C::YR; ++k) {
                if (k >= HY && k < HY + EY) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) yr[k][v] = q[ctr][k - HY][v];
                } else {
                    vld(yr[k], L + (g.ly + k) * C::LW + C::LPAD + g.lx);
                }
            }

            T un[EY][VEC];
#pragma unroll
            for (int e = 0; e < EY; ++e) {
                T xs[C::NXV * VEC];
#pragma unroll
                for (int j = 0; j < C::NXV; ++j) {
                    T tmp[VEC];
                    if (j * VEC == C::LPAD) {  // this thread's own vector
#pragma unroll
                        for (int v = 0; v < VEC; ++v) tmp[v] = q[ctr][e][v];
                    } else {
                        vld(tmp, L + (g.ly + e + HY) * C::LW + g.lx + j * VEC);
                    }
#pragma unroll
                    for (int v = 0; v < VEC; ++v) xs[j * VEC + v] = tmp[v];
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const T u0 = q[ctr][e][v];
                    T acc;
                    if constexpr (R > 4) {
                        acc = T(C::NDIM * W.w[0]) * u0;
#pragma unroll
                        for (int l = 1; l <= R; ++l) acc = fma_t(T(W.w[l]), xs[C::LPAD + v + l] + xs[C::LPAD + v - l], acc);
                        if (C::NDIM == 3) {
#pragma unroll
                            for (int l = 1; l <= R; ++l) acc = fma_t(T(W.w[l]), yr[HY + e + l][v] + yr[HY + e - l][v], acc);
                        }
#pragma unroll
                        for (int l = 1; l <= R; ++l) acc = fma_t(T(W.w[l]), q[ctr + l][e][v] + q[ctr - l][e][v], acc);
                    } else {
                        acc = T(0);
#pragma unroll
                        for (int l = 1; l <= R; ++l)
                            acc = fma_t(T(W.w[l]), (xs[C::LPAD + v + l] - u0) + (xs[C::LPAD + v - l] - u0), acc);
                        if (C::NDIM == 3) {
#pragma unroll
                            for (int l = 1; l <= R; ++l)
                                acc = fma_t(T(W.w[l]), (yr[HY + e + l][v] - u0) + (yr[HY + e - l][v] - u0), acc);
                        }
#pragma unroll
                        for (int l = 1; l <= R; ++l)
                            acc = fma_t(T(W.w[l]), (q[ctr + l][e][v] - u0) + (q[ctr - l][e][v] - u0), acc);
                    }
                    if constexpr (DAMP) {
                        const T G = gxy[e][v] * (damped ? gz[cs] : T(1));
                        un[e][v] = G * fma_t(cv[cs][e][v], acc, T(2) * u0 - G * pv[cs][e][v]);
                    } else {
                        un[e][v] = fma_t(cv[cs][e][v], acc, T(2) * u0 - pv[cs][e][v]);
                    }
                }
            }

            if constexpr (LEAN) {  // u^{n-1} and c of the next plane, into the registers just used
                const auto bp = plane_buf(prev, pxy, z + 1 + R, more), bc = plane_buf(cc, pxy, z + 1 + R, more);
#pragma unroll
                for (int e = 0; e < EY; ++e) {
                    bld<LD>(pv[0][e], bp, g.obr[e]);
                    bld<LD>(cv[0][e], bc, g.obr[e]);
                }
                if constexpr (DAMP) gz[0] = load_gz(z + 1);
            }

            // fused sources (added before the store) and receivers (recorded after them)
#pragma unroll
            for (int i = kInlineSources - 1; i >= 0; --i)
                if (z == srcz[i]) {
#pragma unroll
                    for (int e = 0; e < EY; ++e)
#pragma unroll
                        for (int v = 0; v < VEC; ++v)
                            if (g.gx + v == s.isrc[i].x && g.gy + e == s.isrc[i].y) un[e][v] += srcv[i];
                }
            if (z == nev.z) {
                auto source = [&](int code, T u) {
                    const SourceInfo si = s.src[~code];
                    return step < si.nsamp ? u + T(si.scale) * as_global(static_cast<const T *>(si.wav))[step] : u;
                };
                if (!nev.look) {
#pragma unroll
                    for (int e = 0; e < EY; ++e)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            const int code = nev.code[e][v];
                            if (code >= 0) {
                                if (trow) trow[code] = un[e][v];
                            } else if (code != kNoEvent) {
                                un[e][v] = source(code, un[e][v]);
                            }
                        }
                    nev.z = 0x7fffffff;
                } else {
                    nev.z = look_events<C>(s, g, nev.code, z, [&](int code, auto e, auto v) __attribute__((always_inline)) {
                        if (code >= 0) {
                            if (trow) trow[code] = un[e][v];
                        } else {
                            un[e][v] = source(code, un[e][v]);
                        }
                    });
                }
            }

            // a vector that straddles the end of its row keeps the padding behind it zero
            const auto bo = plane_buf(out, pxy, z + R);
#pragma unroll
            for (int e = 0; e < EY; ++e) {
#pragma unroll
                for (int v = 1; v < VEC; ++v) un[e][v] = g.gx + v < s.nx ? un[e][v] : T(0);
                bst<kNontemporal>(bo, g.obr[e], un[e]);
            }
#pragma unroll
            for (int k = 0; k < P - 1; ++k)
#pragma unroll
                for (int e = 0; e < EY; ++e)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) q[k][e][v] = q[k + 1][e][v];
            bz = (bz + 1 == NB) ? 0 : bz + 1;
            bh = (bh + 1 == NB) ? 0 : bh + 1;
        });
    }
}

// Where a workgroup finds its shot's descriptor.  FROM_ARGS: in the launch arguments, where it
// is read with scalar loads that wait for nothing but the launch itself.  FROM_TABLE: in a
// batch's table in device memory, where each shot also counts its own steps.  FROM_CONTEXT: in
// the context's workspace, for captured launches, so that a replay finds the sources,
// receivers and sponge of its own time.  (One build for the last two costs small batches the
// choice of step and fields, 1-2 %: eight 256^2 FP32 r = 4 4.70 -> 4.80 us per step.)
enum { FROM_ARGS = 0, FROM_TABLE = 1, FROM_CONTEXT = 2 };

template <class C, int FROM, bool DAMP, int LD>
__device__ __forceinline__ void fwd_body(const LaunchArgs &a)
{
    typedef typename C::type T;
    __shared__ __attribute__((aligned(16))) T lds[C::lds_fwd(DAMP)];
    int wg = blockIdx.x;
    if (a.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    if constexpr (FROM == FROM_ARGS) {
        const ShotDesc &s = a.one;
        const int64_t step = a.step;
        const T *cur;
        const T *prev;
        T *out;
        if (a.cur) {
            cur = static_cast<const T *>(a.cur);
            prev = static_cast<const T *>(a.prev);
            out = static_cast<T *>(a.out);
        } else {
            cur = static_cast<const T *>(s.buf[step & 1]);
            prev = static_cast<const T *>(s.buf[(step + 1) & 1]);
            out = static_cast<T *>(s.buf[(step + 1) & 1]);
        }
        const int tx = wg % s.tiles_x;
        const int t2 = wg / s.tiles_x;
        const int ty = t2 % s.tiles_y;
        const int cz = t2 / s.tiles_y;
        if (cz >= s.chunks_z) return;
        fwd_tile<C, DAMP, LD>(s, cur, prev, out, step, a.record != 0, tx, ty, cz, lds);
    } else {
        int shot = a.shot0, local = wg;
        if (FROM == FROM_TABLE && a.nshots > 1) {
            wg += a.wg0;
            int lo = a.shot0, hi = a.shot0 + a.nshots;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (a.wg_prefix[mid] <= wg)
                    lo = mid;
                else
                    hi = mid;
            }
            shot = lo;
            local = wg - a.wg_prefix[lo];
        }
        ShotDesc *sp = a.shots + shot;
        int64_t step = a.step;
        if constexpr (FROM == FROM_TABLE) {
            step = sp->ctr[a.slot];
            const bool active = step < sp->target;
            if (local == 0 && threadIdx.x == 0) sp->ctr[a.slot ^ 1] = active ? step + 1 : step;
            if (!active) return;
        }
        // the descriptor but for its counters is constant while the steps run
        const __attribute__((address_space(4))) int *cp = (const __attribute__((address_space(4))) int *)(uintptr_t)sp;
        int words[sizeof(ShotDesc) / sizeof(int)];
#pragma unroll
        for (int i = 0; i < (int)(sizeof(ShotDesc) / sizeof(int)); ++i) words[i] = cp[i];
        ShotDesc s = __builtin_bit_cast(ShotDesc, words);
        s.buf[0] = as_global(s.buf[0]);
        s.buf[1] = as_global(s.buf[1]);
        s.c = as_global(s.c);
        s.ev_ptr = as_global(s.ev_ptr);
        s.ev = as_global(s.ev);
        s.src = as_global(s.src);
        s.traces = as_global(s.traces);
        s.damp = as_global(s.damp);
#pragma unroll
        for (int i = 0; i < kInlineSources; ++i) s.isrc[i].wav = as_global(s.isrc[i].wav);
        const T *cur = static_cast<const T *>(step & 1 ? s.buf[1] : s.buf[0]);
        T *out = static_cast<T *>(step & 1 ? s.buf[0] : s.buf[1]);
        const T *prev = out;
        if (FROM == FROM_CONTEXT && a.cur) {
            cur = static_cast<const T *>(as_global(a.cur));
            prev = static_cast<const T *>(as_global(a.prev));
            out = static_cast<T *>(as_global(a.out));
        }
        const int tx = local % s.tiles_x;
        const int t2 = local / s.tiles_x;
        const int ty = t2 % s.tiles_y;
        const int cz = t2 / s.tiles_y;
        if (cz >= s.chunks_z) return;
        fwd_tile<C, DAMP, LD>(s, cur, prev, out, step, a.record != 0, tx, ty, cz, lds);
    }
}

template <class C, int FROM, bool DAMP, int LD>
__global__ __launch_bounds__(C::NT) void fwd_kernel(LaunchArgs a)
{
    fwd_body<C, FROM, DAMP, LD>(a);
}

// the same step built for C::OCC waves per SIMD
template <class C, int FROM, bool DAMP, int LD>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::OCC > 0 ? C::OCC : 1)))
void fwd_kernel_occ(LaunchArgs a)
{
    fwd_body<C, FROM, DAMP, LD>(a);
}

// ------------------------------------------------------------------ adjoint step

// One step of the discrete adjoint in the variable mu = c * lambda, fused with the
// imaging condition:
//     mu^k = 2 mu^{k+1} - mu^{k+2} + c Lh mu^{k+1} + resid_amp c_j resid[k-1][j] e_j
//     t    = mu^k * Lh u^{k-1}
// mu^{k+1} and u^{k-1} march in z together, each with its own threads (adj_half).  The
// imaging term t is summed in the working precision, blocked by
// checkpoint segment so that the rounding error grows with the segment length plus
// the number of segments instead of with the number of steps:
//     gmode 0: gseg += t         (inside a segment)
//     gmode 1: gseg  = t         (first step of a segment)
//     gmode 2: g    += gseg + t  (last step of a segment)
//     gmode 3: g    += t         (unblocked)
enum { GM_ACC = 0, GM_FIRST = 1, GM_FOLD = 2, GM_DIRECT = 3 };

// One half of the workgroup's threads (ROLE 0) advances mu over the tile and chunk, the
// other half (ROLE 1) evaluates Lh u^{k-1} over the same tile and accumulates the image: thread t of
// each half owns the same points.  Each half keeps one register queue and stages one field,
// so a tile holds twice the waves that it would with both queues in every thread, each with
// half the registers, loads and arithmetic of a plane.  ROLE 0 leaves mu^k of plane z in mx
// and ROLE 1 adds plane z's image after the next plane's barrier, the only one of a plane:
// the two buffers of mx alternate, and plane z's is rewritten two barriers later.
//
// What bounds it: HBM for large grids (28 B per point; 256^3 r = 4: 96 -> 87 us per step,
// 5.4 TB/s), and before the split, for r = 8, the registers of two queues (more than 256,
// so one wave per SIMD): 192^3 89 -> 56 us, 93x118x141 36 -> 18 us.
template <class C, int ROLE, int LD>
__device__ __forceinline__ void adj_half(const ShotDesc &s, const typename C::type *__restrict__ field,
                                         typename C::type *mout, const typename C::type *g1,
                                         const typename C::type *g2, typename C::type *gout,
                                         const typename C::type *__restrict__ rrow, typename C::type ramp,
                                         const TileGeom<C> &g, typename C::type *lds, typename C::type *mx)
{
    typedef typename C::type T;
    constexpr int R = C::R, VEC = C::VEC, EY = C::EY, HPT = C::HPT, HY = C::HY;
    constexpr int P = 2 * R + 2;
    constexpr int HOFF = C::HOFF, NB = C::NB;
    constexpr StencilWeights<R> W{};
    const T *__restrict__ cc = static_cast<const T *>(s.c);
    const int64_t pxy = s.pxy;

    EventBounds<C> evb;
    if constexpr (ROLE == 0) evb.load(s, g);

    // the queue and the halo work as in fwd_tile; pv and cv are ROLE 0's, g1 and g2 of a
    // plane are loaded while it is computed and used one plane later
    T q[P][EY][VEC], hv[2][HPT][VEC], hp[HOFF > 0 ? HOFF : 1][HPT][VEC];
    T pv[2][EY][VEC], cv[2][EY][VEC];
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) {
        const auto b = plane_buf(field, pxy, g.z0 + k);
#pragma unroll
        for (int e = 0; e < EY; ++e) bld<0>(q[k][e], b, g.obl[e]);
    }
#pragma unroll
    for (int j = 0; j < HOFF; ++j) {
        const auto b = plane_buf(field, pxy, g.z0 + j + R, g.z0 + j < g.z1);
#pragma unroll
        for (int k = 0; k < HPT; ++k) bld<0>(hp[j][k], b, g.hob[k]);
    }
    if constexpr (ROLE == 0) {
        const auto bp = plane_buf(mout, pxy, g.z0 + R), bc = plane_buf(cc, pxy, g.z0 + R);
#pragma unroll
        for (int e = 0; e < EY; ++e) {
            bld<LD>(pv[0][e], bp, g.obr[e]);
            bld<LD>(cv[0][e], bc, g.obr[e]);
        }
    }
    {
        const auto bh = plane_buf(field, pxy, g.z0 + HOFF + R, g.z0 + HOFF < g.z1);
#pragma unroll
        for (int k = 0; k < HPT; ++k) bld<0>(hv[0][k], bh, g.hob[k]);
    }
    // the next plane with events, and of its columns the residual, where `has` says so, or the
    // bits of the place in the list (with registers for both the kernel holds fewer waves)
    int nev_z = 0x7fffffff, has = 0;
    bool look = false;
    T next[EY][VEC];
    if constexpr (ROLE == 0) {
        EventNext<C> nev;
        nev.first(s, g, evb);
        nev_z = nev.z;
        look = nev.look;
#pragma unroll
        for (int e = 0; e < EY; ++e)
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const int code = nev.code[e][v];
                next[e][v] = look ? bits_of<T>(code) : T(0);
                if (evb.any && !look && code >= 0) {
                    next[e][v] = rrow[code];
                    has |= 1 << (e * VEC + v);
                }
            }
    }
    int bz = g.z0 % NB, bh = (g.z0 + HOFF) % NB;
#pragma unroll
    for (int j = 0; j < HOFF; ++j) {
        T *L = lds + ((g.z0 + j) % NB) * C::LDS;
#pragma unroll
        for (int k = 0; k < HPT; ++k)
            if (g.has(k)) vst(L + g.hl[k], hp[j][k]);
    }

    // ROLE 1: Lh u, g1 and g2 of the plane before
    T lap[EY][VEC], gv[2][EY][VEC], gv2[2][EY][VEC];
    auto finish = [&](int z, const T (&a1)[EY][VEC], const T (&a2)[EY][VEC]) __attribute__((always_inline)) {
        const auto bg = plane_buf(gout, pxy, z + R);
        const T *M = mx + (z & 1) * (C::BX * C::BY);
#pragma unroll
        for (int e = 0; e < EY; ++e) {
            T m[VEC], gn[VEC];
            vld(m, M + (g.ly + e) * C::BX + g.lx);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                gn[v] = fma_t(m[v], lap[e][v], a1[e][v]);
                if (g2) gn[v] = gn[v] + a2[e][v];
                if (v > 0 && g.gx + v >= s.nx) gn[v] = T(0);  // padding behind the row stays zero
            }
            bst<kNontemporal>(bg, g.obr[e], gn);
        }
    };

    for (int zb = g.z0; zb < g.z1; zb += 2) {
        static_for<2>([&](auto st_) __attribute__((always_inline)) {
            constexpr int cs = decltype(st_)::value, ns = cs ^ 1;
            const int z = zb + cs;
            if (z >= g.z1) return;
            const bool more = z + 1 < g.z1;
            {
                const auto bt = plane_buf(field, pxy, z + 1 + 2 * R, more);
#pragma unroll
                for (int e = 0; e < EY; ++e) bld<0>(q[2 * R + 1][e], bt, g.obl[e]);
            }
            if constexpr (ROLE == 0) {
                const auto bp = plane_buf(mout, pxy, z + 1 + R, more), bc = plane_buf(cc, pxy, z + 1 + R, more);
#pragma unroll
                for (int e = 0; e < EY; ++e) {
                    bld<LD>(pv[ns][e], bp, g.obr[e]);
                    bld<LD>(cv[ns][e], bc, g.obr[e]);
                }
            } else {
                const auto b1 = plane_buf(g1, pxy, z + R, g1 != nullptr), b2 = plane_buf(g2, pxy, z + R, g2 != nullptr);
#pragma unroll
                for (int e = 0; e < EY; ++e) {
                    bld<LD>(gv[cs][e], b1, g.obr[e]);
                    bld<LD>(gv2[cs][e], b2, g.obr[e]);
                }
            }
            {
                const auto bh2 = plane_buf(field, pxy, z + 1 + HOFF + R, z + 1 + HOFF < g.z1);
#pragma unroll
                for (int k = 0; k < HPT; ++k) bld<0>(hv[ns][k], bh2, g.hob[k]);
            }
            T *L = lds + bz * C::LDS;
#pragma unroll
            for (int e = 0; e < EY; ++e) vst(L + (g.ly + e + HY) * C::LW + C::LPAD + g.lx, q[R][e]);
            {
                T *LH = lds + bh * C::LDS;
#pragma unroll
                for (int k = 0; k < HPT; ++k)
                    if (g.has(k)) vst(LH + g.hl[k], hv[cs][k]);
            }
            __syncthreads();
            if constexpr (ROLE == 1)
                if (z > g.z0) finish(z - 1, gv[ns], gv2[ns]);

            T yr[C::YR][VEC];
#pragma unroll
            for (int j = 0; j < C::YR; ++j) {
                if (j >= HY && j < HY + EY) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) yr[j][v] = q[R][j - HY][v];
                } else {
                    vld(yr[j], L + (g.ly + j) * C::LW + C::LPAD + g.lx);
                }
            }
            T mnew[EY][VEC];
#pragma unroll
            for (int e = 0; e < EY; ++e) {
                T xs[C::NXV * VEC];
#pragma unroll
                for (int j = 0; j < C::NXV; ++j) {
                    T tmp[VEC];
                    if (j * VEC == C::LPAD) {  // this thread's own vector
#pragma unroll
                        for (int v = 0; v < VEC; ++v) tmp[v] = q[R][e][v];
                    } else {
                        vld(tmp, L + (g.ly + e + HY) * C::LW + g.lx + j * VEC);
                    }
#pragma unroll
                    for (int v = 0; v < VEC; ++v) xs[j * VEC + v] = tmp[v];
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const T u0 = q[R][e][v];
                    T acc = T(0);
#pragma unroll
                    for (int l = 1; l <= R; ++l)
                        acc = fma_t(T(W.w[l]), (xs[C::LPAD + v + l] - u0) + (xs[C::LPAD + v - l] - u0), acc);
                    if (C::NDIM == 3) {
#pragma unroll
                        for (int l = 1; l <= R; ++l)
                            acc = fma_t(T(W.w[l]), (yr[HY + e + l][v] - u0) + (yr[HY + e - l][v] - u0), acc);
                    }
#pragma unroll
                    for (int l = 1; l <= R; ++l)
                        acc = fma_t(T(W.w[l]), (q[R + l][e][v] - u0) + (q[R - l][e][v] - u0), acc);
                    if constexpr (ROLE == 0)
                        mnew[e][v] = fma_t(cv[cs][e][v], acc, T(2) * u0 - pv[cs][e][v]);
                    else
                        lap[e][v] = acc;
                }
            }

            if constexpr (ROLE == 0) {
                // adjoint sources: the residual enters at the receivers, scaled by c there
                if (z == nev_z) {
                    if (!look) {
#pragma unroll
                        for (int e = 0; e < EY; ++e)
#pragma unroll
                            for (int v = 0; v < VEC; ++v)
                                if (has >> (e * VEC + v) & 1)
                                    mnew[e][v] = fma_t(ramp * cv[cs][e][v], next[e][v], mnew[e][v]);
                        nev_z = 0x7fffffff;
                    } else {
                        int at[EY][VEC];
#pragma unroll
                        for (int e = 0; e < EY; ++e)
#pragma unroll
                            for (int v = 0; v < VEC; ++v) at[e][v] = bits_to_int(next[e][v]);
                        nev_z = look_events<C>(s, g, at, z, [&](int code, auto e, auto v) __attribute__((always_inline)) {
                            if (code >= 0) mnew[e][v] = fma_t(ramp * cv[cs][e][v], rrow[code], mnew[e][v]);
                        });
#pragma unroll
                        for (int e = 0; e < EY; ++e)
#pragma unroll
                            for (int v = 0; v < VEC; ++v) next[e][v] = bits_of<T>(at[e][v]);
                    }
                }
                const auto bpm = plane_buf(mout, pxy, z + R);
                T *M = mx + (z & 1) * (C::BX * C::BY);
#pragma unroll
                for (int e = 0; e < EY; ++e) {
#pragma unroll
                    for (int v = 1; v < VEC; ++v) mnew[e][v] = g.gx + v < s.nx ? mnew[e][v] : T(0);
                    vst(M + (g.ly + e) * C::BX + g.lx, mnew[e]);
                    bst<kNontemporal>(bpm, g.obr[e], mnew[e]);
                }
            }
#pragma unroll
            for (int j = 0; j < P - 1; ++j)
#pragma unroll
                for (int e = 0; e < EY; ++e)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) q[j][e][v] = q[j + 1][e][v];
            bz = (bz + 1 == NB) ? 0 : bz + 1;
            bh = (bh + 1 == NB) ? 0 : bh + 1;
        });
    }
    __syncthreads();
    if constexpr (ROLE == 1) {
        if ((g.z1 - 1 - g.z0) & 1)
            finish(g.z1 - 1, gv[1], gv2[1]);
        else
            finish(g.z1 - 1, gv[0], gv2[0]);
    }
}

template <class C, int LD>
__global__ __launch_bounds__(2 * C::NT) void adj_kernel(AdjArgs a)
{
    typedef typename C::type T;
    __shared__ __attribute__((aligned(16))) T lds[2 * C::NB * C::LDS + 2 * C::BX * C::BY];
    int wg = blockIdx.x;
    if (a.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    const int tx = wg % a.tiles_x;
    const int t2 = wg / a.tiles_x;
    const int ty = t2 % a.tiles_y;
    const int cz = t2 / a.tiles_y;
    if (cz >= a.chunks_z) return;
    const bool image = __builtin_amdgcn_readfirstlane((int)threadIdx.x) >= C::NT;  // uniform over a wave

    const ShotDesc &s = a.one;
    TileGeom<C> g;
    g.init(s, tx, ty, cz, a.zch, (int)threadIdx.x - (image ? C::NT : 0));
    if (g.z0 >= g.z1) return;

    // imaging accumulator: g1 (added through the FMA), g2 (added after it), gout (stored)
    T *const grad = static_cast<T *>(a.grad), *const gseg = static_cast<T *>(a.gseg);
    const T *g1 = a.gmode == GM_FIRST ? nullptr : a.gmode == GM_DIRECT ? grad : gseg;
    const T *g2 = a.gmode == GM_FOLD ? grad : nullptr;
    T *gout = (a.gmode == GM_ACC || a.gmode == GM_FIRST) ? gseg : grad;
    T *const mx = lds + 2 * C::NB * C::LDS;
    const int64_t nrec = a.live ? *as_global(static_cast<const int64_t *>(s.traces)) : s.nrec;
    if (image)
        adj_half<C, 1, LD>(s, static_cast<const T *>(a.u_km1), nullptr, g1, g2, gout, nullptr, T(0), g,
                       lds + C::NB * C::LDS, mx);
    else
        adj_half<C, 0, LD>(s, static_cast<const T *>(a.mu_cur), static_cast<T *>(a.mu_out), nullptr, nullptr, nullptr,
                       static_cast<const T *>(a.resid) + (a.k - 1) * nrec, T(a.resid_amp), g, lds, mx);
}

// ------------------------------------------------------------------ registry

// Roles of a forward tile entry: reached with fd_set_tuning alone, or one the library
// chooses from by itself, FINE ones only where z chunks are short (they have no early halo
// and a small tile's larger share of it), or the build for 4 waves per SIMD that stands in
// for the chosen tile of the same shape on mid-size grids.
enum { FWD_OPTION = 0, FWD_AUTO = 1, FWD_FINE = 2, FWD_TWIN = 3 };

struct FwdEntry {
    const char *name;
    int bx, by, nt;
    void (*launch)(const LaunchArgs &, int nwg, hipStream_t);
    const void *kernel;  // the __global__ function (for occupancy queries)
    int role;
    float cost;          // relative time per point of the tile, where it streams well
    float cached_cost;   // FINE tiles on grids that stay in the last-level cache: the same there
    int cached_zch;      // and the planes per chunk to use (0: as elsewhere)
};

// Roles of an adjoint tile entry: reached with fd_set_adj_tuning alone, one the library
// chooses from by itself, or the one it takes where a chunk is a single plane.
enum { ADJ_OPTION = 0, ADJ_AUTO = 1, ADJ_ONE_PLANE = 2 };

struct AdjEntry {
    const char *name;
    int bx, by, nt;
    void (*launch)(const AdjArgs &, int nwg, hipStream_t);
    const void *kernel;
    int role;
    float cost;  // as in FwdEntry
};

template <class C, int FROM, bool DAMP, int LD>
constexpr auto fwd_kernel_of()
{
    if constexpr (C::OCC > 0)
        return &fwd_kernel_occ<C, FROM, DAMP, LD>;
    else
        return &fwd_kernel<C, FROM, DAMP, LD>;
}

// OPTION tiles have no build for fields that stay in the cache, and one for batches; captured
// launches have one.  Such a single build is the damped, nontemporal one, which is right for
// every shot.  TWIN tiles have neither: the tile they stand in for takes the same launch.
template <class C, int ROLE, bool DAMP>
void launch_fwd_as(const LaunchArgs &a, int nwg, hipStream_t st)
{
    const dim3 grid(nwg), block(C::NT);
    constexpr int KEEP = kPointLoads<ROLE != FWD_OPTION>, ONCE = kPointLoads<false>;
    if (!a.shots) {
        if (a.cached)
            hipLaunchKernelGGL((fwd_kernel_of<C, FROM_ARGS, DAMP, KEEP>()), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((fwd_kernel_of<C, FROM_ARGS, DAMP, ONCE>()), grid, block, 0, st, a);
        return;
    }
    if (a.step >= 0) {
        if constexpr (DAMP && ROLE != FWD_TWIN)
            hipLaunchKernelGGL((fwd_kernel_of<C, FROM_CONTEXT, DAMP, ONCE>()), grid, block, 0, st, a);
        return;
    }
    if constexpr (ROLE == FWD_AUTO || ROLE == FWD_FINE) {
        if (a.cached)
            hipLaunchKernelGGL((fwd_kernel_of<C, FROM_TABLE, DAMP, KEEP>()), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((fwd_kernel_of<C, FROM_TABLE, DAMP, ONCE>()), grid, block, 0, st, a);
    } else if constexpr (DAMP && ROLE == FWD_OPTION) {
        hipLaunchKernelGGL((fwd_kernel_of<C, FROM_TABLE, DAMP, ONCE>()), grid, block, 0, st, a);
    }
}

template <class C, int ROLE>
void launch_fwd(const LaunchArgs &a, int nwg, hipStream_t st)
{
    if (a.damped || (ROLE == FWD_OPTION && a.shots))
        launch_fwd_as<C, ROLE, true>(a, nwg, st);
    else
        launch_fwd_as<C, ROLE, false>(a, nwg, st);
}

template <class C, int ROLE>
void launch_adj(const AdjArgs &a, int nwg, hipStream_t st)
{
    constexpr int KEEP = kPointLoads<ROLE != ADJ_OPTION>, ONCE = kPointLoads<false>;
    if (a.cached)
        hipLaunchKernelGGL((adj_kernel<C, KEEP>), dim3(nwg), dim3(2 * C::NT), 0, st, a);
    else
        hipLaunchKernelGGL((adj_kernel<C, ONCE>), dim3(nwg), dim3(2 * C::NT), 0, st, a);
}

template <class C, int ROLE>
FwdEntry fwd_entry(const char *name, float cost, float cached_cost = 0, int cached_zch = 0)
{
    return FwdEntry{name, C::BX, C::BY, C::NT, &launch_fwd<C, ROLE>,
                    reinterpret_cast<const void *>(fwd_kernel_of<C, FROM_ARGS, false, kNontemporal>()), ROLE, cost, cached_cost,
                    cached_zch};
}

template <class C, int ROLE>
AdjEntry adj_entry(const char *name, float cost)
{
    return AdjEntry{name, C::BX, C::BY, 2 * C::NT, &launch_adj<C, ROLE>,
                    reinterpret_cast<const void *>(&adj_kernel<C, kNontemporal>), ROLE, cost};
}

// Implemented in the per-dtype translation units.
const FwdEntry *fwd_configs_f32(int r, int ndim, int *count);
const FwdEntry *fwd_configs_f64(int r, int ndim, int *count);
const AdjEntry *adj_configs_f32(int r, int ndim, int *count);
const AdjEntry *adj_configs_f64(int r, int ndim, int *count);

}  // namespace fdw
