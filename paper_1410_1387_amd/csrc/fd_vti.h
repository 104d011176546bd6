// fd_vti.h -- gfx950 kernel for the two-field VTI propagator.
//
// One launch performs one step of the centred time scheme of Sec. 1 of Medina,
// St-Cyr and Warburton applied to the pseudo-acoustic VTI equations (p) and (q):
//     p^{n+1} = 2 p^n - p^{n-1} + ax * Sxy + az * Sz + sources
//     q^{n+1} = 2 q^n - q^{n-1} + an * Sxy + az * Sz + sources
// with ax, an, az = dt^2 (nu_x^2, nu_n^2, nu_z^2) / h^2 and
//     Sxy = 2 w_0 p + sum_{l=1..RXY} w_l (p_{x+l} + p_{x-l} + p_{y+l} + p_{y-l})
//           (the symmetric xy stencil of Sec. 1, acting on p only),
//     Sz  = sum_{l=-RZ..RZ} Wz[z][l] q_{z+l}
//           (the per-plane z stencil of Sec. 1 with 2 RZ + 1 weights per plane,
//            variable spacing absorbed in the weights, acting on q only).
// Both sums are evaluated in the centre-weight form of the paper (two operations
// per neighbour pair): with RXY = 12 the difference form would double the vector
// work of the xy part, and this kernel is meant to stay memory-bound.
//
// Design (no MFMA: a star stencil is not a dense contraction):
//  - A workgroup owns a BX x BY tile of the xy plane and marches a chunk of z
//    planes.  Each thread owns one 16-byte vector of x points in one row.
//  - p is needed with its xy neighbours only, q with its z neighbours only.  So the
//    plane z of p^n, with its RXY-wide x/y halo, is staged in LDS (two buffers, one
//    barrier per plane), and q^n of the thread's column is kept for planes
//    z-RZ .. z+RZ in a register queue that shifts by one plane per step.
//  - Global traffic is x-contiguous 16-byte vectors: p^n and q^n once per point
//    (plus the p halo and the q chunk prologue), p^{n-1}, q^{n-1} and the three
//    coefficient fields with nontemporal loads (see kPointLoads), p^{n+1} and q^{n+1}
//    written with nontemporal stores over p^{n-1} and q^{n-1}.  Every load of the
//    next plane is issued one plane ahead of its use.
//  - The z weights of plane z are uniform across the workgroup (scalar loads).
//  - Loads without branches, sources and receivers as in the acoustic kernel.
//
// What bounds it: HBM for large grids (36 B per point in FP32: 512^3 R_xy = 12, R_z = 8
// 862 -> 831 us per step, 5.81 TB/s, when the loads lost their branches and the tile
// became 128x16), the latency of a plane for small ones (93x118x141 22.6 -> 15.1 us, of which
// 3 since the point-wise loads keep their lines where the fields fit the last-level cache).
#pragma once

#include "fd_stencil.h"

namespace fdw {

template <typename T, int RXY_, int RZ_, int TXN_, int TYN_>
struct VtiCfg {
    typedef T type;
    static constexpr int RXY = RXY_;
    static constexpr int RZ = RZ_;
    static constexpr int R = RXY, HY = RXY, GZ = RZ, EY = 1;  // as TileGeom names them
    static constexpr int TXN = TXN_;                          // threads along x
    static constexpr int TYN = TYN_;                          // threads (= rows) along y
    static constexpr int VEC = V16<T>::N;
    static constexpr int NT = TXN * TYN;
    static constexpr int BX = TXN * VEC;
    static constexpr int BY = TYN;
    static constexpr int LPAD = (RXY + VEC - 1) / VEC * VEC;  // x halo rounded to vectors
    static constexpr int LW = BX + 2 * LPAD;
    static constexpr int LH = BY + 2 * RXY;
    static constexpr int LDS = LW * LH;                       // elements per LDS plane
    // Waves per SIMD that the kernel may hold (0: what its registers allow): one more shortens
    // the chunks or has the compute unit stream more rows at once (320^3 R_xy = 8, R_z = 4
    // 238 us against 217, 128^3 4, 2 15.0 against 14.4, FP64 45x61x222 4, 4 10.6 against 10.0).
    static constexpr int max_waves()
    {
        if (sizeof(T) == 8 && RXY == 2 && RZ == 1) return 0;
        const bool deep = sizeof(T) == 4 ? RXY * RZ >= 32 || (RXY == 12 && NT == 64)
                                         : RXY * RZ >= 16 && !(RXY == 4 && TYN == 16);
        return deep || NT == 512 ? 2 : 3;
    }
    static constexpr int LDS_ALL = lds_limited<T>(2 * LDS, max_waves(), NT);
    static constexpr int NXV = 2 * LPAD / VEC + 1;            // vectors per row for x neighbours
    static constexpr int NHY = 2 * RXY * TXN;                 // y-halo vectors per plane
    static constexpr int NHS = LPAD / VEC;                    // x-halo vectors per side per row
    static constexpr int NHX = 2 * BY * NHS;
    static constexpr int NH = NHY + NHX;
    static constexpr int HPT = (NH + NT - 1) / NT;            // halo vectors per thread
    static constexpr int NWZ = 2 * RZ + 1;
    static_assert(256 % BX == 0 && 64 % BY == 0, "tile must divide the layout alignment");
};

// cb: which of the two buffers of each field holds level n
template <class C, int LD>
__device__ __forceinline__ void vti_tile(const VtiDesc &s, int64_t step, int cb, int tx, int ty, int cz,
                                         typename C::type *lds)
{
    typedef typename C::type T;
    constexpr int RXY = C::RXY, RZ = C::RZ, VEC = C::VEC, HPT = C::HPT, NWZ = C::NWZ;
    constexpr int P = 2 * RZ + 2;  // q planes z-RZ .. z+RZ and the slot receiving z+RZ+1
    constexpr StencilWeights<RXY> W{};
    const int nb = cb ^ 1;
    const T *__restrict__ pcur = static_cast<const T *>(s.pbuf[cb]);
    const T *__restrict__ qcur = static_cast<const T *>(s.qbuf[cb]);
    const T *pprev = static_cast<const T *>(s.pbuf[nb]);  // read point-wise, then overwritten
    const T *qprev = static_cast<const T *>(s.qbuf[nb]);
    T *pout = static_cast<T *>(s.pbuf[nb]);
    T *qout = static_cast<T *>(s.qbuf[nb]);
    const T *__restrict__ fax = static_cast<const T *>(s.ax);
    const T *__restrict__ fan = static_cast<const T *>(s.an);
    const T *__restrict__ faz = static_cast<const T *>(s.az);
    const T *__restrict__ wz = static_cast<const T *>(s.wz);
    const int64_t pxy = s.pxy;

    TileGeom<C> g;
    g.init(s, tx, ty, cz, s.zch, threadIdx.x);
    if (g.z0 >= g.z1) return;  // uniform over the workgroup
    const uint32_t ob = g.obr[0];

    EventBounds<C> evb;
    evb.load(s, g);

    // the samples of a source inside this tile and chunk (see fwd_tile)
    int srcz[kInlineSources];
    T srcp[kInlineSources], srcq[kInlineSources];
#pragma unroll
    for (int i = 0; i < kInlineSources; ++i) {
        const VtiInlineSource &is = s.isrc[i];
        srcz[i] = -1;
        srcp[i] = srcq[i] = T(0);
        if (i < s.nisrc && is.z >= g.z0 && is.z < g.z1 && is.x >= g.x0 && is.x < g.x0 + C::BX && is.y >= g.y0 &&
            is.y < g.y0 + C::BY && step < is.src.nsamp) {
            const T sv = static_cast<const T *>(is.src.wav)[step];
            srcz[i] = is.z;
            srcp[i] = T(is.src.scale_p) * sv;
            srcq[i] = T(is.src.scale_q) * sv;
        }
    }

    T q[P][VEC];
    T pc[2][VEC], pm[2][VEC], qm[2][VEC], a1[2][VEC], a2[2][VEC], a3[2][VEC];
    T hv[2][HPT][VEC];

    // prologue: q planes z0-RZ .. z0+RZ into slots 0 .. 2RZ; everything of plane z0 into set 0
#pragma unroll
    for (int k = 0; k <= 2 * RZ; ++k) bld<0>(q[k], plane_buf(qcur, pxy, g.z0 + k), ob);
    auto load_plane = [&](auto set, int z, bool on) __attribute__((always_inline)) {
        constexpr int i = decltype(set)::value;
        const auto bp = plane_buf(pcur, pxy, z + RZ, on);
        bld<0>(pc[i], bp, ob);
        bld<LD>(pm[i], plane_buf(pprev, pxy, z + RZ, on), ob);
        bld<LD>(qm[i], plane_buf(qprev, pxy, z + RZ, on), ob);
        bld<LD>(a1[i], plane_buf(fax, pxy, z + RZ, on), ob);
        bld<LD>(a2[i], plane_buf(fan, pxy, z + RZ, on), ob);
        bld<LD>(a3[i], plane_buf(faz, pxy, z + RZ, on), ob);
#pragma unroll
        for (int k = 0; k < HPT; ++k) bld<0>(hv[i][k], bp, g.hob[k]);
    };
    load_plane(std::integral_constant<int, 0>{}, g.z0, true);

    EventNext<C> nev;
    nev.first(s, g, evb);
    const int64_t row = step - s.rec_base;
    const bool rec = row >= 0 && row < s.rec_cap;
    T *const trp = rec && s.traces_p ? static_cast<T *>(s.traces_p) + row * s.nrec : nullptr;
    T *const trq = rec && s.traces_q ? static_cast<T *>(s.traces_q) + row * s.nrec : nullptr;

    for (int zb = g.z0; zb < g.z1; zb += 2) {
        static_for<2>([&](auto st_) __attribute__((always_inline)) {
            constexpr int cs = decltype(st_)::value, ns = cs ^ 1;
            constexpr int tail = 2 * RZ + 1;
            const int z = zb + cs;
            if (z >= g.z1) return;
            const bool more = z + 1 < g.z1;
            bld<0>(q[tail], plane_buf(qcur, pxy, z + 1 + 2 * RZ, more), ob);
            load_plane(std::integral_constant<int, ns>{}, z + 1, more);

            // this plane's z weights (uniform: scalar loads)
            const T *__restrict__ wrow = wz + (int64_t)z * NWZ;
            T wk[NWZ];
#pragma unroll
            for (int j = 0; j < NWZ; ++j) wk[j] = wrow[j];

            // stage plane z of p^n (interior from registers, halo) in LDS buffer cs;
            // buffer cs was last read two planes ago, before the previous barrier
            T *L = lds + cs * C::LDS;
            vst(L + (g.ly + RXY) * C::LW + C::LPAD + g.lx, pc[cs]);
#pragma unroll
            for (int k = 0; k < HPT; ++k)
                if (g.has(k)) vst(L + g.hl[k], hv[cs][k]);
            __syncthreads();

            // Sxy from LDS
            T sxy[VEC];
            {
                T xs[C::NXV * VEC];
#pragma unroll
                for (int j = 0; j < C::NXV; ++j) {
                    T tmp[VEC];
                    if (j * VEC == C::LPAD) {  // this thread's own vector
#pragma unroll
                        for (int v = 0; v < VEC; ++v) tmp[v] = pc[cs][v];
                    } else {
                        vld(tmp, L + (g.ly + RXY) * C::LW + g.lx + j * VEC);
                    }
#pragma unroll
                    for (int v = 0; v < VEC; ++v) xs[j * VEC + v] = tmp[v];
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    T acc = T(2.0 * W.w[0]) * pc[cs][v];
#pragma unroll
                    for (int l = 1; l <= RXY; ++l)
                        acc = fma_t(T(W.w[l]), xs[C::LPAD + v + l] + xs[C::LPAD + v - l], acc);
                    sxy[v] = acc;
                }
#pragma unroll
                for (int l = 1; l <= RXY; ++l) {
                    T up[VEC], dn[VEC];
                    vld(up, L + (g.ly + RXY - l) * C::LW + C::LPAD + g.lx);
                    vld(dn, L + (g.ly + RXY + l) * C::LW + C::LPAD + g.lx);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) sxy[v] = fma_t(T(W.w[l]), up[v] + dn[v], sxy[v]);
                }
            }

            // Sz from the queue
            T sz[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                T acc = wk[0] * q[0][v];
#pragma unroll
                for (int j = 1; j < NWZ; ++j) acc = fma_t(wk[j], q[j][v], acc);
                sz[v] = acc;
            }

            T pn[VEC], qn[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const T p0 = pc[cs][v], q0 = q[RZ][v];
                const T zt = a3[cs][v] * sz[v];
                pn[v] = fma_t(a1[cs][v], sxy[v], (T(2) * p0 - pm[cs][v]) + zt);
                qn[v] = fma_t(a2[cs][v], sxy[v], (T(2) * q0 - qm[cs][v]) + zt);
            }

            // fused sources (before the store) and receivers (after them)
#pragma unroll
            for (int i = kInlineSources - 1; i >= 0; --i)
                if (z == srcz[i]) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        if (g.gx + v == s.isrc[i].x && g.gy == s.isrc[i].y) {
                            pn[v] += srcp[i];
                            qn[v] += srcq[i];
                        }
                }
            if (z == nev.z) {
                auto event = [&](int code, T &p, T &qv) __attribute__((always_inline)) {
                    if (code >= 0) {
                        if (trp) trp[code] = p;
                        if (trq) trq[code] = qv;
                    } else if (code != kNoEvent) {
                        const VtiSource si = s.src[~code];
                        if (step < si.nsamp) {
                            const T sv = as_global(static_cast<const T *>(si.wav))[step];
                            p += T(si.scale_p) * sv;
                            qv += T(si.scale_q) * sv;
                        }
                    }
                };
                if (!nev.look) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) event(nev.code[0][v], pn[v], qn[v]);
                    nev.z = 0x7fffffff;
                } else {
                    nev.z = look_events<C>(s, g, nev.code, z, [&](int code, auto, auto v) __attribute__((always_inline)) {
                        event(code, pn[v], qn[v]);
                    });
                }
            }

            // a vector that straddles the end of its row keeps the padding behind it zero
#pragma unroll
            for (int v = 1; v < VEC; ++v)
                if (g.gx + v >= s.nx) pn[v] = qn[v] = T(0);
            bst<kNontemporal>(plane_buf(pout, pxy, z + RZ), ob, pn);
            bst<kNontemporal>(plane_buf(qout, pxy, z + RZ), ob, qn);
#pragma unroll
            for (int k = 0; k < P - 1; ++k)
#pragma unroll
                for (int v = 0; v < VEC; ++v) q[k][v] = q[k + 1][v];
        });
    }
}

template <class C, int LD>
__global__ __launch_bounds__(C::NT) void vti_kernel(VtiDesc s, int64_t step)
{
    typedef typename C::type T;
    __shared__ __attribute__((aligned(16))) T lds[C::LDS_ALL];
    int wg = blockIdx.x;
    if (s.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    const int tx = wg % s.tiles_x;
    const int t2 = wg / s.tiles_x;
    const int ty = t2 % s.tiles_y;
    const int cz = t2 / s.tiles_y;
    if (cz >= s.chunks_z) return;
    vti_tile<C, LD>(s, step, (int)(step & 1), tx, ty, cz, lds);
}

// The same for captured launches: the descriptor is read from the context's workspace, so that
// a replay finds the sources and receivers of its own time (a build of its own, because
// choosing in the launch, or a longer argument, costs small grids 2-9 %).
template <class C>
__global__ __launch_bounds__(C::NT) void vti_kernel_live(const VtiDesc *live, int64_t step)
{
    typedef typename C::type T;
    __shared__ __attribute__((aligned(16))) T lds[C::LDS_ALL];
    const auto *words = (const __attribute__((address_space(4))) int *)(uintptr_t)live;
    int copy[sizeof(VtiDesc) / sizeof(int)];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(VtiDesc) / sizeof(int)); ++i) copy[i] = words[i];
    VtiDesc s = __builtin_bit_cast(VtiDesc, copy);
    s.wz = as_global(s.wz);
    s.ev_ptr = as_global(s.ev_ptr);
    s.ev = as_global(s.ev);
    s.src = as_global(s.src);
    s.traces_p = as_global(s.traces_p);
    s.traces_q = as_global(s.traces_q);
#pragma unroll
    for (int i = 0; i < kInlineSources; ++i) s.isrc[i].src.wav = as_global(s.isrc[i].src.wav);
    // level n first: an index by parity would keep the copy in scratch memory
    void *const p0 = s.pbuf[0], *const q0 = s.qbuf[0];
    const bool odd = step & 1;
    s.pbuf[0] = odd ? s.pbuf[1] : p0;
    s.pbuf[1] = odd ? p0 : s.pbuf[1];
    s.qbuf[0] = odd ? s.qbuf[1] : q0;
    s.qbuf[1] = odd ? q0 : s.qbuf[1];
    int wg = blockIdx.x;
    if (s.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    const int tx = wg % s.tiles_x;
    const int t2 = wg / s.tiles_x;
    const int ty = t2 % s.tiles_y;
    const int cz = t2 / s.tiles_y;
    if (cz >= s.chunks_z) return;
    vti_tile<C, kNontemporal>(s, step, 0, tx, ty, cz, lds);
}

// Roles: reached with fd_vti_set_tuning alone, or one the library chooses from by itself.
enum { VTI_OPTION = 0, VTI_AUTO = 1 };

struct VtiEntry {
    const char *name;
    int rxy, rz, bx, by, nt;
    // live: null, or the descriptor in device memory (captured launches)
    void (*launch)(const VtiDesc &, const VtiDesc *live, int64_t step, int nwg, hipStream_t);
    const void *kernel;
    int role;
    float cost;  // as in FwdEntry
};

template <class C, int ROLE>
void launch_vti(const VtiDesc &d, const VtiDesc *live, int64_t step, int nwg, hipStream_t st)
{
    constexpr int KEEP = kPointLoads<ROLE != VTI_OPTION>, ONCE = kPointLoads<false>;
    if (live)
        hipLaunchKernelGGL((vti_kernel_live<C>), dim3(nwg), dim3(C::NT), 0, st, live, step);
    else if (d.cached)
        hipLaunchKernelGGL((vti_kernel<C, KEEP>), dim3(nwg), dim3(C::NT), 0, st, d, step);
    else
        hipLaunchKernelGGL((vti_kernel<C, ONCE>), dim3(nwg), dim3(C::NT), 0, st, d, step);
}

template <class C, int ROLE>
VtiEntry vti_entry(const char *name, float cost)
{
    return VtiEntry{name, C::RXY, C::RZ, C::BX, C::BY, C::NT, &launch_vti<C, ROLE>,
                    reinterpret_cast<const void *>(&vti_kernel<C, kNontemporal>), ROLE, cost};
}

// Implemented in the per-dtype translation units.
const VtiEntry *vti_configs_f32(int rxy, int rz, int *count);
const VtiEntry *vti_configs_f64(int rxy, int rz, int *count);

}  // namespace fdw
