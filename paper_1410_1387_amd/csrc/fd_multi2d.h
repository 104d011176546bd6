// fd_multi2d.h -- several leapfrog steps of a 2-D grid in one launch.
//
// A 2-D grid is small: one step of 256 x 256 FP64 points moves 2 MB, a third of a
// microsecond at HBM rate, while a launch that returns at once takes 2.3 us and one that
// loads and stores 4 us.  So a workgroup loads its tile widened by k radii, advances it k
// steps in LDS and registers, each step over a region narrower by one radius (the points
// outside it that the tile would need are recomputed by several workgroups), and stores the
// tile.  No workgroup waits for another.
//
// The widened tile is cut into strips of M rows and one x vector, one per thread.  A thread
// keeps u^n, u^{n-1} and c of its strip in registers; u^n of the whole region is in LDS, in
// two buffers that alternate, so that a step takes one barrier.  A strip reads M + 2R
// vectors along z and 2 LPAD / VEC per row along x for M rows.  The arithmetic of a point is
// the single-step kernel's, so the results are bitwise its results.
//
// What costs: the vector work of the widened region (r = 4, k = 8, 32 x 32 points: 3.8 times
// the tile's on average over the steps; at 420 x 300 about 0.9 of the 2.8 us of a step) and
// what it does not hide, the latencies of LDS, barriers, load and store.  Figures per grid, single step against these, stand at the tables.
#pragma once

#include "fd_stencil.h"

namespace fdw {

template <typename T, int R_, int K_, int TX_, int TZ_, int M_ = 4>
struct Multi2dCfg {
    typedef T type;
    static constexpr int R = R_, K = K_, TX = TX_, TZ = TZ_, M = M_;
    static constexpr int VEC = V16<T>::N;
    static constexpr int LPAD = (R + VEC - 1) / VEC * VEC;
    static constexpr int HX = (K * R + VEC - 1) / VEC * VEC;  // x halo of the region
    static constexpr int HZ = (K * R + M - 1) / M * M;        // z halo
    static constexpr int W = TX + 2 * HX, H = TZ + 2 * HZ;
    static constexpr int NSX = W / VEC, NSZ = H / M;
    static constexpr int NT = (NSX * NSZ + 63) / 64 * 64;     // one strip per thread
    static constexpr int LDS = W * (H + 2 * M);               // one buffer: M guard rows on either side
    static_assert(TX % VEC == 0 && TZ % M == 0 && NT <= 1024, "strips cover the tile");
};

struct Multi2dArgs {
    ShotDesc one;
    const void *cur;    // u^n
    const void *prev;   // u^{n-1}
    void *out;          // u^{n+k}: not cur or prev
    void *out_prev;     // u^{n+k-1}
    void *all;          // if set, u^{n+1} .. u^{n+k} go to consecutive fields from here instead
    int64_t field;      // bytes from one field to the next
    int64_t step;       // n
    int32_t k;          // steps of this launch, 1 .. K
    int32_t record, tiles_x, tiles_z, xcd_remap, pad0;
};

// Event codes of a strip's points (kNoEvent: none); `look` if a point has several, which
// are then looked up.
template <class C>
__device__ __forceinline__ void strip_events(const ShotDesc &s, int gx, int gz, int (&code)[C::M][C::VEC], bool &any,
                                             bool &look)
{
    constexpr int M = C::M, VEC = C::VEC;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int v = 0; v < VEC; ++v) code[m][v] = kNoEvent;
    if (!s.ev_ptr) return;
    int p[VEC + 1];
#pragma unroll
    for (int v = 0; v <= VEC; ++v) p[v] = s.ev_ptr[min(gx + v, s.nx)];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        int e = p[v];
        const int hi = p[v + 1];
        if (hi - e > 1) e = lower_bound_z(s.ev, e, hi, gz);
        for (; e < hi; ++e) {
            const Event ev = s.ev[e];
            if (ev.z >= gz + M) break;
            if (ev.z < gz) continue;
            any = true;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                look = look || (ev.z == gz + m && code[m][v] != kNoEvent);
                code[m][v] = ev.z == gz + m ? ev.code : code[m][v];
            }
        }
    }
}

// Row m of a strip from its x neighbours xs and its column neighbours zw.
template <class C, bool DIFF, int NX, int NZ>
__device__ __forceinline__ void row_stencil(typename C::type (&acc)[C::VEC], const typename C::type (&xs)[NX],
                                            const typename C::type (&zw)[NZ][C::VEC], int m)
{
    typedef typename C::type T;
    constexpr int R = C::R, LPAD = C::LPAD;
    constexpr StencilWeights<R> Wt{};
#pragma unroll
    for (int v = 0; v < C::VEC; ++v) {
        const T u0 = xs[LPAD + v];
        if constexpr (DIFF) {
            acc[v] = T(0);
#pragma unroll
            for (int l = 1; l <= R; ++l)
                acc[v] = fma_t(T(Wt.w[l]), (xs[LPAD + v + l] - u0) + (xs[LPAD + v - l] - u0), acc[v]);
#pragma unroll
            for (int l = 1; l <= R; ++l)
                acc[v] = fma_t(T(Wt.w[l]), (zw[R + m + l][v] - u0) + (zw[R + m - l][v] - u0), acc[v]);
        } else {
            acc[v] = T(2 * Wt.w[0]) * u0;
#pragma unroll
            for (int l = 1; l <= R; ++l) acc[v] = fma_t(T(Wt.w[l]), xs[LPAD + v + l] + xs[LPAD + v - l], acc[v]);
#pragma unroll
            for (int l = 1; l <= R; ++l) acc[v] = fma_t(T(Wt.w[l]), zw[R + m + l][v] + zw[R + m - l][v], acc[v]);
        }
    }
}

// The unscaled stencil of a strip, its values in u and its neighbours in LDS (L: the strip's
// first row).  DIFF: summed as differences to the centre, the form of the single-step kernel
// for radii <= 4 and of the adjoint.
template <class C, bool DIFF>
__device__ __forceinline__ void strip_stencil(typename C::type (&acc)[C::M][C::VEC],
                                              const typename C::type (&u)[C::M][C::VEC], const typename C::type *L)
{
    typedef typename C::type T;
    constexpr int R = C::R, M = C::M, VEC = C::VEC, LPAD = C::LPAD, W = C::W;
    constexpr StencilWeights<R> Wt{};
    T zw[M + 2 * R][VEC];
#pragma unroll
    for (int i = 0; i < M + 2 * R; ++i) {
        if (i >= R && i < R + M) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) zw[i][v] = u[i - R][v];
        } else {
            vld(zw[i], L + (i - R) * W);
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        constexpr int NXV = 2 * LPAD / VEC + 1;
        T xs[NXV * VEC];
#pragma unroll
        for (int i = 0; i < NXV; ++i) {
            T tmp[VEC];
            if (i * VEC == LPAD) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) tmp[v] = u[m][v];
            } else {
                vld(tmp, L + m * W - LPAD + i * VEC);
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) xs[i * VEC + v] = tmp[v];
        }
        row_stencil<C, DIFF>(acc[m], xs, zw, m);
    }
}

template <class C, bool DAMP>
__global__ __launch_bounds__(C::NT) void multi2d_kernel(Multi2dArgs a)
{
    typedef typename C::type T;
    constexpr int R = C::R, M = C::M, VEC = C::VEC, W = C::W;
    __shared__ __attribute__((aligned(16))) T lds[2 * C::LDS];
    __shared__ T samples[kInlineSources][C::K];
    int wg = blockIdx.x;
    if (a.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    const ShotDesc &s = a.one;
    const int tx = wg % a.tiles_x, tz = wg / a.tiles_x;
    const int k = a.k;
    const int tid = threadIdx.x;
    const int sx = tid % C::NSX, sz = tid / C::NSX;  // this thread's strip of the region
    const int lx = sx * VEC, lz = sz * M;
    const int gx = tx * C::TX - C::HX + lx, gz = tz * C::TZ - C::HZ + lz;
    const bool strip = sz < C::NSZ;
    const bool xin = gx >= 0 && gx < s.nx;           // a vector never straddles x = 0
    const bool tile = strip && lx >= C::HX && lx < C::HX + C::TX && lz >= C::HZ && lz < C::HZ + C::TZ;

    // byte offsets of the strip's rows within a field (fields are well below 2 GiB here)
    const int bytes = (int)a.field;
    uint32_t ob[M];
    bool zin[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        zin[m] = strip && xin && gz + m >= 0 && gz + m < s.nz;
        ob[m] = zin[m] ? (uint32_t)((int)s.off0 + (gz + m) * (int)s.px + gx) * (uint32_t)sizeof(T) : kOffGrid;
    }
    // rows and vectors of the region that step j (1 .. k) computes: the tile and the
    // (k - j) R points around it that later steps need
    auto active = [&](int j) {
        const int e = (k - j) * R;
        return strip && lz + M > C::HZ - e && lz < C::HZ + C::TZ + e && lx + VEC > C::HX - e && lx < C::HX + C::TX + e;
    };

    auto buf = [&](const void *f) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(f), 0, bytes, 0x00027000);
    };
    T u[M][VEC], pv[M][VEC], cv[M][VEC];
    {
        const auto bu = buf(a.cur), bp = buf(a.prev), bc = buf(s.c);
        const bool first = active(1);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            bld<0>(u[m], bu, ob[m]);
            bld<0>(pv[m], bp, first ? ob[m] : kOffGrid);
            bld<0>(cv[m], bc, first ? ob[m] : kOffGrid);
        }
    }
    T gxv[VEC], gzv[M];
    if constexpr (DAMP) {
        const auto bd = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(s.damp), 0,
                                                          (s.nx + s.ny + s.nz) * (int)sizeof(T), 0x00027000);
        const T one = bld1<T>(bd, (uint32_t)s.nx * (uint32_t)sizeof(T));  // the unit axis
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            gxv[v] = bld1<T>(bd, xin ? (uint32_t)(gx + v) * (uint32_t)sizeof(T) : kOffGrid) * one;
#pragma unroll
        for (int m = 0; m < M; ++m)
            gzv[m] = bld1<T>(bd, zin[m] ? (uint32_t)(s.nx + s.ny + gz + m) * (uint32_t)sizeof(T) : kOffGrid);
    }

    // sources: the samples of the k steps go to LDS, the thread that owns the point adds them
    if (tid < kInlineSources * C::K) {
        const int i = tid / C::K, j = tid % C::K;
        T v = T(0);
        if (i < s.nisrc && a.step + j < s.isrc[i].nsamp)
            v = T(s.isrc[i].scale) * static_cast<const T *>(s.isrc[i].wav)[a.step + j];
        samples[i][j] = v;
    }
    int src[kInlineSources], nsmp[kInlineSources];  // the strip's point (row * VEC + lane) or -1; samples left
#pragma unroll
    for (int i = 0; i < kInlineSources; ++i) {
        const int m = s.isrc[i].z - gz, v = s.isrc[i].x - gx;
        src[i] = i < s.nisrc && strip && m >= 0 && m < M && v >= 0 && v < VEC ? m * VEC + v : -1;
        nsmp[i] = (int)max((int64_t)0, min((int64_t)k, s.isrc[i].nsamp - a.step));
    }

    // receivers of the strip's points inside the tile
    int code[M][VEC];
    bool any = false, look = false;
    if (a.record && s.ev_zlo < (tz + 1) * C::TZ && s.ev_zhi >= tz * C::TZ && tile && xin)
        strip_events<C>(s, gx, gz, code, any, look);

    // points outside the grid occur in regions that cross its edge only
    const bool edge_x = tx * C::TX - C::HX + W > s.nx;
    const bool edge = edge_x || tx * C::TX < C::HX || tz * C::TZ < C::HZ || tz * C::TZ - C::HZ + C::H > s.nz;

    T *const L0 = lds + (M + lz) * W + lx;
    if (strip) {
#pragma unroll
        for (int m = 0; m < M; ++m) vst(L0 + m * W, u[m]);
    }
    __syncthreads();

#pragma unroll 1
    for (int j = 1; j <= k; ++j) {
        const T *L = L0 + ((j - 1) & 1) * C::LDS;
        if (active(j)) {
            T acc[M][VEC], un[M][VEC];
            strip_stencil<C, (R <= 4)>(acc, u, L);
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    if constexpr (DAMP) {
                        const T G = gxv[v] * gzv[m];
                        un[m][v] = G * fma_t(cv[m][v], acc[m][v], T(2) * u[m][v] - G * pv[m][v]);
                    } else {
                        un[m][v] = fma_t(cv[m][v], acc[m][v], T(2) * u[m][v] - pv[m][v]);
                    }
                }
            // The rare cases compare inside their branches: as loop invariants their lane
            // masks would fill the scalar registers and be spilled and read back every step.
#pragma unroll
            for (int i = kInlineSources - 1; i >= 0; --i)
                if (src[i] >= 0 && j <= nsmp[i]) {
                    const T add = samples[i][j - 1];
                    int at = src[i];
                    asm volatile("" : "+v"(at));
#pragma unroll
                    for (int m = 0; m < M; ++m)
#pragma unroll
                        for (int v = 0; v < VEC; ++v)
                            if (at == m * VEC + v) un[m][v] += add;
                }
            // the solution is zero outside the grid
            if (edge_x) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 1; v < VEC; ++v) un[m][v] = gx + v < s.nx ? un[m][v] : T(0);
            }
            if (edge) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) un[m][v] = zin[m] ? un[m][v] : T(0);
            }
            if (any) {
                const int64_t row = a.step + j - 1 - s.rec_base;
                if (row >= 0 && row < s.rec_cap) {
                    T *const tr = static_cast<T *>(s.traces) + row * s.nrec;
#pragma unroll
                    for (int m = 0; m < M; ++m)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            int c = code[m][v];
                            asm volatile("" : "+v"(c));
                            if (c == kNoEvent) continue;
                            if (!look) {
                                tr[c] = un[m][v];
                            } else {
                                const int hi = s.ev_ptr[gx + v + 1];
                                int e = lower_bound_z(s.ev, s.ev_ptr[gx + v], hi, gz + m);
                                for (; e < hi && s.ev[e].z == gz + m; ++e) tr[s.ev[e].code] = un[m][v];
                            }
                        }
                }
            }
            T *Ln = L0 + (j & 1) * C::LDS;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                vst(Ln + m * W, un[m]);
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    pv[m][v] = u[m][v];
                    u[m][v] = un[m][v];
                }
            }
            if (a.all && tile) {
                const auto bo = buf(static_cast<char *>(a.all) + (int64_t)(j - 1) * a.field);
#pragma unroll
                for (int m = 0; m < M; ++m) bst<0>(bo, ob[m], u[m]);
            }
        }
        __syncthreads();
    }
    if (!a.all && tile) {
        const auto bo = buf(a.out), bq = buf(a.out_prev);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            bst<0>(bo, ob[m], u[m]);
            bst<0>(bq, ob[m], pv[m]);
        }
    }
}

// ------------------------------------------------------------------ adjoint

// k adjoint steps in one launch: mu as multi2d_kernel takes u, on the widened tile, and the
// image of every step on the tile, by threads of their own.  These own a strip of the tile
// each, evaluate L u of the step's forward state, which they read with its neighbours from
// memory a step ahead, and after the barrier add its product with mu, read from LDS, to the
// image in registers.  The arithmetic is adj_kernel's, so the results are bitwise its
// results.
struct Adj2dArgs {
    ShotDesc one;
    const void *cur;      // mu^{k0+1}
    const void *prev;     // mu^{k0+2}
    void *out;            // mu^{k0-k+1}: not cur or prev
    void *out_prev;       // mu^{k0-k+2}
    const void *states0;  // forward state of slot 0
    const void *states1;  // of slot 1, consecutive fields from there on
    int64_t slot;         // of u^{k0-1}, the state of the first step
    const void *g_in;     // the image's sum so far, or null for zero
    const void *g_add;    // added to it at the end, or null
    void *g_out;
    const void *resid;    // [T][nrec]
    double resid_amp;
    int64_t field;        // bytes from one field to the next
    int64_t k0;
    int32_t k, tiles_x, tiles_z, xcd_remap;
};

// Rows of an image thread's strip.  The fewer, the more threads share the work and the fewer
// registers a strip with its neighbours takes (two rows: r = 4 FP64 3.1 us per step against
// 7.0 with four rows, which spill); at r = 1 four rows fit a third workgroup on the CU
// (1203 x 801 FP32 2.7 us against 6.3).
template <class C>
constexpr int kImageRows = C::R == 1 ? 4 : 2;

template <class C>
constexpr int adj2d_image_threads = (C::TX / C::VEC * (C::TZ / kImageRows<C>) + 63) / 64 * 64;

template <class C>
__global__ __launch_bounds__(C::NT + adj2d_image_threads<C>) void adj2d_kernel(Adj2dArgs a)
{
    typedef typename C::type T;
    constexpr int R = C::R, M = C::M, VEC = C::VEC, LPAD = C::LPAD, W = C::W;
    __shared__ __attribute__((aligned(16))) T lds[2 * C::LDS];
    int wg = blockIdx.x;
    if (a.xcd_remap) wg = xcd_remap(wg, (int)gridDim.x);
    const ShotDesc &s = a.one;
    const int tx = wg % a.tiles_x, tz = wg / a.tiles_x;
    const int k = a.k;
    const int bytes = (int)a.field;
    auto buf = [&](const void *f) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(f), 0, bytes, 0x00027000);
    };
    auto offset = [&](int x, int z, bool on) {
        return on && x >= 0 && x < s.nx && z >= 0 && z < s.nz
                   ? (uint32_t)((int)s.off0 + z * (int)s.px + x) * (uint32_t)sizeof(T)
                   : kOffGrid;
    };

    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) >= C::NT) {  // the image; uniform over a wave
        constexpr int MI = kImageRows<C>;
        const int t = threadIdx.x - C::NT;
        const bool strip = t < C::TX / VEC * (C::TZ / MI);
        const int lx = t % (C::TX / VEC) * VEC, lz = strip ? t / (C::TX / VEC) * MI : 0;
        const int gx = tx * C::TX + lx, gz = tz * C::TZ + lz;
        constexpr int NS = LPAD / VEC;  // x neighbour vectors on a side
        T zw[MI + 2 * R][VEC], xn[MI][2 * NS][VEC];
        // Neighbours outside the grid are read as they are, zeros of the padding or (below the
        // field) out of the buffer's range.  The offsets are made in every step from one
        // register: as loop invariants they would take as many as the values.
        uint32_t o0 = offset(gx, gz, strip);
        const uint32_t row = (uint32_t)s.px * (uint32_t)sizeof(T);
        auto load = [&](int64_t slot) {
            const auto b = buf(slot ? static_cast<const char *>(a.states1) + (slot - 1) * a.field : a.states0);
            asm volatile("" : "+v"(o0));
#pragma unroll
            for (int i = 0; i < MI + 2 * R; ++i) bld<0>(zw[i], b, o0 + (uint32_t)(i - R) * row);
#pragma unroll
            for (int m = 0; m < MI; ++m)
#pragma unroll
                for (int i = 0; i < 2 * NS; ++i)
                    bld<0>(xn[m][i], b, o0 + (uint32_t)m * row +
                                            (uint32_t)((i < NS ? i - NS : i - NS + 1) * VEC * (int)sizeof(T)));
        };
        load(a.slot);
        T g[MI][VEC], lap[MI][VEC];
        {
            const auto bi = buf(a.g_in);
#pragma unroll
            for (int m = 0; m < MI; ++m) bld<0>(g[m], bi, offset(gx, gz + m, strip && a.g_in));
        }
        const T *const M0 = lds + (M + C::HZ + lz) * W + C::HX + lx;
        auto image = [&](int j) {  // step j's mu is in LDS, its L u in lap
            const T *Lm = M0 + (j & 1) * C::LDS;
#pragma unroll
            for (int m = 0; m < MI; ++m) {
                T mu[VEC];
                vld(mu, Lm + m * W);
#pragma unroll
                for (int v = 0; v < VEC; ++v) g[m][v] = fma_t(mu[v], lap[m][v], g[m][v]);
            }
        };
        __syncthreads();
#pragma unroll 1
        for (int j = 1; j <= k; ++j) {
            if (j > 1) image(j - 1);
#pragma unroll
            for (int m = 0; m < MI; ++m) {
                T xs[(2 * NS + 1) * VEC];
#pragma unroll
                for (int i = 0; i < 2 * NS + 1; ++i)
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        xs[i * VEC + v] = i == NS ? zw[R + m][v] : xn[m][i < NS ? i : i - 1][v];
                row_stencil<C, true>(lap[m], xs, zw, m);
            }
            __builtin_amdgcn_sched_barrier(0);  // into the registers just used
            if (j < k) load(a.slot - j);
            __syncthreads();
        }
        image(k);
        const auto bo = buf(a.g_out), ba = buf(a.g_add);
#pragma unroll
        for (int m = 0; m < MI; ++m) {
            T add[VEC];
            bld<0>(add, ba, offset(gx, gz + m, strip && a.g_add));
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                if (a.g_add) g[m][v] = g[m][v] + add[v];
                if (v > 0 && gx + v >= s.nx) g[m][v] = T(0);  // padding behind the row stays zero
            }
            bst<0>(bo, offset(gx, gz + m, strip), g[m]);
        }
        return;
    }

    const int tid = threadIdx.x;
    const int sx = tid % C::NSX, sz = tid / C::NSX;
    const int lx = sx * VEC, lz = sz * M;
    const int gx = tx * C::TX - C::HX + lx, gz = tz * C::TZ - C::HZ + lz;
    const bool strip = sz < C::NSZ;
    const bool xin = gx >= 0 && gx < s.nx;
    const bool tile = strip && lx >= C::HX && lx < C::HX + C::TX && lz >= C::HZ && lz < C::HZ + C::TZ;
    uint32_t ob[M];
    bool zin[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        ob[m] = offset(gx, gz + m, strip);
        zin[m] = ob[m] != kOffGrid;
    }
    auto active = [&](int j) {  // as in multi2d_kernel
        const int e = (k - j) * R;
        return strip && lz + M > C::HZ - e && lz < C::HZ + C::TZ + e && lx + VEC > C::HX - e && lx < C::HX + C::TX + e;
    };
    T u[M][VEC], pv[M][VEC], cv[M][VEC];
    {
        const auto bu = buf(a.cur), bp = buf(a.prev), bc = buf(s.c);
        const bool first = active(1);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            bld<0>(u[m], bu, ob[m]);
            bld<0>(pv[m], bp, first ? ob[m] : kOffGrid);
            bld<0>(cv[m], bc, first ? ob[m] : kOffGrid);
        }
    }
    // adjoint sources: the residual enters at the receivers of the whole region
    int code[M][VEC];
    bool any = false, look = false;
    if (strip && xin && s.ev_zlo < gz + M && s.ev_zhi >= gz) strip_events<C>(s, gx, gz, code, any, look);
    const T ramp = T(a.resid_amp);
    const bool edge_x = tx * C::TX - C::HX + W > s.nx;
    const bool edge = edge_x || tx * C::TX < C::HX || tz * C::TZ < C::HZ || tz * C::TZ - C::HZ + C::H > s.nz;

    T *const L0 = lds + (M + lz) * W + lx;
    if (strip) {
#pragma unroll
        for (int m = 0; m < M; ++m) vst(L0 + m * W, u[m]);
    }
    __syncthreads();
#pragma unroll 1
    for (int j = 1; j <= k; ++j) {
        if (active(j)) {
            const T *const rrow = static_cast<const T *>(a.resid) + (a.k0 - j) * s.nrec;
            T rn[M][VEC];
            if (any && !look) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        if (code[m][v] >= 0) rn[m][v] = rrow[code[m][v]];
            }
            T acc[M][VEC], un[M][VEC];
            strip_stencil<C, true>(acc, u, L0 + ((j - 1) & 1) * C::LDS);
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    un[m][v] = fma_t(cv[m][v], acc[m][v], T(2) * u[m][v] - pv[m][v]);
            if (any) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        int c = code[m][v];
                        asm volatile("" : "+v"(c));
                        if (c == kNoEvent) continue;
                        if (!look) {
                            if (c >= 0) un[m][v] = fma_t(ramp * cv[m][v], rn[m][v], un[m][v]);
                        } else {
                            const int hi = s.ev_ptr[gx + v + 1];
                            int e = lower_bound_z(s.ev, s.ev_ptr[gx + v], hi, gz + m);
                            for (; e < hi && s.ev[e].z == gz + m; ++e)
                                if (s.ev[e].code >= 0)
                                    un[m][v] = fma_t(ramp * cv[m][v], rrow[s.ev[e].code], un[m][v]);
                        }
                    }
            }
            if (edge_x) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 1; v < VEC; ++v) un[m][v] = gx + v < s.nx ? un[m][v] : T(0);
            }
            if (edge) {
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) un[m][v] = zin[m] ? un[m][v] : T(0);
            }
            T *Ln = L0 + (j & 1) * C::LDS;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                vst(Ln + m * W, un[m]);
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    pv[m][v] = u[m][v];
                    u[m][v] = un[m][v];
                }
            }
        }
        __syncthreads();
    }
    if (tile) {
        const auto bo = buf(a.out), bq = buf(a.out_prev);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            bst<0>(bo, ob[m], u[m]);
            bst<0>(bq, ob[m], pv[m]);
        }
    }
}

struct Multi2dEntry {
    int tx, tz, kmax;
    int per_cu;  // for grids of up to this many tiles per CU; 0: for any
    void (*launch)(const Multi2dArgs &, hipStream_t);
};

template <class C>
void launch_multi2d(const Multi2dArgs &a, hipStream_t st)
{
    const dim3 grid(a.tiles_x * a.tiles_z), block(C::NT);
    if (a.one.damp)
        hipLaunchKernelGGL((multi2d_kernel<C, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((multi2d_kernel<C, false>), grid, block, 0, st, a);
}

template <class C>
Multi2dEntry multi2d_entry(int per_cu)
{
    return Multi2dEntry{C::TX, C::TZ, C::K, per_cu, &launch_multi2d<C>};
}

struct Adj2dEntry {
    int tx, tz, kmax;
    int per_cu;  // as in Multi2dEntry
    void (*launch)(const Adj2dArgs &, hipStream_t);
};

template <class C>
void launch_adj2d(const Adj2dArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(adj2d_kernel<C>, dim3(a.tiles_x * a.tiles_z), dim3(C::NT + adj2d_image_threads<C>), 0, st, a);
}

template <class C>
Adj2dEntry adj2d_entry(int per_cu)
{
    return Adj2dEntry{C::TX, C::TZ, C::K, per_cu, &launch_adj2d<C>};
}

// Implemented in the per-dtype translation units: the entries of a radius, in order of preference.
const Multi2dEntry *multi2d_configs_f32(int r, int *count);
const Multi2dEntry *multi2d_configs_f64(int r, int *count);
const Adj2dEntry *adj2d_configs_f32(int r, int *count);
const Adj2dEntry *adj2d_configs_f64(int r, int *count);

}  // namespace fdw
