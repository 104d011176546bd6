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
// What bounds it: the vector work of the widened region (r = 4, k = 4, 32 x 16 points: 2.6
// times the tile's) and, on small grids, the latency of load, k steps and store.
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

template <class C, bool DAMP>
__global__ __launch_bounds__(C::NT) void multi2d_kernel(Multi2dArgs a)
{
    typedef typename C::type T;
    constexpr int R = C::R, M = C::M, VEC = C::VEC, LPAD = C::LPAD, W = C::W;
    constexpr StencilWeights<R> Wt{};
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

    // receivers of the strip's points inside the tile; several at one point are looked up
    int code[M][VEC];
    bool any = false, look = false;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int v = 0; v < VEC; ++v) code[m][v] = kNoEvent;
    if (a.record && s.ev_ptr && s.ev_zlo < (tz + 1) * C::TZ && s.ev_zhi >= tz * C::TZ && tile && xin) {
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
            T un[M][VEC];
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
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const T u0 = u[m][v];
                    T acc;
                    if constexpr (R > 4) {
                        acc = T(2 * Wt.w[0]) * u0;
#pragma unroll
                        for (int l = 1; l <= R; ++l) acc = fma_t(T(Wt.w[l]), xs[LPAD + v + l] + xs[LPAD + v - l], acc);
#pragma unroll
                        for (int l = 1; l <= R; ++l) acc = fma_t(T(Wt.w[l]), zw[R + m + l][v] + zw[R + m - l][v], acc);
                    } else {
                        acc = T(0);
#pragma unroll
                        for (int l = 1; l <= R; ++l)
                            acc = fma_t(T(Wt.w[l]), (xs[LPAD + v + l] - u0) + (xs[LPAD + v - l] - u0), acc);
#pragma unroll
                        for (int l = 1; l <= R; ++l)
                            acc = fma_t(T(Wt.w[l]), (zw[R + m + l][v] - u0) + (zw[R + m - l][v] - u0), acc);
                    }
                    if constexpr (DAMP) {
                        const T G = gxv[v] * gzv[m];
                        un[m][v] = G * fma_t(cv[m][v], acc, T(2) * u0 - G * pv[m][v]);
                    } else {
                        un[m][v] = fma_t(cv[m][v], acc, T(2) * u0 - pv[m][v]);
                    }
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

// Implemented in the per-dtype translation units: the entries of a radius, in order of preference.
const Multi2dEntry *multi2d_configs_f32(int r, int *count);
const Multi2dEntry *multi2d_configs_f64(int r, int *count);

}  // namespace fdw
