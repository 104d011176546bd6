// fd_host.h -- host-side helpers shared by the translation units of the C ABI
// (library-internal, hidden from the exported symbol table).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace fdw {

// Records a printf-style message as the calling thread's last error and returns code.
__attribute__((visibility("hidden"), format(printf, 2, 3))) int host_fail(int code, const char *fmt, ...);

// Compute units of the current device.
__attribute__((visibility("hidden"))) int device_cus();

// Workgroups of `kernel` (nt threads) the whole device runs at once.
__attribute__((visibility("hidden"))) int resident_slots(const void *kernel, int nt);

// Whether calls on `stream` are being captured into a graph (the null stream cannot be).
__attribute__((visibility("hidden"))) bool capturing(hipStream_t stream);

// Planes per z chunk for tiles_xy tiles over nz planes with a z halo of r planes.
__attribute__((visibility("hidden"))) int choose_zch(int64_t tiles_xy, int64_t nz, int r, int slots);

// Estimated time of one launch, in points: the points the busiest CU computes (its share of
// the workgroups, idle lanes and a prologue of 0.3 r planes included) at the tile's own
// cost, the latency of a chunk's planes, about 300 points each, and of a workgroup's start,
// longer the more waves it has.  Only its order among the tiles of one grid matters: over
// cubes of 48 to 512 points and ten ragged grids it picks a tile within 2 % of the best on
// average (at worst 5 % off for radius 4, 9 % for one cube at radius 6).
template <class Entry>
double tile_cost(const Entry &e, int64_t nwg, int64_t zch, int r, int cus)
{
    return (double)((nwg + cus - 1) / cus) * e.bx * e.by * e.cost * ((double)zch + 0.3 * r) + 300.0 * (double)zch +
           1.5 * e.nt;
}

// The same for a FINE tile on fields that stay in the last-level cache: its many workgroups
// hide each other's latency.  With it the choice over 13 such grids is within 1 % of the best
// tile and chunk on average for r <= 3 (6 % without), 2 % for r = 4 (7 %), 2-3 % in FP64 (7 %).
template <class Entry>
double cached_tile_cost(const Entry &e, int64_t nwg, int64_t zch, int r, int cus)
{
    return (double)((nwg + cus - 1) / cus) * e.bx * e.by * e.cached_cost * ((double)zch + 0.3 * r) + 1.5 * e.nt;
}

// Whether `bytes` of fields that every step reads and writes stay in the 256 MB last-level
// cache from one step to the next.  Then loads that a step makes once per point (u^{n-1},
// c, ...) keep their lines; otherwise they are nontemporal, so that they do not push out the
// lines of u^n that neighbouring tiles share.  Measured, nontemporal -> cached, us per step:
// 96x118x141 FP32 r = 4 10.3 -> 9.1, 160^3 19.1 -> 16.2, 192^3 (85 MB) 25.3 -> 23.6, 256^3
// (201 MB) 45.8 -> 44.2; past the line 480x303x130 (227 MB) 69.4 -> 70.5, 140x440x330 (244
// MB) 60.0 -> 60.5, 288^3 (287 MB) 73.6 -> 76.1, 320^3 (393 MB) 87.6 -> 109; VTI 192^3 (198
// MB) 62 -> 57.6, 160^3 FP64 (229 MB) 50.6 -> 50.9, 256^3 (470 MB) 103 -> 124.
constexpr double kCacheBytes = 208.0 * (1 << 20);
inline bool cache_keeps(double bytes) { return bytes <= kCacheBytes; }

// Planes per chunk of a FINE tile, or rows of a 2-D one, on fields that stay in the last-level cache; count(Z) is
// the number of workgroups with chunks of at most Z of nz planes.  Where there are plenty,
// short chunks in many rounds are best: a chunk's first planes come from the L2 that the
// chunk below has just filled, and the CUs stay balanced.  Otherwise one round, but of at
// most eight waves per CU: more of them push each other's planes out.  Best measured length
// against one round of all places, us per step: 201x119x333 r = 2 2 planes 22.1 (9: 25.1),
// r = 4 4 planes 25.5 (12: 29.9); 160^3 r = 4 8 planes 15.2 (6: 15.8), 93x118x141 4 planes
// 8.2 (3: 8.4); a batch of seven 78..152-cubes 6 planes 50.9 (23: 55);
// 2-D 4096^2 r = 8 4 rows 39.7 (22: 51), 2500^2 FP64 4 rows 30.6 (17: 39), 1203x801 r = 5 2
// rows 6.2 (1: 6.6).
template <class Count>
int fine_zch(const Count &count, int64_t nz, int nt, int short_zch, int cus)
{
    const int64_t waves = nt / 64;
    if (count(std::min<int64_t>(4, nz)) * waves >= 20 * cus) return (int)std::min<int64_t>(short_zch, nz);
    int64_t z = 1;
    while (z < nz && count(z) * waves > 8 * cus) ++z;
    return (int)z;
}

// A tile entry (bx x by points, nt threads, its kernel) laid out over one grid.
template <class Entry>
struct TileChoice {
    const Entry *e = nullptr;
    int64_t tx = 0, ty = 0, nwg = 0;
    int zch = 0;
};

template <class Entry>
TileChoice<Entry> plan_tile(const Entry &e, int64_t nx, int64_t ny, int64_t nz, int r)
{
    TileChoice<Entry> t;
    t.e = &e;
    t.tx = (nx + e.bx - 1) / e.bx;
    t.ty = (ny + e.by - 1) / e.by;
    t.zch = choose_zch(t.tx * t.ty, nz, r, resident_slots(e.kernel, e.nt));
    t.nwg = t.tx * t.ty * ((nz + t.zch - 1) / t.zch);
    return t;
}

}  // namespace fdw
