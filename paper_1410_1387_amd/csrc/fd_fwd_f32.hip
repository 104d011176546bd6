// fd_fwd_f32.hip -- explicit instantiations of the forward stencil kernels for float
// and the (radius, ndim) -> tile-configuration table the host side dispatches on.
// Written by gen_registry.py; edit the tile lists there.
#include "fd_stencil.h"

// Compiled once per radius, with FD_RADIUS set.
namespace fdw {
#if FD_RADIUS == 1
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 1, 3, 16, 16, 1>, FWD_AUTO>("f32 r1 3d tile 64x16 (256 thr, 1 row/thr)", 1.35f),
    fwd_entry<TileCfg<float, 1, 3, 32, 16, 1>, FWD_AUTO>("f32 r1 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 1, 3, 16, 32, 1>, FWD_AUTO>("f32 r1 3d tile 64x32 (512 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 1, 3, 8, 8, 1, 4, 0, false, 0>, FWD_FINE>("f32 r1 3d tile 32x8 (64 thr, 1 row/thr)", 1.25f, 0.9f, 2),
    fwd_entry<TileCfg<float, 1, 3, 32, 16, 1, 4, 4, false, 1>, FWD_TWIN>("f32 r1 3d tile 128x16 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
    fwd_entry<TileCfg<float, 1, 3, 16, 32, 1, 4, 4, false, 1>, FWD_TWIN>("f32 r1 3d tile 64x32 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 1, 2, 64, 1, 1>, FWD_AUTO>("f32 r1 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 2
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 2, 3, 16, 16, 1>, FWD_AUTO>("f32 r2 3d tile 64x16 (256 thr, 1 row/thr)", 1.35f),
    fwd_entry<TileCfg<float, 2, 3, 32, 16, 1>, FWD_AUTO>("f32 r2 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 2, 3, 16, 32, 1>, FWD_AUTO>("f32 r2 3d tile 64x32 (512 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 2, 3, 8, 8, 1, 4, 0, false, 0>, FWD_FINE>("f32 r2 3d tile 32x8 (64 thr, 1 row/thr)", 1.25f, 0.9f, 2),
    fwd_entry<TileCfg<float, 2, 3, 32, 16, 1, 4, 4, false, 2>, FWD_TWIN>("f32 r2 3d tile 128x16 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
    fwd_entry<TileCfg<float, 2, 3, 16, 32, 1, 4, 4, false, 2>, FWD_TWIN>("f32 r2 3d tile 64x32 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 2, 2, 64, 1, 1>, FWD_AUTO>("f32 r2 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 3
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 3, 3, 16, 16, 1>, FWD_AUTO>("f32 r3 3d tile 64x16 (256 thr, 1 row/thr)", 1.35f),
    fwd_entry<TileCfg<float, 3, 3, 32, 16, 1>, FWD_AUTO>("f32 r3 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 3, 3, 16, 32, 1>, FWD_AUTO>("f32 r3 3d tile 64x32 (512 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 3, 3, 8, 8, 1, 4, 0, false, 0>, FWD_FINE>("f32 r3 3d tile 32x8 (64 thr, 1 row/thr)", 1.25f, 0.9f, 2),
    fwd_entry<TileCfg<float, 3, 3, 32, 16, 1, 4, 4, false, 3>, FWD_TWIN>("f32 r3 3d tile 128x16 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
    fwd_entry<TileCfg<float, 3, 3, 16, 32, 1, 4, 4, false, 3>, FWD_TWIN>("f32 r3 3d tile 64x32 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 3, 2, 64, 1, 1>, FWD_AUTO>("f32 r3 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 4
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 4, 3, 16, 16, 1>, FWD_AUTO>("f32 r4 3d tile 64x16 (256 thr, 1 row/thr)", 1.35f),
    fwd_entry<TileCfg<float, 4, 3, 16, 16, 2>, FWD_OPTION>("f32 r4 3d tile 64x32 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 32, 8, 2>, FWD_OPTION>("f32 r4 3d tile 128x16 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 16, 8, 4>, FWD_OPTION>("f32 r4 3d tile 64x32 (128 thr, 4 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 16, 32, 2>, FWD_OPTION>("f32 r4 3d tile 64x64 (512 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 32, 16, 2>, FWD_OPTION>("f32 r4 3d tile 128x32 (512 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 8, 32, 2>, FWD_OPTION>("f32 r4 3d tile 32x64 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 8, 32, 1>, FWD_OPTION>("f32 r4 3d tile 32x32 (256 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 16, 16, 1, 4, 4>, FWD_OPTION>("f32 r4 3d tile 64x16 (256 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 32, 16, 1>, FWD_AUTO>("f32 r4 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 16, 32, 1>, FWD_AUTO>("f32 r4 3d tile 64x32 (512 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 4, 3, 8, 8, 1, 4, 0, false, 0>, FWD_FINE>("f32 r4 3d tile 32x8 (64 thr, 1 row/thr)", 1.25f, 1.25f, 4),
    fwd_entry<TileCfg<float, 4, 3, 32, 16, 1, 4, 4, false, 3>, FWD_TWIN>("f32 r4 3d tile 128x16 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
    fwd_entry<TileCfg<float, 4, 3, 16, 32, 1, 4, 4, false, 3>, FWD_TWIN>("f32 r4 3d tile 64x32 (512 thr, 1 row/thr, built for 4 waves/SIMD)", 1.0f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 4, 2, 64, 1, 1>, FWD_AUTO>("f32 r4 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 5
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 5, 3, 32, 16, 1>, FWD_AUTO>("f32 r5 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 5, 3, 16, 16, 1>, FWD_AUTO>("f32 r5 3d tile 64x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 5, 3, 8, 16, 1>, FWD_FINE>("f32 r5 3d tile 32x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 5, 2, 64, 1, 1>, FWD_AUTO>("f32 r5 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 6
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 6, 3, 32, 16, 1>, FWD_AUTO>("f32 r6 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 6, 3, 16, 16, 1>, FWD_AUTO>("f32 r6 3d tile 64x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 6, 3, 8, 16, 1>, FWD_FINE>("f32 r6 3d tile 32x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 6, 2, 64, 1, 1>, FWD_AUTO>("f32 r6 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 7
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 7, 3, 32, 16, 1>, FWD_AUTO>("f32 r7 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 7, 3, 16, 16, 1>, FWD_AUTO>("f32 r7 3d tile 64x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 7, 3, 8, 16, 1>, FWD_FINE>("f32 r7 3d tile 32x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 7, 2, 64, 1, 1>, FWD_AUTO>("f32 r7 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 8
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<float, 8, 3, 32, 16, 1>, FWD_AUTO>("f32 r8 3d tile 128x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 16, 16, 1>, FWD_AUTO>("f32 r8 3d tile 64x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<float, 8, 3, 32, 8, 1>, FWD_OPTION>("f32 r8 3d tile 128x8 (256 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 16, 32, 1>, FWD_OPTION>("f32 r8 3d tile 64x32 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 32, 16, 1, 2>, FWD_OPTION>("f32 r8 3d tile 64x16 (512 thr, 1 row/thr, 8-byte vectors)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 32, 8, 1, 2>, FWD_OPTION>("f32 r8 3d tile 64x8 (256 thr, 1 row/thr, 8-byte vectors)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 64, 8, 1, 2>, FWD_OPTION>("f32 r8 3d tile 128x8 (512 thr, 1 row/thr, 8-byte vectors)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 16, 16, 1, 2>, FWD_OPTION>("f32 r8 3d tile 32x16 (256 thr, 1 row/thr, 8-byte vectors)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 64, 4, 1, 2>, FWD_OPTION>("f32 r8 3d tile 128x4 (256 thr, 1 row/thr, 8-byte vectors)", 1.0f),
    fwd_entry<TileCfg<float, 8, 3, 8, 16, 1>, FWD_FINE>("f32 r8 3d tile 32x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<float, 8, 2, 64, 1, 1>, FWD_AUTO>("f32 r8 2d tile 256x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif

#define FD_CAT_(a, b) a##b
#define FD_CAT(a, b) FD_CAT_(a, b)
const FwdEntry *FD_CAT(fwd_configs_f32_r, FD_RADIUS)(int ndim, int *count)
{
    *count = (int)((ndim == 3 ? sizeof(k3) : sizeof(k2)) / sizeof(FwdEntry));
    return ndim == 3 ? k3 : k2;
}

#if FD_RADIUS == 1
const FwdEntry *fwd_configs_f32_r2(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r3(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r4(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r5(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r6(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r7(int ndim, int *count);
const FwdEntry *fwd_configs_f32_r8(int ndim, int *count);
const FwdEntry *fwd_configs_f32(int r, int ndim, int *count)
{
    *count = 0;
    if (ndim != 2 && ndim != 3) return nullptr;
    switch (r) {
    case 1: return fwd_configs_f32_r1(ndim, count);
    case 2: return fwd_configs_f32_r2(ndim, count);
    case 3: return fwd_configs_f32_r3(ndim, count);
    case 4: return fwd_configs_f32_r4(ndim, count);
    case 5: return fwd_configs_f32_r5(ndim, count);
    case 6: return fwd_configs_f32_r6(ndim, count);
    case 7: return fwd_configs_f32_r7(ndim, count);
    case 8: return fwd_configs_f32_r8(ndim, count);
    default: return nullptr;
    }
}
#endif

}  // namespace fdw
