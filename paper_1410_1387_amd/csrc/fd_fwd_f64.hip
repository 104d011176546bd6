// fd_fwd_f64.hip -- explicit instantiations of the forward stencil kernels for double
// and the (radius, ndim) -> tile-configuration table the host side dispatches on.
// Written by gen_registry.py; edit the tile lists there.
#include "fd_stencil.h"

// Compiled once per radius, with FD_RADIUS set.
namespace fdw {
#if FD_RADIUS == 1
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 1, 3, 16, 16, 2>, FWD_AUTO>("f64 r1 3d tile 32x32 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 1, 3, 16, 32, 1, 2, 0, false, 0>, FWD_AUTO>("f64 r1 3d tile 32x32 (512 thr, 1 row/thr)", 0.95f),
    fwd_entry<TileCfg<double, 1, 3, 8, 16, 1, 2, 0, false, 0>, FWD_FINE>("f64 r1 3d tile 16x16 (128 thr, 1 row/thr)", 1.15f, 0.9f, 2),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 1, 2, 64, 1, 1>, FWD_AUTO>("f64 r1 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 2
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 2, 3, 16, 16, 2>, FWD_AUTO>("f64 r2 3d tile 32x32 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 2, 3, 16, 32, 1, 2, 0, false, 0>, FWD_AUTO>("f64 r2 3d tile 32x32 (512 thr, 1 row/thr)", 0.95f),
    fwd_entry<TileCfg<double, 2, 3, 8, 16, 1, 2, 0, false, 0>, FWD_FINE>("f64 r2 3d tile 16x16 (128 thr, 1 row/thr)", 1.15f, 0.9f, 2),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 2, 2, 64, 1, 1>, FWD_AUTO>("f64 r2 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 3
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 3, 3, 16, 16, 2>, FWD_AUTO>("f64 r3 3d tile 32x32 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 3, 3, 16, 32, 1, 2, 0, false, 0>, FWD_AUTO>("f64 r3 3d tile 32x32 (512 thr, 1 row/thr)", 0.95f),
    fwd_entry<TileCfg<double, 3, 3, 8, 16, 1, 2, 0, false, 0>, FWD_FINE>("f64 r3 3d tile 16x16 (128 thr, 1 row/thr)", 1.15f, 0.9f, 3),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 3, 2, 64, 1, 1>, FWD_AUTO>("f64 r3 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 4
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 4, 3, 16, 16, 2>, FWD_AUTO>("f64 r4 3d tile 32x32 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 4, 3, 32, 16, 1>, FWD_OPTION>("f64 r4 3d tile 64x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 4, 3, 32, 8, 2>, FWD_OPTION>("f64 r4 3d tile 64x16 (256 thr, 2 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 4, 3, 16, 16, 1>, FWD_OPTION>("f64 r4 3d tile 32x16 (256 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 4, 3, 16, 32, 1, 2, 0, false, 0>, FWD_AUTO>("f64 r4 3d tile 32x32 (512 thr, 1 row/thr)", 0.85f),
    fwd_entry<TileCfg<double, 4, 3, 8, 16, 1, 2, 0, false, 0>, FWD_FINE>("f64 r4 3d tile 16x16 (128 thr, 1 row/thr)", 1.15f, 1.0f, 4),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 4, 2, 64, 1, 1>, FWD_AUTO>("f64 r4 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 5
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 5, 3, 16, 16, 1>, FWD_AUTO>("f64 r5 3d tile 32x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<double, 5, 3, 32, 16, 1>, FWD_AUTO>("f64 r5 3d tile 64x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 5, 3, 8, 16, 1>, FWD_FINE>("f64 r5 3d tile 16x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 5, 2, 64, 1, 1>, FWD_AUTO>("f64 r5 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 6
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 6, 3, 16, 16, 1>, FWD_AUTO>("f64 r6 3d tile 32x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<double, 6, 3, 32, 16, 1>, FWD_AUTO>("f64 r6 3d tile 64x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 6, 3, 8, 16, 1>, FWD_FINE>("f64 r6 3d tile 16x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 6, 2, 64, 1, 1>, FWD_AUTO>("f64 r6 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 7
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 7, 3, 16, 16, 1>, FWD_AUTO>("f64 r7 3d tile 32x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<double, 7, 3, 32, 16, 1>, FWD_AUTO>("f64 r7 3d tile 64x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 7, 3, 8, 16, 1>, FWD_FINE>("f64 r7 3d tile 16x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 7, 2, 64, 1, 1>, FWD_AUTO>("f64 r7 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif
#if FD_RADIUS == 8
static const FwdEntry k3[] = {
    fwd_entry<TileCfg<double, 8, 3, 16, 16, 1>, FWD_AUTO>("f64 r8 3d tile 32x16 (256 thr, 1 row/thr)", 1.1f),
    fwd_entry<TileCfg<double, 8, 3, 32, 16, 1>, FWD_AUTO>("f64 r8 3d tile 64x16 (512 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 8, 3, 32, 8, 1>, FWD_OPTION>("f64 r8 3d tile 64x8 (256 thr, 1 row/thr)", 1.0f),
    fwd_entry<TileCfg<double, 8, 3, 8, 16, 1>, FWD_FINE>("f64 r8 3d tile 16x16 (128 thr, 1 row/thr)", 1.17f),
};
static const FwdEntry k2[] = {
    fwd_entry<TileCfg<double, 8, 2, 64, 1, 1>, FWD_AUTO>("f64 r8 2d tile 128x1 (64 thr, 1 row/thr)", 1.0f, 1.0f, 4),
};
#endif

#define FD_CAT_(a, b) a##b
#define FD_CAT(a, b) FD_CAT_(a, b)
const FwdEntry *FD_CAT(fwd_configs_f64_r, FD_RADIUS)(int ndim, int *count)
{
    *count = (int)((ndim == 3 ? sizeof(k3) : sizeof(k2)) / sizeof(FwdEntry));
    return ndim == 3 ? k3 : k2;
}

#if FD_RADIUS == 1
const FwdEntry *fwd_configs_f64_r2(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r3(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r4(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r5(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r6(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r7(int ndim, int *count);
const FwdEntry *fwd_configs_f64_r8(int ndim, int *count);
const FwdEntry *fwd_configs_f64(int r, int ndim, int *count)
{
    *count = 0;
    if (ndim != 2 && ndim != 3) return nullptr;
    switch (r) {
    case 1: return fwd_configs_f64_r1(ndim, count);
    case 2: return fwd_configs_f64_r2(ndim, count);
    case 3: return fwd_configs_f64_r3(ndim, count);
    case 4: return fwd_configs_f64_r4(ndim, count);
    case 5: return fwd_configs_f64_r5(ndim, count);
    case 6: return fwd_configs_f64_r6(ndim, count);
    case 7: return fwd_configs_f64_r7(ndim, count);
    case 8: return fwd_configs_f64_r8(ndim, count);
    default: return nullptr;
    }
}
#endif

}  // namespace fdw
