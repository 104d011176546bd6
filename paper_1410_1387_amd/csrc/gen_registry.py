"""Writes the kernel-registry translation units fd_fwd_{f32,f64}.hip,
fd_adj_{f32,f64}.hip and fd_vti_{f32,f64}.hip: explicit template instantiations of the
stencil kernels and the (radius, ndim) -> tile-configuration tables (for the VTI
kernel: (xy radius, z radius) -> tiles) the host side dispatches on.

Tile shapes are (threads along x, threads along y, rows per thread); the first entry
of each list is the default.  Rerun after editing the lists:
    python paper_1410_1387_amd/csrc/gen_registry.py
"""

import os

HERE = os.path.dirname(os.path.abspath(__file__))

# 3-D forward tiles: (shape, role, relative cost per point).  AUTO tiles are what the library
# chooses from by itself (fd_create, fd_batch_set), FINE ones too where z chunks are short,
# TWIN ones are a chosen tile's build for 4 waves per SIMD; OPTION tiles are reached with
# fd_set_tuning alone.  The costs are fitted to sweeps of every tile over cubes of 48 to 512
# points and ten ragged grids (how near the library's choice then comes to the best tile
# stands at tile_cost).
# FP32, radii <= 4.  Tiles of 512 threads, one workgroup per CU, stream best: 512^3 r = 4
# takes 353 us with 128x16, 354 with 64x32, against 414 for 64x16 (256 threads, three
# workgroups per CU, so three times as many places in memory streamed at once); small
# grids and ragged rows are better covered by the smaller tiles (96^3: 7.4 us with 32x8
# against 8.7; 320^3: 87 with 64x32 against 97 with 128x16).
F32_3D_AUTO = [((16, 16, 1), "AUTO", 1.35), ((32, 16, 1), "AUTO", 1.0), ((16, 32, 1), "AUTO", 1.1),
               ((8, 8, 1, None, 0, False, 0), "FINE", 1.25),
               ((32, 16, 1, None, 4, False, 3), "TWIN", 1.0), ((16, 32, 1, None, 4, False, 3), "TWIN", 1.0)]
F32_3D_OPTIONS = [(16, 16, 2), (32, 8, 2), (16, 8, 4), (16, 32, 2), (32, 16, 2), (8, 32, 2), (8, 32, 1),
                  (16, 16, 1, None, 4)]
# FP32, radii above 4: one row per thread (two exceed 256 VGPRs and spill)
F32_3D_BIG_R_AUTO = [((32, 16, 1), "AUTO", 1.0), ((16, 16, 1), "AUTO", 1.1), ((8, 16, 1), "FINE", 1.17)]
F32_3D_BIG_R_OPTIONS = [(32, 8, 1), (16, 32, 1), (32, 16, 1, 2), (32, 8, 1, 2), (64, 8, 1, 2), (16, 16, 1, 2),
                        (64, 4, 1, 2)]
# FP64: 32x32 with two rows per thread or with 512 threads and no early halo (512^3 r = 4:
# 791 and 726 us), 16x16 for small grids (64^3: 6.1 against 6.6 us); radii above 4 keep one
# row per thread (two spill at r >= 7), 64x16 with 512 threads for large grids (384^3 r = 8:
# 362 us against 388 for 32x16)
F64_3D_AUTO = [((16, 16, 2), "AUTO", 1.0), ((16, 32, 1, None, 0, False, 0), "AUTO", 0.95),
               ((8, 16, 1, None, 0, False, 0), "FINE", 1.15)]
F64_3D_OPTIONS = [(32, 16, 1), (32, 8, 2), (16, 16, 1)]
F64_3D_BIG_R_AUTO = [((16, 16, 1), "AUTO", 1.1), ((32, 16, 1), "AUTO", 1.0), ((8, 16, 1), "FINE", 1.17)]
F64_3D_BIG_R_OPTIONS = [(32, 8, 1)]
# FINE tiles of grids that stay in the last-level cache: relative cost per point and planes per
# chunk (224^3 r = 2 FP32: 29.1 us with chunks of 2 planes, 30.0 of 4, 33.9 with 128x16; 192^3
# FP64 35.1 against 39.9; r = 3 FP64 40.2 with 3 planes against 43.8 with 2, twelve cubes of 96
# 64 against 72, but in FP32 192^3 22.4 with 3 against 21.5 with 2).  At larger radii a short
# chunk's first planes cost too much (201x119x333 r = 8: 34.5 us with 4 planes, 31.7 with 128x16).
FINE_CACHED = {"f32": {1: ("0.9f", 2), 2: ("0.9f", 2), 3: ("0.9f", 2), 4: ("1.25f", 4)},
               "f64": {1: ("0.9f", 2), 2: ("0.9f", 2), 3: ("0.9f", 3), 4: ("1.0f", 4)}}
# FP64 r = 4: 512 threads and half the workgroups stream better the longer the chunks (512^3 724
# us against 790, 480^3 624 against 685, 352^3 245 against 261, 256^3 84.4 against 84.7).  Not
# measured at r = 1 to 3, which keep the cost of the tile table
COSTS = {("f64", 4, (16, 32, 1)): 0.85}
SWEEP_RADII = {4, 8}      # radii that get the OPTION tiles
F2D = (64, 1, 1)          # 2-D forward and adjoint: one row of 64 threads; chunks as FINE tiles'
# 3-D adjoint tiles: (shape, role, relative cost per point); half of a tile's threads own mu,
# half u, so a workgroup has twice the threads of the shape.  FP32, radii <= 4: the library
# takes the 128-wide tile or one of the 64-wide ones by how rows fill them, then the cheaper
# (per step: 256^3 r = 4 87 us with 128x16, 94 with 64x16; 320^3 180 with 64x32, 191 with
# 128x16; 64^3 5.2 with 64x16, 6.7 with 128x16).
ADJ_F32_3D = [((32, 16, 1), "AUTO", 1.0), ((16, 32, 1), "AUTO", 1.0), ((16, 16, 1), "AUTO", 1.05)]
ADJ_F32_3D_OPTIONS = [(8, 16, 1), (32, 8, 1), (8, 8, 1)]
# radii above 4: 32x8 (192^3 r = 8: 56 us against 61 for 64x16), 64x16 where a chunk is one
# plane (64^3: 6.6 us against 7.2)
ADJ_F32_3D_BIG_R = [((8, 8, 1), "AUTO", 1.0), ((16, 16, 1), "ONE_PLANE", 1.0)]
# FP64: radii <= 4 64x16, two rows per thread (192^3 r = 4: 74 us against 84 with one row and
# 1024 threads, which spills); radii above 4 16x16 (160^3 r = 8: 63 us against 75 for 64x8)
ADJ_F64_3D = [((32, 8, 2), "AUTO", 1.0)]
ADJ_F64_3D_BIG_R = [((8, 16, 1), "AUTO", 1.0)]
ADJ_OPTION_RADII = {4}
# VTI kernel: (xy radius, z radius) pairs and tile shapes (threads along x, rows along y)
VTI_RADII = [(2, 1), (2, 2), (4, 1), (4, 2), (4, 4), (8, 1), (8, 2), (8, 4), (8, 8),
             (12, 1), (12, 2), (12, 4), (12, 8)]
# candidates with their relative cost per point (512^3 R_xy = 12, R_z = 8: 831 us with
# 128x16, 899 with 64x16; 96^3 11.6 with 32x8, 12.4 with 128x16), and options
VTI_F32 = [((16, 16), "AUTO", 1.1), ((32, 16), "AUTO", 1.0), ((8, 8), "AUTO", 1.12)]
VTI_F64 = [((16, 16), "AUTO", 1.2), ((32, 16), "AUTO", 1.0), ((8, 8), "AUTO", 1.2)]
VTI_OPTIONS = [((32, 8), "OPTION", 1.0), ((16, 8), "OPTION", 1.0)]
VTI_SWEEP = {(12, 8), (4, 4)}

HDR = """// {fname} -- explicit instantiations of the {what} stencil kernels for {T}
// and the (radius, ndim) -> tile-configuration table the host side dispatches on.
// Written by gen_registry.py; edit the tile lists there.
#include "fd_stencil.h"

namespace fdw {{
"""


def cfgname(T, R, nd, txn, tyn, ey, vec=None, occ=0):
    full = 4 if T == "float" else 2
    vec = vec or full
    bx = txn * vec
    by = tyn * ey if nd == 3 else 1
    nt = txn * (tyn if nd == 3 else 1)
    name = f"{'f32' if T == 'float' else 'f64'} r{R} {nd}d tile {bx}x{by} ({nt} thr, {ey if nd == 3 else 1} row/thr"
    if vec != full:
        name += f", {vec * (4 if T == 'float' else 8)}-byte vectors"
    if occ:
        name += f", built for {occ} waves/SIMD"
    return name + ")"


def tilecfg(T, R, nd, txn, tyn, ey, vec=None, occ=0, lean=None, hoff=None):
    """TileCfg<...> for a tile tuple (threads along x, threads along y, rows per thread
    [, x points per thread (None: one 16-byte vector) [, waves per SIMD the forward
    kernel is built for (0: the compiler's choice) [, one set of prefetch registers
    [, planes the halo is fetched ahead]]]])."""
    full = 4 if T == "float" else 2
    args = [T, R, nd, txn, tyn, ey]
    if vec or occ or lean is not None:
        args.append(vec or full)
    if occ or lean is not None:
        args.append(occ)
    if lean is not None:
        args += ["true" if lean else "false", min(hoff, R)]
    return f"TileCfg<{', '.join(str(a) for a in args)}>"


def fwd_file(T, auto, options, auto_big_r, options_big_r):
    """Forward kernels: one section per radius, compiled one object each (FD_RADIUS)."""
    tag = "f32" if T == "float" else "f64"
    out = HDR.format(fname=f"fd_fwd_{tag}.hip", what="forward", T=T)
    out = out.replace("namespace fdw {\n", "// Compiled once per radius, with FD_RADIUS set.\nnamespace fdw {\n")
    for R in range(1, 9):
        au, op = (auto, options) if R <= 4 else (auto_big_r, options_big_r)
        rows = [au[0]]
        if R in SWEEP_RADII:  # the options keep their numbers; at R > 4 the second tile is one of them
            rows += (au[1:2] if R > 4 else []) + [(o, "OPTION", 1.0) for o in op] + (au[2:] if R > 4 else au[1:])
        else:
            rows += au[1:]
        out += f"#if FD_RADIUS == {R}\nstatic const FwdEntry k3[] = {{\n"
        for cfg, role, cost in rows:
            cost = COSTS.get((tag, R, cfg[:3]), cost) if role == "AUTO" else cost
            name = cfgname(T, R, 3, *cfg[:5])
            cached = "".join(f", {v}" for v in FINE_CACHED[tag].get(R, ())) if role == "FINE" else ""
            out += f'    fwd_entry<{tilecfg(T, R, 3, *cfg)}, FWD_{role}>("{name}", {cost}f{cached}),\n'
        out += "};\n"
        txn = F2D[0]
        out += f"static const FwdEntry k2[] = {{\n"
        out += f'    fwd_entry<TileCfg<{T}, {R}, 2, {txn}, 1, 1>, FWD_AUTO>("{cfgname(T, R, 2, txn, 1, 1)}", 1.0f, 1.0f, 4),\n'
        out += "};\n#endif\n"
    out += ("\n#define FD_CAT_(a, b) a##b\n#define FD_CAT(a, b) FD_CAT_(a, b)\n"
            f"const FwdEntry *FD_CAT(fwd_configs_{tag}_r, FD_RADIUS)(int ndim, int *count)\n{{\n"
            "    *count = (int)((ndim == 3 ? sizeof(k3) : sizeof(k2)) / sizeof(FwdEntry));\n"
            "    return ndim == 3 ? k3 : k2;\n}\n\n#if FD_RADIUS == 1\n")
    for R in range(2, 9):
        out += f"const FwdEntry *fwd_configs_{tag}_r{R}(int ndim, int *count);\n"
    out += f"const FwdEntry *fwd_configs_{tag}(int r, int ndim, int *count)\n{{\n    *count = 0;\n"
    out += "    if (ndim != 2 && ndim != 3) return nullptr;\n    switch (r) {\n"
    for R in range(1, 9):
        out += f"    case {R}: return fwd_configs_{tag}_r{R}(ndim, count);\n"
    out += "    default: return nullptr;\n    }\n}\n#endif\n\n}  // namespace fdw\n"
    with open(os.path.join(HERE, f"fd_fwd_{tag}.hip"), "w") as f:
        f.write(out)


def adj_file(T, d3, d3_big_r, options=()):
    """Adjoint kernels: the 3-D tiles of each radius and one 2-D shape.  No early halo: its
    ring measured 2 % faster at 512^3 and slower everywhere below."""
    tag = "f32" if T == "float" else "f64"
    out = HDR.format(fname=f"fd_adj_{tag}.hip", what="adjoint", T=T)
    for R in range(1, 9):
        lst = d3 if R <= 4 else d3_big_r
        lst = lst + [(o, "OPTION", 1.0) for o in options if R in ADJ_OPTION_RADII]
        out += f"static const AdjEntry a3_r{R}[] = {{\n"
        for cfg, role, cost in lst:
            out += (f'    adj_entry<{tilecfg(T, R, 3, *cfg, None, 0, False, 0)}, ADJ_{role}>('
                    f'"{cfgname(T, R, 3, *cfg)}", {cost}f),\n')
        out += "};\n"
        txn = F2D[0]
        out += (f"static const AdjEntry a2_r{R}[] = {{adj_entry<{tilecfg(T, R, 2, txn, 1, 1, None, 0, False, 0)}, ADJ_AUTO>"
                f'("{cfgname(T, R, 2, txn, 1, 1)}", 1.0f)}};\n')
    out += "\nconst AdjEntry *adj_configs_" + tag + "(int r, int ndim, int *count)\n{\n    switch (r * 10 + ndim) {\n"
    for R in range(1, 9):
        for nd in (2, 3):
            out += (f"    case {R * 10 + nd}: *count = (int)(sizeof(a{nd}_r{R}) / sizeof(AdjEntry)); "
                    f"return a{nd}_r{R};\n")
    out += "    default: *count = 0; return nullptr;\n    }\n}\n\n"
    out += "}  // namespace fdw\n"
    with open(os.path.join(HERE, f"fd_adj_{tag}.hip"), "w") as f:
        f.write(out)


def vti_file(T, tiles):
    tag = "f32" if T == "float" else "f64"
    vec = 4 if T == "float" else 2
    out = HDR.format(fname=f"fd_vti_{tag}.hip", what="VTI", T=T).replace('#include "fd_stencil.h"',
                                                                         '#include "fd_vti.h"')
    for (rxy, rz) in VTI_RADII:
        lst = tiles + (VTI_OPTIONS if (rxy, rz) in VTI_SWEEP else [])
        out += f"static const VtiEntry v_{rxy}_{rz}[] = {{\n"
        for (txn, tyn), role, cost in lst:
            name = f"{tag} vti rxy{rxy} rz{rz} tile {txn * vec}x{tyn} ({txn * tyn} thr)"
            out += f'    vti_entry<VtiCfg<{T}, {rxy}, {rz}, {txn}, {tyn}>, VTI_{role}>("{name}", {cost}f),\n'
        out += "};\n"
    out += "\nconst VtiEntry *vti_configs_" + tag + "(int rxy, int rz, int *count)\n{\n    switch (rxy * 100 + rz) {\n"
    for (rxy, rz) in VTI_RADII:
        out += (f"    case {rxy * 100 + rz}: *count = (int)(sizeof(v_{rxy}_{rz}) / sizeof(VtiEntry)); "
                f"return v_{rxy}_{rz};\n")
    out += "    default: *count = 0; return nullptr;\n    }\n}\n\n}  // namespace fdw\n"
    with open(os.path.join(HERE, f"fd_vti_{tag}.hip"), "w") as f:
        f.write(out)


if __name__ == "__main__":
    fwd_file("float", F32_3D_AUTO, F32_3D_OPTIONS, F32_3D_BIG_R_AUTO, F32_3D_BIG_R_OPTIONS)
    fwd_file("double", F64_3D_AUTO, F64_3D_OPTIONS, F64_3D_BIG_R_AUTO, F64_3D_BIG_R_OPTIONS)
    adj_file("float", ADJ_F32_3D, ADJ_F32_3D_BIG_R, ADJ_F32_3D_OPTIONS)
    adj_file("double", ADJ_F64_3D, ADJ_F64_3D_BIG_R)
    vti_file("float", VTI_F32)
    vti_file("double", VTI_F64)
