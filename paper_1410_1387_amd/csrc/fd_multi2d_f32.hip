// fd_multi2d_f32.hip -- the several-steps-per-launch kernels of 2-D F32 grids.
//
// Microseconds per step measured on this card, single-step kernel -> these, by grid:
//          256^2         512^2         1203 x 800    1600^2
//   r = 1  4.11 -> 2.14  4.27 -> 2.15  5.43 -> 2.35   8.40 -> 3.37
//   r = 2  4.29 -> 2.37  4.48 -> 2.41  5.94 -> 3.37   9.10 -> 5.36
//   r = 3  4.39 -> 2.66  4.65 -> 2.69  6.41 -> 3.62   9.72 -> 9.04
//   r = 4  4.52 -> 2.84  4.85 -> 2.90  6.81 -> 4.37  10.30 -> 9.22
//   r = 5  4.31 -> 2.87  4.52 -> 2.89  6.31 (2 steps, 64x32: 6.90)
//   r = 6  4.40 -> 3.15  4.62 -> 3.14  6.56 (2 steps, 64x32: 7.20)
//   r = 7  4.49 -> 3.52  4.70 -> 3.50  6.05 (2 steps, 64x32: 7.63)
//   r = 8  4.55 -> 3.98  4.86 -> 4.05  6.28 (2 steps, 64x32: 7.36)
#include "fd_multi2d.h"

namespace fdw {

static const Multi2dEntry m_r1[] = {
    multi2d_entry<Multi2dCfg<float, 1, 8, 64, 32>>(0),
};
static const Multi2dEntry m_r2[] = {
    multi2d_entry<Multi2dCfg<float, 2, 8, 32, 32>>(1),
    multi2d_entry<Multi2dCfg<float, 2, 4, 64, 32>>(0),
};
static const Multi2dEntry m_r3[] = {
    multi2d_entry<Multi2dCfg<float, 3, 8, 32, 32>>(1),
    multi2d_entry<Multi2dCfg<float, 3, 4, 64, 32>>(0),
};
static const Multi2dEntry m_r4[] = {
    multi2d_entry<Multi2dCfg<float, 4, 8, 32, 32>>(1),
    multi2d_entry<Multi2dCfg<float, 4, 3, 64, 32>>(2),
    multi2d_entry<Multi2dCfg<float, 4, 2, 64, 32>>(0),
};
static const Multi2dEntry m_r5[] = {
    multi2d_entry<Multi2dCfg<float, 5, 6, 32, 32>>(1),
};
static const Multi2dEntry m_r6[] = {
    multi2d_entry<Multi2dCfg<float, 6, 5, 32, 32>>(1),
};
static const Multi2dEntry m_r7[] = {
    multi2d_entry<Multi2dCfg<float, 7, 4, 32, 32>>(1),
};
static const Multi2dEntry m_r8[] = {
    multi2d_entry<Multi2dCfg<float, 8, 3, 32, 32>>(1),
};

const Multi2dEntry *multi2d_configs_f32(int r, int *count)
{
    switch (r) {
    case 1: *count = (int)(sizeof(m_r1) / sizeof(Multi2dEntry)); return m_r1;
    case 2: *count = (int)(sizeof(m_r2) / sizeof(Multi2dEntry)); return m_r2;
    case 3: *count = (int)(sizeof(m_r3) / sizeof(Multi2dEntry)); return m_r3;
    case 4: *count = (int)(sizeof(m_r4) / sizeof(Multi2dEntry)); return m_r4;
    case 5: *count = (int)(sizeof(m_r5) / sizeof(Multi2dEntry)); return m_r5;
    case 6: *count = (int)(sizeof(m_r6) / sizeof(Multi2dEntry)); return m_r6;
    case 7: *count = (int)(sizeof(m_r7) / sizeof(Multi2dEntry)); return m_r7;
    case 8: *count = (int)(sizeof(m_r8) / sizeof(Multi2dEntry)); return m_r8;
    default: *count = 0; return nullptr;
    }
}

// The adjoint.  Microseconds per step, single-step kernel -> these:
//          150 x 128     420 x 300     512^2         1203 x 801    1600^2
//   r = 1  3.13 -> 2.24  3.55 -> 2.24  3.79 -> 2.29   5.62 -> 2.74  13.8 ->  6.6
//   r = 2  3.31 -> 2.54  3.70 -> 2.57  3.93 -> 2.57   6.10 -> 5.25  14.6 -> 11.5
//   r = 3  3.39 -> 3.01  3.83 -> 3.00  4.08 -> 3.01   6.56 (6 steps: 9.03)
//   r = 4  3.52 -> 3.15  4.00 -> 3.15  4.25 -> 3.19   7.00 -> 6.05  15.1 -> 14.1
// For larger radii the single step is as good.
static const Adj2dEntry a_r1[] = {
    adj2d_entry<Multi2dCfg<float, 1, 8, 32, 32>>(0),
};
static const Adj2dEntry a_r2[] = {
    adj2d_entry<Multi2dCfg<float, 2, 8, 32, 32>>(1),
    adj2d_entry<Multi2dCfg<float, 2, 4, 32, 16>>(0),
};
static const Adj2dEntry a_r3[] = {
    adj2d_entry<Multi2dCfg<float, 3, 6, 32, 32>>(1),
};
static const Adj2dEntry a_r4[] = {
    adj2d_entry<Multi2dCfg<float, 4, 6, 32, 32>>(1),
    adj2d_entry<Multi2dCfg<float, 4, 4, 64, 32>>(0),
};

const Adj2dEntry *adj2d_configs_f32(int r, int *count)
{
    switch (r) {
    case 1: *count = (int)(sizeof(a_r1) / sizeof(Adj2dEntry)); return a_r1;
    case 2: *count = (int)(sizeof(a_r2) / sizeof(Adj2dEntry)); return a_r2;
    case 3: *count = (int)(sizeof(a_r3) / sizeof(Adj2dEntry)); return a_r3;
    case 4: *count = (int)(sizeof(a_r4) / sizeof(Adj2dEntry)); return a_r4;
    default: *count = 0; return nullptr;
    }
}

}  // namespace fdw
