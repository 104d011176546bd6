// fd_multi2d_f64.hip -- the several-steps-per-launch kernels of 2-D F64 grids.
//
// Microseconds per step measured on this card, single-step kernel -> these, by grid:
//          256^2         512^2         1203 x 800    1600^2
//   r = 1  3.96 -> 1.67  4.41 -> 1.72  6.85 -> 3.51  14.76 ->  7.24
//   r = 2  4.05 -> 1.69  4.70 -> 2.02  7.65 -> 4.74  15.92 -> 11.16
//   r = 3  4.20 -> 2.09  4.99 -> 2.47  8.22 -> 6.34  16.37 -> 14.75
//   r = 4  4.33 -> 2.35  5.26 -> 2.82  8.78 -> 6.95  16.88 -> 14.66
//   r = 5  4.12 -> 2.51  4.91 -> 2.93  8.50 (3 steps, 32x32:  9.19)
//   r = 6  4.18 -> 2.62  5.08 -> 3.44  8.49 (3 steps, 32x32: 10.84)
//   r = 7  4.29 -> 3.22  5.20 -> 3.77  8.74 (3 steps, 32x32: 12.13)
//   r = 8  4.40 -> 3.84  5.50 -> 4.10  8.90 (2 steps, 32x32: 12.28)
#include "fd_multi2d.h"

namespace fdw {

static const Multi2dEntry m_r1[] = {
    multi2d_entry<Multi2dCfg<double, 1, 8, 32, 32>>(1),
    multi2d_entry<Multi2dCfg<double, 1, 6, 32, 32>>(0),
};
static const Multi2dEntry m_r2[] = {
    multi2d_entry<Multi2dCfg<double, 2, 8, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 2, 6, 32, 32>>(0),
};
static const Multi2dEntry m_r3[] = {
    multi2d_entry<Multi2dCfg<double, 3, 8, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 3, 6, 32, 32>>(1),
    multi2d_entry<Multi2dCfg<double, 3, 4, 32, 32>>(0),
};
static const Multi2dEntry m_r4[] = {
    multi2d_entry<Multi2dCfg<double, 4, 6, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 4, 4, 32, 32>>(0),
};
static const Multi2dEntry m_r5[] = {
    multi2d_entry<Multi2dCfg<double, 5, 4, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 5, 3, 32, 32>>(1),
};
static const Multi2dEntry m_r6[] = {
    multi2d_entry<Multi2dCfg<double, 6, 4, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 6, 3, 32, 32>>(1),
};
static const Multi2dEntry m_r7[] = {
    multi2d_entry<Multi2dCfg<double, 7, 3, 16, 16>>(1),
    multi2d_entry<Multi2dCfg<double, 7, 3, 32, 32>>(1),
};
static const Multi2dEntry m_r8[] = {
    multi2d_entry<Multi2dCfg<double, 8, 2, 32, 32>>(1),
};

const Multi2dEntry *multi2d_configs_f64(int r, int *count)
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
//   r = 1  2.96 -> 1.55  3.87 -> 1.59  4.61 -> 1.70  10.9 ->  5.5  24.3 -> 12.9
//   r = 2  3.07 -> 1.72  4.14 -> 2.28  4.96 -> 2.38  10.9 ->  8.0  26.1 -> 18.3
//   r = 3  3.17 -> 2.25  4.38 -> 2.91  5.37 -> 3.08  11.4 -> 10.3  27.2 -> 23.6
//   r = 4  3.28 -> 2.16  4.56 -> 3.13  5.65 -> 3.28  11.9 -> 11.5  28.6 -> 26.1
//   r = 5  3.35 -> 2.70  4.77 (2 steps, 32x32: 5.40)
// For larger radii the single step is as good.
static const Adj2dEntry a_r1[] = {
    adj2d_entry<Multi2dCfg<double, 1, 8, 32, 32>>(0),
};
static const Adj2dEntry a_r2[] = {
    adj2d_entry<Multi2dCfg<double, 2, 6, 16, 16>>(1),
    adj2d_entry<Multi2dCfg<double, 2, 4, 32, 32>>(0),
};
static const Adj2dEntry a_r3[] = {
    adj2d_entry<Multi2dCfg<double, 3, 4, 16, 16>>(1),
    adj2d_entry<Multi2dCfg<double, 3, 3, 32, 32>>(0),
};
static const Adj2dEntry a_r4[] = {
    adj2d_entry<Multi2dCfg<double, 4, 6, 16, 16>>(1),
    adj2d_entry<Multi2dCfg<double, 4, 3, 32, 32>>(0),
};
static const Adj2dEntry a_r5[] = {
    adj2d_entry<Multi2dCfg<double, 5, 4, 16, 16>>(1),
};

const Adj2dEntry *adj2d_configs_f64(int r, int *count)
{
    switch (r) {
    case 1: *count = (int)(sizeof(a_r1) / sizeof(Adj2dEntry)); return a_r1;
    case 2: *count = (int)(sizeof(a_r2) / sizeof(Adj2dEntry)); return a_r2;
    case 3: *count = (int)(sizeof(a_r3) / sizeof(Adj2dEntry)); return a_r3;
    case 4: *count = (int)(sizeof(a_r4) / sizeof(Adj2dEntry)); return a_r4;
    case 5: *count = (int)(sizeof(a_r5) / sizeof(Adj2dEntry)); return a_r5;
    default: *count = 0; return nullptr;
    }
}

}  // namespace fdw
