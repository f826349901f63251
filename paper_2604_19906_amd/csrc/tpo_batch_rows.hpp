// Launch settings by the size of the batch.  Each kernel family has a setting for large batches (its tuning
// table) and, per type and n, up to six rows before it: a batch whose fields take at most `mib` MiB takes the
// first row that it fits.
//
// Why the size decides: up to a dozen MiB a launch is one round of workgroups and the fewest elements per workgroup
// finish first; up to about 45 MB of fields non-temporal stores (hint 2) lead by 10 .. 25 %, also where the next call reads
// the result; from there to about 250 MB the result of such a call is still in the last-level cache (256 MB) unless its
// stores pass it, so they do not; up to about half a GB the fields are cached in part, and loads that pass the cache too (hint 3)
// and smaller workgroups lead; beyond, the steady stream decides.  fp64 products of n >= 9 and the fp64 halves take longer batches
// of scalar loads (SB = 40 words) on batches of that middle range; they cost 32 .. 50 spilled scalars (70 .. 140
// vector instructions of a wavefront's 290 .. 1770), which the times below include.
//
// The rows come from a sweep of 15 .. 20 settings per n at 19 sizes from 1 MB to 2.5 GB on MI355X and were then chosen, at 29 sizes,
// over four ways to call: the same fields again, three sets in turn, forward then backward of its result (operators: applied
// to their own result) on one set, and that on three sets.  Time over the settings for large and small batches that
// were there before, geometric means over n = 2 .. 16 in each of the four ways, up to 20 MB / 24 .. 130 MB / 145 .. 320 MB / 400 and
// more MB:
//   operator fp64 0.81 .. 0.83 / 0.88 .. 0.89 / 0.91 .. 0.93 / 0.95 .. 0.96    fp32 0.95 .. 0.96 / 0.96 / 0.97 .. 0.98 / 0.97 .. 0.99
//   separable fp64 0.87 / 0.90 .. 0.93 / 0.91 .. 0.96 / 0.95 .. 0.99           fp32 0.95 / 0.92 .. 0.96 / 0.94 .. 0.98 / 0.98 .. 0.99
//   halves fp64 0.89 / 0.90 .. 0.92 / 0.94 .. 0.95 / 0.96 .. 0.97              fp32 0.98 / 0.97 .. 0.98 / 0.98 .. 0.99 / 0.98 .. 0.99
// 51 of 13440 calls lose more than 5 %, up to 1.09: most take less than 10 us (fp32 n = 10 at 8 MB, halves n = 11 at 16 MB, separable n = 5
// at 12 MB), the others are chains of the fp32 separable form at 180 .. 250 MB (1.05 .. 1.08).  At 4 and 8 GB none of 348 loses 4 %.
// Rows that stored past the cache up to 130 .. 250 MB were 10 .. 25 % faster on sets that take turns without being read, at 100 .. 160
// MB (n = 3 separable and halves 30 %; 1 to 5 % over all n and 24 .. 320 MB), but 1.1 .. 1.55 of the time in the chains (fp32 halves n = 9 at 90 .. 180 MB 1.39 .. 1.55, n = 13 1.2 .. 1.3,
// fp64 halves n = 11 at 48 .. 180 MB 1.07 .. 1.27, operator fp64 n = 5 1.1 .. 1.2).
#pragma once

#include <type_traits>

#include "tpo.h"

namespace tpo {

// Added to the words per batch of scalar loads: the matrices are touched once before the first product (warm_scalar_cache); on
// rows that end where a launch comes to about one workgroup per CU (whole MiB: 171 .. 268 workgroups on 256 CUs).  A row of a kernel
// that has no such step is refused below.
constexpr int kWarm = 256;

// Added as well: the kernel's arguments stay in memory (KernelField), in both halves or in one of them (the operator and the separable
// form: both).  Preloaded ones make a launch about 0.12 us longer and every workgroup's first load one scalar load earlier; kernels of few
// instructions (n <= 4) and the fp64 halves of n = 12 .. 15, which the preloaded registers bring spilled scalars, lose by it until a
// launch takes several rounds of workgroups.  Preloaded over held, one matrix and three: halves n = 1 and 2 1.02 .. 1.08 up to the rows' ends, n = 3
// 1.00 .. 1.07, 4 fp32 1.00 .. 1.05, fp64 0.97 .. 1.05 (0.96 .. 1.01 past 1 MB); n = 12 forward 1.02 .. 1.05 (backward 0.91 .. 0.93), 14 0.99 ..
// 1.02 and 1.02 .. 1.06, 15 1.01 .. 1.03 and 1.03 .. 1.07; on the rows behind, up to 24 MiB, 1.01 .. 1.05 with one matrix, 0.97 .. 1.01
// with three, which were no slower held than before there were preloaded arguments; operator n = 1 and 2 1.00 .. 1.08, separable n = 1 1.02;
// halves n = 9 1.02 with one matrix and 1.00 with three from 50 to 500 MB, n = 10 backward 1.00 .. 1.05 from 50 to 150 MB, 1.00 .. 1.01 beyond
// (forward 0.93 .. 1.00).
constexpr int kHeldForward = 512, kHeldBackward = 1024, kHeld = kHeldForward + kHeldBackward;

// sb: words per batch of scalar loads (matrix_product), with or without the flags above; mm: 4x4x1 matrix-core form (halves in fp32).
struct BatchRow { int mib = 0, g = 0, hint = 0, xcd = 0, sb = 0, mm = 0; };
constexpr int kBatchRows = 6;                   // a row with mib = 0 ends the list
struct BatchRows { BatchRow row[TPO_MAX_N + 1][kBatchRows]; };

// Operator, vector-FMA kernels.
template <typename T> struct PencilRows;
template <> struct PencilRows<double> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{3, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{3, 16, 0, 0, 32 + kHeld}, {253, 16, 0, 0, 32}},
        /* 3 */ {{26, 24, 2, 0, 32}, {253, 24, 0, 0, 32}, {1650, 24, 2, 0, 32}},
        /* 4 */ {{50, 8, 2, 0, 32}, {102, 8, 0, 0, 32}, {142, 8, 2, 0, 32}},
        /* 5 */ {{5, 16, 0, 0, 32}, {37, 8, 2, 0, 32}, {874, 8, 0, 0, 32}},
        /* 6 */ {{14, 3, 0, 0, 32}, {50, 3, 2, 0, 32}},
        /* 7 */ {{14, 1, 0, 0, 32}},
        /* 8 */ {{39, 1, 3, 0, 32}, {100, 1, 2, 0, 0}, {288, 1, 0, 0, 0}},
        /* 9 */ {{4, 1, 0, 0, 32 + kWarm}, {14, 1, 0, 0, 32}, {39, 3, 3, 0, 32}, {66, 3, 2, 0, 40}, {145, 3, 0, 0, 40}},
        /* 10 */ {{5, 1, 3, 0, 32 + kWarm}, {85, 1, 3, 0, 32}, {535, 1, 3, 0, 40}},
        /* 11 */ {{7, 1, 0, 0, 32 + kWarm}, {14, 1, 0, 0, 32}, {39, 1, 3, 0, 32}, {165, 2, 2, 0, 40}, {430, 2, 1, 0, 32}, {1650, 2, 3, 0, 32}},
        /* 12 */ {{53, 1, 3, 0, 32}, {68, 3, 3, 0, 32}, {350, 1, 3, 0, 40}},
        /* 13 */ {{12, 1, 0, 0, 32 + kWarm}, {14, 1, 0, 0, 32}, {53, 1, 3, 1, 32}, {535, 1, 2, 0, 40}, {1650, 3, 1, 0, 40}},
        /* 14 */ {{16, 1, 3, 0, 32 + kWarm}, {53, 1, 3, 0, 32}, {535, 1, 3, 0, 40}},
        /* 15 */ {{20, 1, 0, 0, 32 + kWarm}, {53, 1, 3, 1, 32}, {350, 1, 2, 0, 40}, {535, 1, 3, 0, 32}},
        /* 16 */ {{53, 1, 3, 0, 32}, {142, 2, 2, 0, 40}, {535, 1, 3, 1, 40}},
    }};
};
template <> struct PencilRows<float> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{1, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{1, 16, 0, 0, 32 + kHeld}, {9, 16, 0, 0, 32}, {253, 16, 0, 0, 32}},
        /* 3 */ {{14, 32, 0, 0, 32}, {85, 6, 0, 0, 32}, {253, 32, 0, 0, 32}},
        /* 4 */ {{50, 8, 2, 0, 32}, {184, 3, 2, 0, 32}},
        /* 5 */ {{14, 2, 0, 0, 32}, {26, 8, 2, 0, 32}, {253, 8, 0, 0, 32}},
        /* 6 */ {{53, 6, 2, 0, 32}, {102, 3, 3, 0, 32}},
        /* 7 */ {{14, 1, 0, 0, 32}},
    }};
};
// Separable form, vector-FMA kernels.
template <typename T> struct PencilSepRows;
template <> struct PencilSepRows<double> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{1, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{14, 32, 0, 0, 32}, {253, 16, 0, 0, 32}},
        /* 3 */ {{50, 6, 0, 0, 32}, {142, 16, 0, 0, 32}, {253, 24, 0, 0, 32}, {1650, 24, 2, 0, 32}},
        /* 4 */ {{5, 6, 2, 0, 32}, {20, 4, 3, 0, 32}, {37, 8, 2, 0, 32}},
        /* 5 */ {{9, 16, 0, 0, 32}, {31, 2, 2, 0, 32}, {117, 2, 0, 0, 32}, {245, 2, 2, 0, 32}},
        /* 6 */ {{37, 3, 2, 0, 32}, {50, 3, 0, 0, 32}, {535, 3, 2, 0, 32}},
        /* 7 */ {{9, 1, 1, 0, 32}},
        {},
        /* 9 */ {{5, 2, 0, 0, 32 + kWarm}, {37, 3, 2, 0, 32}, {50, 3, 0, 0, 32}, {184, 2, 3, 0, 32}, {350, 3, 3, 0, 32}},
        /* 10 */ {{3, 1, 3, 0, 32 + kWarm}},
        /* 11 */ {{9, 1, 1, 0, 32}, {50, 1, 2, 0, 32}, {85, 1, 0, 0, 32}, {535, 2, 3, 0, 32}},
        /* 12 */ {{31, 1, 3, 0, 32}},
        /* 13 */ {{9, 1, 0, 0, 32}, {245, 1, 3, 0, 32}, {535, 3, 3, 0, 32}},
        /* 14 */ {{245, 1, 3, 0, 32}},
        /* 15 */ {{14, 1, 0, 0, 32}, {535, 1, 3, 0, 32}},
        {},
    }};
};
template <> struct PencilSepRows<float> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{1, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{184, 32, 2, 0, 32}},
        /* 3 */ {{245, 12, 0, 0, 32}},
        /* 4 */ {{5, 2, 2, 0, 32}, {245, 4, 2, 0, 32}},
        /* 5 */ {{9, 2, 0, 0, 32}, {874, 2, 2, 0, 32}},
        /* 6 */ {{245, 6, 2, 0, 32}},
    }};
};
// fp32 kernels with 4x4x1 matrix-core products: operator, separable form.
struct PencilMmRows {
    static constexpr BatchRows rows = {{
        {}, {}, {}, {}, {}, {}, {},
        /* 7 */ {{31, 2, 2, 1}},
        /* 8 */ {{43, 1, 2, 0}},
        /* 9 */ {{14, 3, 0, 0}, {43, 3, 2, 1}, {145, 3, 0, 1}},
        /* 10 */ {{20, 2, 0, 0}, {50, 3, 2, 1}, {145, 3, 0, 1}, {535, 3, 3, 0}},
        /* 11 */ {{14, 2, 0, 0}, {50, 2, 2, 1}},
        /* 12 */ {{5, 1, 0, 0}},
        /* 13 */ {{9, 1, 0, 0}, {20, 3, 0, 0}, {81, 3, 2, 0}},
        /* 14 */ {{14, 1, 0, 0}, {245, 1, 2, 0}},
        /* 15 */ {{14, 1, 0, 0}},
        {},
    }};
};
struct PencilMmSepRows {
    static constexpr BatchRows rows = {{
        {}, {}, {}, {}, {}, {}, {}, {},
        {},
        /* 9 */ {{14, 3, 0, 0}, {37, 3, 2, 0}, {131, 3, 0, 0}, {245, 3, 2, 0}},
        /* 10 */ {{14, 2, 0, 0}, {37, 3, 2, 0}, {102, 4, 0, 0}, {1650, 4, 2, 0}},
        /* 11 */ {{13, 2, 0, 0}, {43, 2, 2, 0}, {102, 2, 0, 0}, {874, 2, 2, 0}},
        /* 12 */ {{2, 1, 0, 0}},
        /* 13 */ {{9, 1, 0, 0}, {14, 3, 0, 0}, {65, 3, 2, 0}, {145, 3, 0, 0}, {350, 3, 2, 0}},
        /* 14 */ {{9, 1, 0, 0}, {53, 1, 2, 0}},
        /* 15 */ {{9, 1, 0, 0}},
        {},
    }};
};
// Transform halves.
template <typename T> struct TransformRows;
template <> struct TransformRows<double> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{14, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{4, 16, 0, 0, 32 + kHeld}},
        /* 3 */ {{2, 32, 0, 0, 32 + kHeld}},
        /* 4 */ {{1, 2, 2, 1, 32 + kHeld}, {14, 2, 2, 1, 32}, {43, 4, 2, 0, 32}},
        /* 5 */ {{5, 16, 0, 0, 32}, {37, 2, 2, 1, 32}},
        {},
        /* 7 */ {{2, 1, 2, 0, 32}, {43, 1, 2, 1, 32}, {1650, 1, 2, 0, 40}},
        /* 8 */ {{53, 1, 2, 0, 32}, {1650, 1, 2, 0, 40}},
        /* 9 */ {{50, 2, 0, 0, 32}, {1024, 1, 0, 0, 40 + kHeld}},
        /* 10 */ {{5, 1, 2, 0, 32}, {184, 1, 2, 0, 40 + kHeldBackward}, {1650, 1, 0, 0, 40 + kHeldBackward}},
        /* 11 */ {{14, 1, 0, 1, 32}, {37, 1, 2, 0, 40}, {1650, 1, 0, 0, 40}},
        /* 12 */ {{6, 1, 2, 0, 40 + kWarm + kHeldForward}, {1650, 1, 2, 0, 40}},
        /* 13 */ {{9, 1, 0, 0, 40 + kWarm}, {24, 1, 2, 0, 40 + kHeldForward}, {53, 1, 2, 0, 40}, {184, 3, 0, 0, 40}, {1650, 2, 0, 0, 40}},
        /* 14 */ {{10, 1, 2, 0, 40 + kWarm + kHeld}, {24, 1, 2, 0, 40 + kHeld}, {57, 1, 2, 0, 40}, {343, 1, 0, 0, 40}, {535, 1, 2, 0, 40}},
        /* 15 */ {{13, 1, 2, 0, 40 + kWarm + kHeld}, {24, 1, 2, 0, 40 + kHeldForward}, {57, 1, 2, 0, 40}, {350, 1, 0, 0, 40}},
        /* 16 */ {{16, 1, 2, 1, 32 + kWarm}, {53, 1, 2, 1, 32}, {1650, 1, 2, 0, 40}},
    }};
};
template <> struct TransformRows<float> {
    static constexpr BatchRows rows = {{
        {},
        /* 1 */ {{14, 64, 2, 1, 32 + kHeld}},
        /* 2 */ {{14, 16, 0, 0, 32 + kHeld}},
        /* 3 */ {{3, 12, 0, 0, 32 + kHeld}, {53, 12, 0, 0, 32}, {245, 24, 0, 0, 32}},
        /* 4 */ {{6, 12, 2, 0, 32 + kHeld}, {14, 12, 2, 0, 32}},
        /* 5 */ {{43, 2, 2, 1, 32}, {245, 2, 0, 1, 32}},
        /* 6 */ {{9, 12, 2, 0, 32}, {26, 6, 2, 0, 32}, {253, 12, 0, 0, 32}, {535, 4, 2, 0, 32}},
        /* 7 */ {{9, 1, 2, 1, 32}, {184, 1, 2, 1, 0, 1}},
        /* 8 */ {{2, 2, 2, 0, 0, 1}, {26, 3, 2, 0, 0, 1}},
        {},
        {},
        /* 11 */ {{26, 1, 2, 1, 0, 1}},
        /* 12 */ {{53, 3, 2, 1, 0, 1}, {640, 3, 2, 0, 0, 1}},
        /* 13 */ {{9, 1, 2, 1, 0, 1}, {14, 3, 0, 1, 0, 1}, {43, 1, 2, 1, 0, 1}, {253, 3, 0, 1, 0, 1}, {1650, 3, 0, 0, 0, 1}},
        /* 14 */ {{43, 1, 2, 0, 0, 1}, {253, 1, 0, 0, 0, 1}, {535, 1, 2, 0, 0, 1}},
        /* 15 */ {{14, 1, 0, 0, 0, 1}, {43, 1, 2, 0, 0, 1}},
        {},
    }};
};

// Convection term, square shapes: SPLIT and all loads first as in convection_pencil_kernel.  Time over the settings there were
// before, 16 sizes from 1 MB to 2.5 GB: fp32 n = 8 0.82 .. 1.0 (matrix-core form), 10 0.73 .. 0.97, 13 0.65 .. 0.96 up to 2.5 GB (1.01 at 55 .. 110 MB; beyond 2.5 GB three units lead by 1 %), 14 0.73 ..
// 0.96, 9, 11, 12 0.75 .. 0.96 up to 8 MB; fp64 n = 6, 9 0.79 .. 0.95 up to 220 MB, 11 0.87 .. 0.94 up to 22 MB, 12 .. 16 0.95 .. 0.98 up to 22 MB and,
// with SB = 40, 0.89 .. 0.98 at 35 .. 220 MB.
struct ConvectionRow { int mib = 0, g = 0, hint = 0, split = 0, loads_first = 0, sb = 0, mm = 0; };
struct ConvectionRows { ConvectionRow row[TPO_MAX_N + 1][kBatchRows]; };
template <typename T> struct SquareConvectionRows;
template <> struct SquareConvectionRows<double> {
    static constexpr ConvectionRows rows = {{
        {}, {}, {}, {}, {}, {},
        /* 6 */ {{22, 1, 2, 0, 0, 32}, {39, 7, 2, 0, 0, 0}, {123, 6, 2, 1, 0, 0}},
        /* 7 */ {{28, 1, 0, 0, 0, 32}, {123, 1, 2, 1, 0, 32}},
        /* 8 */ {{43, 1, 2, 0, 0, 32}, {123, 1, 2, 1, 0, 0}},
        /* 9 */ {{28, 1, 0, 0, 0, 32}, {66, 3, 2, 0, 0, 0}, {253, 2, 2, 1, 0, 32}},
        /* 10 */ {{8, 1, 2, 0, 0, 32 + kWarm}, {43, 1, 2, 0, 0, 32}, {1010, 1, 2, 1, 0, 40}},
        /* 11 */ {{10, 1, 0, 1, 1, 32 + kWarm}, {22, 2, 0, 1, 1, 32}, {1010, 1, 2, 1, 0, 40}},
        /* 12 */ {{14, 1, 2, 0, 0, 32 + kWarm}, {43, 1, 2, 0, 0, 32}, {253, 1, 2, 1, 0, 40}, {1010, 1, 2, 1, 1, 32}},
        /* 13 */ {{18, 1, 2, 0, 0, 32 + kWarm}, {28, 1, 2, 0, 0, 32}, {173, 1, 2, 1, 0, 40}},
        /* 14 */ {{23, 1, 2, 0, 0, 32 + kWarm}, {28, 1, 2, 0, 0, 32}, {253, 1, 2, 1, 0, 40}},
        /* 15 */ {{28, 1, 2, 0, 0, 32 + kWarm}, {123, 1, 2, 1, 0, 40}, {256, 1, 2, 1, 1, 32}},
        /* 16 */ {{28, 1, 2, 0, 0, 32 + kWarm}},
    }};
};
template <> struct SquareConvectionRows<float> {
    static constexpr ConvectionRows rows = {{
        {}, {}, {}, {}, {}, {}, {}, {}, {},
        /* 9 */ {{2, 1, 0, 0, 1, 0, 1}, {90, 3, 0, 0, 1, 0, 1}},
        /* 10 */ {{5, 1, 0, 0, 1, 0, 1}},
        /* 11 */ {{17, 1, 0, 1, 1, 0, 1}, {253, 2, 2, 1, 0, 0, 1}},
        /* 12 */ {{13, 1, 2, 0, 1, 0, 1}},
        /* 13 */ {{17, 1, 0, 0, 1, 0, 1}, {24, 3, 2, 1, 1, 0, 1}, {2600, 1, 2, 1, 1, 0, 1}},
        /* 14 */ {{17, 1, 0, 0, 1, 0, 1}, {123, 1, 2, 0, 1, 0, 1}},
        /* 15 */ {{17, 1, 0, 0, 1, 0, 1}, {64, 1, 2, 1, 0, 0, 1}},
        {},
    }};
};

// Convection term, over-integrated shapes: the first row of a shape that the batch's fields fit (`mib` MiB; 0: every
// batch, the shape then has no other setting).  form 0: convection_rect_kernel, 1 and 2: convection_rect_large_kernel
// without and with compact lanes.  With the scalars in batches (sb) one unit per workgroup leads in fp64 far beyond the
// first round of workgroups; in fp32 it leads while a launch is about one round.  The best of three forms x
// {1, 2, 3, 4, 6, 8} units x sb at 12 sizes from 1 MB to 2.4 GB, buffers in turns, MI355X; time over the settings of
// ConvRectTable and of the utilisation rule: fp64 (6,7) 0.69 .. 0.90 up to 200 MB, 0.91 .. 0.96 beyond, (5,7), (6,9), (7,9)
// 0.78 .. 0.94 and 0.92 .. 0.97, (8,9) 0.79 .. 0.97 (1.01 at 70 MB), (5,8), (6,8), (8,12) 0.88 .. 0.99, (9,14) 0.85 .. 0.91
// (22 MB: 1.07), (8,10), (9,10) 0.91 .. 0.99 at 76 .. 125 MB, (7,8) 0.93 .. 1.0 (92 .. 108 MB without batches of scalars:
// 1.03 .. 1.06 with them; on fields that are used again (7,8) 1.04 .. 1.07 and (9,10) 1.03 .. 1.07 at 115 .. 320 MB); fp32 (12,14) 0.66 .. 0.97, (9,10) 0.80 .. 0.95, (10,12) 0.79 .. 0.97, (11,12), (11,13), (12,13)
// 0.78 .. 0.96 up to 13 MB, (6,7), (5,7), (7,9), (8,12) 0.88 .. 1.0.  The rule's larger workgroups keep the sizes where
// they still are one round and the smaller ones are not: 1.05 .. 1.12 for (9,10) at 17 .. 19 MB, (10,12) at 16 .. 20,
// (11,12), (11,13), (12,13) at 16 .. 24.
struct ConvRectFirst { int nv, nq, mib, g, form, sb; };
template <typename T> struct ConvRectFirstTable;
template <> struct ConvRectFirstTable<double> {
    static constexpr ConvRectFirst row[] = {
        {5, 6, 16, 1, 0, 32},   {5, 7, 0, 1, 0, 32},    {5, 8, 190, 1, 0, 32},  {5, 8, 0, 4, 1, 32},
        {6, 7, 0, 1, 0, 32},    {6, 8, 2400, 1, 1, 32}, {6, 9, 0, 1, 0, 32},    {7, 8, 78, 1, 0, 32},
        {7, 8, 104, 1, 0, 0},   {7, 8, 400, 1, 0, 32},  {7, 9, 2400, 1, 0, 32}, {8, 9, 0, 1, 0, 32},
        {8, 10, 70, 1, 1, 32},  {8, 10, 122, 2, 2, 32}, {9, 10, 66, 1, 1, 32},  {9, 10, 122, 2, 0, 32},
        {8, 12, 12, 1, 0, 32 + kWarm}, {8, 12, 600, 1, 0, 32}, {9, 14, 13, 1, 0, 32 + kWarm},
    };
};
template <> struct ConvRectFirstTable<float> {
    static constexpr ConvRectFirst row[] = {
        {5, 6, 3, 1, 0, 0},    {5, 7, 0, 4, 0, 0},    {5, 8, 7, 1, 0, 0},    {6, 7, 7, 1, 0, 0},     {6, 8, 20, 1, 0, 0},
        {6, 9, 48, 1, 0, 0},   {7, 9, 50, 1, 0, 0},   {8, 10, 13, 1, 0, 0},  {8, 12, 5, 1, 0, 0},    {9, 10, 15, 2, 1, 0},
        {9, 10, 18, 5, 0, 0},  {9, 10, 31, 2, 1, 0},  {9, 14, 7, 1, 0, 0},   {10, 12, 13, 1, 0, 0},  {10, 12, 20, 3, 0, 0},
        {10, 12, 240, 2, 2, 0}, {11, 12, 13, 1, 0, 0}, {11, 13, 13, 1, 0, 0}, {12, 13, 13, 1, 0, 0}, {12, 14, 0, 1, 0, 0},
    };
};
// The k-th row of a shape ({}: it has no more).
template <typename T>
constexpr ConvRectFirst convection_rect_first(int nv, int nq, int k)
{
    for (const ConvRectFirst &r : ConvRectFirstTable<T>::row)
        if (r.nv == nv && r.nq == nq && k-- == 0) return r;
    return {};
}
// MiB of the last row of a shape (0: no rows).
template <typename T>
constexpr int convection_rect_first_end(int nv, int nq)
{
    int end = 0;
    for (int k = 0; convection_rect_first<T>(nv, nq, k).g != 0; ++k) end = convection_rect_first<T>(nv, nq, k).mib;
    return end;
}
// Whether a batch fits row r of its shape.
template <typename T>
constexpr bool convection_rect_fits(const ConvRectFirst &r, long long num_elems)
{
    const long long per = (10LL * r.nq * r.nq * r.nq + 3LL * r.nv * r.nv * r.nv) * (long long)sizeof(T);
    return r.g != 0 && (r.mib == 0 || num_elems <= ((long long)r.mib << 20) / per);
}

// f(integral_constant<int, K>) for the first row K of n that a batch of num_elems elements (bytes_per_elem of
// fields each) fits; f returns its result.  False: past the rows.
template <const auto &ROWS, int N, int K = 0, typename F>
inline bool for_batch_row(long long num_elems, long long bytes_per_elem, F &&f)
{
    if constexpr (K < kBatchRows) {
        if constexpr (ROWS.row[N][K].mib > 0) {
            if (num_elems <= ((long long)ROWS.row[N][K].mib << 20) / bytes_per_elem) {
                f(std::integral_constant<int, K>{});
                return true;
            }
            return for_batch_row<ROWS, N, K + 1>(num_elems, bytes_per_elem, f);
        }
    }
    return false;
}
template <const auto &ROWS, int N, int K = 0, typename F>
inline void for_each_batch_row(F &&f)
{
    if constexpr (K < kBatchRows) {
        if constexpr (ROWS.row[N][K].mib > 0) {
            f(std::integral_constant<int, K>{});
            for_each_batch_row<ROWS, N, K + 1>(f);
        }
    }
}

// The first row that a batch fits is taken, so a row that is not larger than the one before it would never be.
template <typename ROWS>
constexpr bool batch_rows_in_order(const ROWS &rows)
{
    for (const auto &list : rows.row) {
        int before = 0;
        bool ended = false;
        for (const auto &r : list) {
            if (r.mib > 0 && (ended || r.mib <= before)) return false;
            if (r.mib > 0) before = r.mib;
            else ended = true;
        }
    }
    return true;
}
template <typename T>
constexpr bool convection_rect_first_in_order()
{
    for (const ConvRectFirst &r : ConvRectFirstTable<T>::row) {
        int before = 0;
        for (int k = 0; convection_rect_first<T>(r.nv, r.nq, k).g != 0; ++k) {
            const ConvRectFirst now = convection_rect_first<T>(r.nv, r.nq, k);
            if (now.mib != 0 ? now.mib <= before : convection_rect_first<T>(r.nv, r.nq, k + 1).g != 0) return false;
            before = now.mib;
        }
    }
    return true;
}
static_assert(batch_rows_in_order(PencilRows<double>::rows) && batch_rows_in_order(PencilRows<float>::rows));
static_assert(batch_rows_in_order(PencilSepRows<double>::rows) && batch_rows_in_order(PencilSepRows<float>::rows));
static_assert(batch_rows_in_order(PencilMmRows::rows) && batch_rows_in_order(PencilMmSepRows::rows));
static_assert(batch_rows_in_order(TransformRows<double>::rows) && batch_rows_in_order(TransformRows<float>::rows));
static_assert(batch_rows_in_order(SquareConvectionRows<double>::rows) && batch_rows_in_order(SquareConvectionRows<float>::rows));
static_assert(convection_rect_first_in_order<double>() && convection_rect_first_in_order<float>());

// The flags stand only where a kernel takes them: not in the 4x4x1 forms (mm, or all rows of a family), kWarm not in the over-integrated
// forms 1 and 2, kHeld in no convection kernel.
template <typename ROWS>
constexpr bool flags_are_taken(const ROWS &rows, int flags = kWarm | kHeld)
{
    for (const auto &list : rows.row)
        for (const auto &r : list)
            if ((r.sb & ~255 & ~(r.mm != 0 ? 0 : flags)) != 0) return false;
    return true;
}
template <typename T>
constexpr bool convection_rect_flags_are_taken()
{
    for (const ConvRectFirst &r : ConvRectFirstTable<T>::row)
        if ((r.sb & ~255 & ~(r.form != 0 ? 0 : kWarm)) != 0) return false;
    return true;
}
static_assert(flags_are_taken(PencilRows<double>::rows) && flags_are_taken(PencilRows<float>::rows));
static_assert(flags_are_taken(PencilSepRows<double>::rows) && flags_are_taken(PencilSepRows<float>::rows));
static_assert(flags_are_taken(PencilMmRows::rows, 0) && flags_are_taken(PencilMmSepRows::rows, 0));
static_assert(flags_are_taken(TransformRows<double>::rows) && flags_are_taken(TransformRows<float>::rows));
static_assert(flags_are_taken(SquareConvectionRows<double>::rows, kWarm) && flags_are_taken(SquareConvectionRows<float>::rows, kWarm));
static_assert(convection_rect_flags_are_taken<double>() && convection_rect_flags_are_taken<float>());

// MiB of the last row of n (0: no rows): a setting for smaller batches than that is never taken.
template <typename ROWS>
constexpr int batch_rows_end(const ROWS &rows, int n)
{
    int end = 0;
    for (const auto &r : rows.row[n])
        if (r.mib > 0) end = r.mib;
    return end;
}

// Names a launcher in a call of f(Use<launcher>{}).
template <typename L> struct Use { using type = L; };

// The row as a tuning of the vector-FMA operator kernels, of the 4x4x1 kernels and of the halves.
template <const BatchRows &ROWS, int N, int K>
struct BatchTune {
    static constexpr BatchRow R = ROWS.row[N][K];
    static constexpr int G = R.g, HINT = R.hint, SB = R.sb;
    static constexpr bool DDIRECT = true, XCD = R.xcd != 0, MM = R.mm != 0;
    static constexpr size_t LDS_MIN = 0;
};
template <const ConvectionRows &ROWS, int N, int K>
struct ConvectionBatchTune {
    static constexpr ConvectionRow R = ROWS.row[N][K];
    static constexpr int G = R.g, HINT = R.hint, SB = R.sb;
    static constexpr bool SPLIT = R.split != 0, LOADS_FIRST = R.loads_first != 0, MM = R.mm != 0;
};

}  // namespace tpo
