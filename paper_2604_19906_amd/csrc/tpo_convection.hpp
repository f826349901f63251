// Volume integral of the convective flux (Eq. 1 of the paper).  Per component c and element e:
// the sum over the three flux directions d of a tensor-product operator on the metric-weighted
// flux of that direction, the differentiation matrix D along direction d and the interpolation
// matrix I along the other two.  Cube axes are called l (fastest), m, n below; direction 0 is l:
//
//   F[c,e] = (I (x) I (x) D) (M.P0) + (I (x) D (x) I) (M.P1) + (D (x) I (x) I) (M.P2),
//
// the three factors of a Kronecker product acting on axes n, m, l in that order.  Written here
// for square D, I (as many nodes as quadrature points per direction).  Sum-factorised and with
// the three terms merged as early as the algebra allows, eight mode products per (c, e) instead
// of nine:
//   axis l:  a0 = D (M.P0),  a1 = I (M.P1),  a2 = I (M.P2)
//   axis m:  b01 = I a0 + D a1,  b2 = I a2
//   axis n:  F = I b01 + D b2
// One lane owns one pencil (as in tpo_pencil.hpp), the matrix entries arrive in SGPRs, the
// intermediate cubes live in LDS (three, then two).  A workgroup handles G units; a unit is
// one (element, component) pair, numbered 3*e + c so that the three components of an element,
// which share M_e, run next to each other and find it in cache.  Loads: each lane reads the n
// consecutive words of M_e and of the three P cubes that belong to its (n,m) pencil; stores
// are coalesced (lanes consecutive along (j,i)).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tpo_batch_rows.hpp"
#include "tpo_pencil.hpp"
#include "tpo_pencil_mm.hpp"

namespace tpo {

// Workgroups are dealt round-robin to the 8 accelerator dies, each with its own L2.  With
// SAME_DIE the batches of units are renumbered so that three consecutive batches run on ONE die
// one after the other: block b (die b & 7, slot b >> 3) takes batch ((slot / 3) * 8 + die) * 3 +
// slot % 3.  The three components of an element then find M_e in that die's L2 instead of
// fetching it from HBM three times (measured: 12.1 -> 10.1 cubes read per element at n = 11).
// The grid must be convection_grid<SAME_DIE>(number of batches); blocks past the end exit.
template <bool SAME_DIE>
__host__ __device__ inline long long convection_grid(long long nbatch)
{
    return SAME_DIE ? 24 * ((nbatch + 23) / 24) : nbatch;
}
template <bool SAME_DIE>
__device__ __forceinline__ long long convection_batch()
{
    if constexpr (SAME_DIE) {
        const long long die = blockIdx.x & 7, slot = blockIdx.x >> 3;
        return ((slot / 3) * 8 + die) * 3 + slot % 3;
    } else {
        return blockIdx.x;
    }
}

// SPLIT (two LDS cubes per unit, two more barriers) pays once three cubes of a unit pass about
// 20 KB (fp64 n = 11: 0.825 against 0.87 ms; fp32 n = 13: 1.73 against 1.82 ms; fp64 n = 8 with
// 13 KB: 0.61 against 0.60 ms).
template <typename T, int N>
constexpr bool convection_split()
{
    return 3 * PencilShape<T, N, 1>::CUBE * sizeof(T) > 20 * 1024;
}
// Units per workgroup: best lane utilisation with at most 512 threads and 56 KB of LDS.
template <typename T, int N>
constexpr int convection_group()
{
    const long cubes = convection_split<T, N>() ? 2 : 3;
    int best = 1;
    long best_num = 0, best_den = 1;
    for (int g = 1; g <= 64; ++g) {
        const int p = g * N * N;
        const int nt = ((p + 63) / 64) * 64;
        const long lds = cubes * g * PencilShape<T, N, 1>::CUBE * (long)sizeof(T);
        if (g > 1 && (nt > 512 || lds > 56 * 1024)) break;
        if ((long)p * best_den > best_num * nt) {
            best = g;
            best_num = p;
            best_den = nt;
        }
    }
    return best;
}

// Words per batch of scalar loads in the vector-FMA products (matrix_product): batches in fp64 for n >= 7 and
// from 77 entries on where n_q != n_v (not for n = 9, which they take from 64 to 76 registers and from eight to six
// wavefronts per SIMD): they give 0.73 .. 0.95 of the time at 0.5 MB and 0.80 .. 1.00 at 2.5 GB ((8,10) and (9,10) lose 4 to 6 % at
// 100 .. 250 MB, (10,15) 3 to 7 % at 28 .. 48 MB).  With the units of the large settings smaller matrices lose as much as
// they gain ((6,6) up to 1.10, (7,8) and (8,9) 1.05 at 100 .. 320 MB); the rows by batch size, mostly of one unit, say for themselves
// (fp64 (5,7), (6,7), (7,8), (8,9) gain).  In fp32 the fences cost more than the waits (up to 1.12 on n_q >= 9 from 60 MB on).
template <typename T, int NV, int NQ = NV>
constexpr int convection_batch_words()
{
    if (sizeof(T) == 4) return 0;
    if (NV == NQ) return NV >= 7 && NV != 9 ? kScalarBatch : 0;
    return NV * NQ >= 77 ? kScalarBatch : 0;
}

// HINT bit 0 / 1: non-temporal loads / stores.  XCD: the SAME_DIE renumbering above.
// SPLIT: the third term's axis-l and axis-m products run after the first two terms have been
// merged, in the LDS cube that merge frees: two cubes per unit instead of three (more
// workgroups per CU) for two more barriers.
// LOADS_FIRST: see the loads.
template <typename T, int N, int G, int HINT, bool XCD, bool SPLIT, bool LOADS_FIRST, int SB>
__global__ void __launch_bounds__((PencilShape<T, N, G>::NT))
convection_pencil_kernel(const T *__restrict__ Pq, const T *__restrict__ Mq, const T *Dm_,
                         const T *Im_, T *__restrict__ F, long long num_elems)
{
    using Sh = PencilShape<T, N, G>;
    constexpr int P = Sh::P, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *lds = reinterpret_cast<T *>(tpo_lds);

    const TPO_CONSTANT T *Dm = (const TPO_CONSTANT T *)Dm_;
    const TPO_CONSTANT T *Im = (const TPO_CONSTANT T *)Im_;

    const int tid = threadIdx.x;
    const int g = tid / P;
    const int p = tid - g * P;
    const int hi = p / N;
    const int lo = p - hi * N;
    const long long units = 3 * num_elems;
    const long long nbatch = (units + G - 1) / G;
    const long long batch = convection_batch<XCD>();
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const long long unit = batch * G + g;
    const bool on = (tid < G * P) && (unit < units);
    const long long e = on ? unit / 3 : 0;
    const int c = on ? (int)(unit - 3 * e) : 0;
    constexpr size_t QC = (size_t)N * N * N;

    T *c0 = lds + (size_t)(g < G ? g : 0) * (SPLIT ? 2 : 3) * CUBE;
    T *c1 = c0 + CUBE;
    T *c2 = SPLIT ? c1 : c1 + CUBE;

    T x[N], y[N], z[N];
    T x2[N];                     // SPLIT: M.P2 of the lane's (n,m) pencil, kept for later
    static_assert(SPLIT || !LOADS_FIRST, "the third load waits where SPLIT keeps the third term");

    // axis l: lane (n,m) = (hi,lo) owns the n consecutive words [e][n][m][0..N-1] of M and P
    if (on) {
        T mq[N];
        load_words<(HINT & 1) != 0>(Mq + (size_t)e * QC + (size_t)(p * N), mq);
        if constexpr (LOADS_FIRST) {
            // All four long loads go out before anything waits for one of them (the fences keep the third
            // one, whose use is far below, from sinking).  It takes 19 .. 31 registers more per lane.
            T x01[2][N];
            auto load_p = [&](int dir, T (&w)[N]) {
                const size_t cube = ((size_t)(c * 3 + dir) * (size_t)num_elems + (size_t)e) * QC;
                load_words<(HINT & 1) != 0>(Pq + cube + (size_t)(p * N), w);
            };
            load_p(0, x01[0]);
            load_p(1, x01[1]);
            load_p(2, x2);
#pragma unroll
            for (int dir = 0; dir < 3; ++dir) {
                T (&w)[N] = dir < 2 ? x01[dir] : x2;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int l = 0; l < N; ++l) w[l] *= mq[l];
                if (dir < 2) {
                    if (dir == 0) warm_scalar_cache<SB, N * N>(Dm, Im);
                    mode_product<T, N, false, SB>(dir == 0 ? Dm : Im, w, y);
                    T *dst = dir == 0 ? c0 : c1;
#pragma unroll
                    for (int i = 0; i < N; ++i) dst[hi * PA + lo * PB + i] = y[i];
                }
            }
        } else {
#pragma unroll
            for (int dir = 0; dir < 3; ++dir) {
                const size_t cube = ((size_t)(c * 3 + dir) * (size_t)num_elems + (size_t)e) * QC;
                load_words<(HINT & 1) != 0>(Pq + cube + (size_t)(p * N), x);
#pragma unroll
                for (int l = 0; l < N; ++l) x[l] *= mq[l];
                if (SPLIT && dir == 2) {
#pragma unroll
                    for (int l = 0; l < N; ++l) x2[l] = x[l];
                } else {
                    if (dir == 0) warm_scalar_cache<SB, N * N>(Dm, Im);
                    mode_product<T, N, false, SB>(dir == 0 ? Dm : Im, x, y);
                    T *dst = dir == 0 ? c0 : (dir == 1 ? c1 : c2);
#pragma unroll
                    for (int i = 0; i < N; ++i) dst[hi * PA + lo * PB + i] = y[i];
                }
            }
        }
    }
    __syncthreads();

    // axis m: lane (n,i) = (hi,lo)
    if (on) {
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = c0[hi * PA + m * PB + lo];
        mode_product<T, N, false, SB>(Im, x, y);
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = c1[hi * PA + m * PB + lo];
        mode_product<T, N, false, SB>(Dm, x, z);
#pragma unroll
        for (int j = 0; j < N; ++j) c0[hi * PA + j * PB + lo] = y[j] + z[j];
    }
    if constexpr (SPLIT) {
        __syncthreads();                      // every lane has read its pencils of cube 1
        if (on) {                             // axis l of the third term: lane (n,m)
            mode_product<T, N, false, SB>(Im, x2, y);
#pragma unroll
            for (int i = 0; i < N; ++i) c2[hi * PA + lo * PB + i] = y[i];
        }
        __syncthreads();
    }
    if (on) {
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = c2[hi * PA + m * PB + lo];
        mode_product<T, N, false, SB>(Im, x, y);
#pragma unroll
        for (int j = 0; j < N; ++j) c2[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // axis n: lane (j,i) = (hi,lo); stores are consecutive over lanes
    if (on) {
#pragma unroll
        for (int n = 0; n < N; ++n) x[n] = c0[n * PA + hi * PB + lo];
        mode_product<T, N, false, SB>(Im, x, y);
#pragma unroll
        for (int n = 0; n < N; ++n) x[n] = c2[n * PA + hi * PB + lo];
        mode_product<T, N, false, SB>(Dm, x, z);
        const size_t out = ((size_t)c * (size_t)num_elems + (size_t)e) * QC;
#pragma unroll
        for (int k = 0; k < N; ++k) gstore<(HINT & 2) != 0>(F + out + (size_t)(k * P + p), y[k] + z[k]);
    }
}

// fp32 form with the mode products issued as 4x4x1 matrix-core outer products
// (tpo_pencil_mm.hpp): same data movement; the coefficient tables of D and I (both used
// untransposed) stay in registers for the whole kernel.  The matrix instructions run on whole
// wavefronts, outside the `on` branches (their broadcast coefficients come from active lanes
// only).
template <int N, int G, int HINT, bool XCD, bool SPLIT, bool LOADS_FIRST>
__global__ void __launch_bounds__((PencilShape<float, N, G>::NT))
convection_mm_kernel(const float *__restrict__ Pq, const float *__restrict__ Mq,
                     const float *__restrict__ Dm, const float *__restrict__ Im,
                     float *__restrict__ F, long long num_elems)
{
    using Sh = PencilShape<float, N, G>;
    using MS = MmShape<N>;
    constexpr int P = Sh::P, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE, NY = MS::NY;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    float *lds = reinterpret_cast<float *>(tpo_lds);

    const TPO_CONSTANT float *Dc = (const TPO_CONSTANT float *)Dm;
    const TPO_CONSTANT float *Ic = (const TPO_CONSTANT float *)Im;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const long long units = 3 * num_elems;
    const long long nbatch = (units + G - 1) / G;
    const long long batch = convection_batch<XCD>();
    if (XCD && batch >= nbatch) return;
    // Lanes without a pencil never write; with LOADS_FIRST they read pencil 0 of the workgroup's first
    // unit (there is one), else the global loads leave them out.
    const int g_ = tid / P;
    const bool on = (tid < G * P) && (batch * G + g_ < units);
    const int g = on || !LOADS_FIRST ? g_ : 0;
    const int p = on || !LOADS_FIRST ? tid - g_ * P : 0;
    const int hi = p / N;
    const int lo = p - hi * N;
    const long long unit = batch * G + g;
    const long long e = on || LOADS_FIRST ? unit / 3 : 0;
    const int c = on || LOADS_FIRST ? (int)(unit - 3 * e) : 0;
    constexpr size_t QC = (size_t)N * N * N;

    float *c0 = lds + (size_t)(g < G ? g : 0) * (SPLIT ? 2 : 3) * CUBE;   // p < P: inside the cube
    float *c1 = c0 + CUBE;
    float *c2 = SPLIT ? c1 : c1 + CUBE;

    float tab_d[MS::NTAB], tab_i[MS::NTAB];
    float x[N], y[NY], z[NY], mq[N];
    float xd[3][N];              // M.P of the lane's (n,m) pencil; SPLIT keeps the third for later
    auto load_tables = [&]() {
#pragma unroll
        for (int t = 0; t < MS::NTAB; ++t) {
            tab_d[t] = mm_coef<N>(Dm, false, t, lane);
            tab_i[t] = mm_coef<N>(Im, false, t, lane);
        }
    };
    // LOADS_FIRST: all four long loads go out before the tables, and the tables before anything waits for one of them.  (Without the
    // second fence the products with M_e move up between the loads of the tables, whose last words then are a round trip of their own:
    // n = 10, 14 and 15 1.03 .. 1.09 of the time at 30 MB .. 1 GB; up to 16 MB n = 11 and 13 .. 16 0.98 .. 1.00.)  From n = 13
    // on on large batches; below, the registers they hold cost more than the wait there, but less with the few units per workgroup of
    // the rows for small batches (n = 9 .. 12) and at n = 10.  At 3 GB, first against last:
    // n = 13 617 / 651 us, 14 726 / 768, 16 606 / 633; n = 12 614 / 588, 11 636 / 565, 9 605 / 542.  On smaller
    // batches, time over that with densely packed tables and the loads last, first / last: 8 MB n = 13 1.01 /
    // 1.03, 14 0.96 / 1.00, 15 0.99 / 1.00, 16 0.95 / 1.00; 150 MB 1.03 / 1.01, 1.02 / 0.96, 1.02 / 1.01, 0.99 / 1.00; 600 MB 0.94 /
    // 1.02, 0.96 / 0.98, 0.97 / 0.97, 0.97 / 0.96.
    // The branch on `on` is what keeps the compiler from moving the loads of the others up.
    auto load_field = [&](const float *f, float (&w)[N]) {
        if (LOADS_FIRST || on) {
            load_words<(HINT & 1) != 0>(f + (size_t)e * QC + (size_t)(p * N), w);
        } else {
#pragma unroll
            for (int l = 0; l < N; ++l) w[l] = 0.0f;
        }
    };
    auto load_p = [&](int dir) { load_field(Pq + (size_t)(c * 3 + dir) * (size_t)num_elems * QC, xd[dir]); };

    // axis l: lane (n,m) = (hi,lo)
    if constexpr (!LOADS_FIRST) load_tables();
    load_field(Mq, mq);
    if constexpr (LOADS_FIRST) {
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) load_p(dir);
        __builtin_amdgcn_sched_barrier(0);
        load_tables();
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
        if constexpr (!LOADS_FIRST) load_p(dir);
#pragma unroll
        for (int l = 0; l < N; ++l) xd[dir][l] *= mq[l];
        if (!(SPLIT && dir == 2)) {
            if (dir == 0) mode_product_mm<N, false>(tab_d, Dc, xd[dir], y);
            else mode_product_mm<N, false>(tab_i, Ic, xd[dir], y);
            float *dst = dir == 0 ? c0 : (dir == 1 ? c1 : c2);
            if (on) {
#pragma unroll
                for (int i = 0; i < N; ++i) dst[hi * PA + lo * PB + i] = y[i];
            }
        }
    }
    __syncthreads();

    // axis m: lane (n,i) = (hi,lo)
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = c0[hi * PA + m * PB + lo];
    mode_product_mm<N, false>(tab_i, Ic, x, y);
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = c1[hi * PA + m * PB + lo];
    mode_product_mm<N, false>(tab_d, Dc, x, z);
    if (on) {
#pragma unroll
        for (int j = 0; j < N; ++j) c0[hi * PA + j * PB + lo] = y[j] + z[j];
    }
    if constexpr (SPLIT) {
        __syncthreads();                      // every lane has read its pencils of cube 1
        mode_product_mm<N, false>(tab_i, Ic, xd[2], y);       // axis l of the third term: lane (n,m)
        if (on) {
#pragma unroll
            for (int i = 0; i < N; ++i) c2[hi * PA + lo * PB + i] = y[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = c2[hi * PA + m * PB + lo];
    mode_product_mm<N, false>(tab_i, Ic, x, y);
    if (on) {
#pragma unroll
        for (int j = 0; j < N; ++j) c2[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // axis n: lane (j,i) = (hi,lo)
#pragma unroll
    for (int n = 0; n < N; ++n) x[n] = c0[n * PA + hi * PB + lo];
    mode_product_mm<N, false>(tab_i, Ic, x, y);
#pragma unroll
    for (int n = 0; n < N; ++n) x[n] = c2[n * PA + hi * PB + lo];
    mode_product_mm<N, false>(tab_d, Dc, x, z);
    if (on) {
        const size_t out = ((size_t)c * (size_t)num_elems + (size_t)e) * QC;
#pragma unroll
        for (int k = 0; k < N; ++k) gstore<(HINT & 2) != 0>(F + out + (size_t)(k * P + p), y[k] + z[k]);
    }
}

// ---- rectangular form: n_q quadrature points and n_v nodes per direction, n_q != n_v ----------
// Same scheme (vector-FMA pencils, two LDS cubes per unit, the third term's first two products
// after the merge of the first two terms); the lane sets differ per axis: n_q*n_q pencils along
// l, n_q*n_v along m, n_v*n_v along n.

template <typename T, int NV, int NQ, int G>
struct ConvRectShape {
    static constexpr int NB = NQ > NV ? NQ : NV;
    static constexpr int L = NB * NB;                          // lanes per unit
    static constexpr int NT = ((G * L + 63) / 64) * 64;
    static constexpr int PB = (NV & 1) ? NV : NV + 1;          // row pitch (fastest axis: i)
    static constexpr int PA = ((NB * PB) & 1) ? NB * PB : NB * PB + 1;
    static constexpr int CUBE = NQ * PA;
    static constexpr size_t LDS_BYTES = (size_t)2 * G * CUBE * sizeof(T);
};

template <typename T, int NV, int NQ, int G, int HINT, bool XCD, int SB>
__global__ void __launch_bounds__((ConvRectShape<T, NV, NQ, G>::NT))
convection_rect_kernel(const T *__restrict__ Pq, const T *__restrict__ Mq, const T *Dm_,
                       const T *Im_, T *__restrict__ F, long long num_elems)
{
    using Sh = ConvRectShape<T, NV, NQ, G>;
    constexpr int L = Sh::L, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *lds = reinterpret_cast<T *>(tpo_lds);

    const TPO_CONSTANT T *Dm = (const TPO_CONSTANT T *)Dm_;
    const TPO_CONSTANT T *Im = (const TPO_CONSTANT T *)Im_;

    const int tid = threadIdx.x;
    const int g = tid / L;
    const int p = tid - g * L;
    const long long units = 3 * num_elems;
    const long long nbatch = (units + G - 1) / G;
    const long long batch = convection_batch<XCD>();
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const long long unit = batch * G + g;
    const bool live = (tid < G * L) && (unit < units);
    const long long e = live ? unit / 3 : 0;
    const int c = live ? (int)(unit - 3 * e) : 0;
    constexpr size_t QC = (size_t)NQ * NQ * NQ, VC = (size_t)NV * NV * NV;
    const bool on_l = live && p < NQ * NQ;              // pencils along l: lane (n,m)
    const bool on_m = live && p < NQ * NV;              // pencils along m: lane (n,i)
    const bool on_n = live && p < NV * NV;              // pencils along n: lane (j,i)

    T *c0 = lds + (size_t)(g < G ? g : 0) * 2 * CUBE;
    T *c1 = c0 + CUBE;

    T xq[NQ], x2[NQ], yv[NV], zv[NV];

    // axis l: lane (n,m) owns the NQ consecutive words [e][n][m][0..NQ-1] of M and P
    if (on_l) {
        const int nn = p / NQ, mm = p - nn * NQ;
        T mq[NQ];
        load_words<(HINT & 1) != 0>(Mq + (size_t)e * QC + (size_t)(p * NQ), mq);
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
            const size_t cube = ((size_t)(c * 3 + dir) * (size_t)num_elems + (size_t)e) * QC;
            load_words<(HINT & 1) != 0>(Pq + cube + (size_t)(p * NQ), xq);
#pragma unroll
            for (int l = 0; l < NQ; ++l) xq[l] *= mq[l];
            if (dir == 2) {
#pragma unroll
                for (int l = 0; l < NQ; ++l) x2[l] = xq[l];
            } else {
                if (dir == 0) warm_scalar_cache<SB, NV * NQ>(Dm, Im);
                matrix_product<T, NV, NQ, false, SB>(dir == 0 ? Dm : Im, xq, yv);
                T *dst = dir == 0 ? c0 : c1;
#pragma unroll
                for (int i = 0; i < NV; ++i) dst[nn * PA + mm * PB + i] = yv[i];
            }
        }
    }
    __syncthreads();

    // axis m, first two terms merged: lane (n,i)
    const int bn = p / NV, bi = p - bn * NV;
    if (on_m) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c0[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c1[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Dm, xq, zv);
    }
    __syncthreads();                                    // every pencil of cubes 0 and 1 has been read
    if (on_m) {
#pragma unroll
        for (int j = 0; j < NV; ++j) c0[bn * PA + j * PB + bi] = yv[j] + zv[j];
    }
    // axis l of the third term, into the freed cube 1: lane (n,m)
    if (on_l) {
        const int nn = p / NQ, mm = p - nn * NQ;
        matrix_product<T, NV, NQ, false, SB>(Im, x2, yv);
#pragma unroll
        for (int i = 0; i < NV; ++i) c1[nn * PA + mm * PB + i] = yv[i];
    }
    __syncthreads();
    // axis m of the third term: lane (n,i)
    if (on_m) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c1[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int j = 0; j < NV; ++j) c1[bn * PA + j * PB + bi] = yv[j];   // the lane's own pencil
    }
    __syncthreads();

    // axis n: lane (j,i); stores are consecutive over lanes
    if (on_n) {
        const int jj = p / NV, ii = p - jj * NV;
#pragma unroll
        for (int n = 0; n < NQ; ++n) xq[n] = c0[n * PA + jj * PB + ii];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int n = 0; n < NQ; ++n) xq[n] = c1[n * PA + jj * PB + ii];
        matrix_product<T, NV, NQ, false, SB>(Dm, xq, zv);
        const size_t out = ((size_t)c * (size_t)num_elems + (size_t)e) * VC;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            gstore<(HINT & 2) != 0>(F + out + (size_t)(k * NV * NV + p), yv[k] + zv[k]);
    }
}

// The same phases for batches that pass the last-level cache.  Every phase works out its unit and
// addresses where it uses them instead of once for all lanes and phases: fp64 (8,12) with compact
// lanes then takes 84 instead of 97 registers (five wavefronts per SIMD instead of four), and the
// loads leave earlier (fp64 (8,10), one unit, same occupancy: 441 against 488 us on 2.5 GB).  On
// batches that stay in the cache the form above is up to 8 % ahead (fp64 (9,11), fp32 (11,12)).
// COMPACT: the lanes of the axis-m and axis-n phases are numbered through over the workgroup's units
// with that phase's own pencil count, so that these phases (fewer pencils) leave whole wavefronts
// idle; otherwise a unit keeps its NQ*NQ lanes throughout and part of every wavefront idles, which
// spreads the stores over more wavefronts.
template <typename T, int NV, int NQ, int G, int HINT, bool XCD, bool COMPACT, int SB>
__global__ void __launch_bounds__((ConvRectShape<T, NV, NQ, G>::NT))
convection_rect_large_kernel(const T *__restrict__ Pq, const T *__restrict__ Mq, const T *Dm_,
                             const T *Im_, T *__restrict__ F, long long num_elems)
{
    using Sh = ConvRectShape<T, NV, NQ, G>;
    constexpr int PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *lds = reinterpret_cast<T *>(tpo_lds);

    const TPO_CONSTANT T *Dm = (const TPO_CONSTANT T *)Dm_;
    const TPO_CONSTANT T *Im = (const TPO_CONSTANT T *)Im_;

    const int tid = threadIdx.x;
    const long long units = 3 * num_elems;
    const long long nbatch = (units + G - 1) / G;
    const long long batch = convection_batch<XCD>();
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const long long left = units - batch * G;
    const int here = left < G ? (int)left : G;          // units of this workgroup
    constexpr size_t QC = (size_t)NQ * NQ * NQ, VC = (size_t)NV * NV * NV;

    const int gl = tid / (NQ * NQ), pl = tid - gl * (NQ * NQ);      // pencils along l: lane (n,m)
    constexpr int PM = NQ * NV, PN = NV * NV, LM = COMPACT ? PM : NQ * NQ, LN = COMPACT ? PN : NQ * NQ;
    const int gm = tid / LM, pm = tid - gm * LM;                    // pencils along m: lane (n,i)
    const int gn = tid / LN, pn = tid - gn * LN;                    // pencils along n: lane (j,i)
    const bool on_l = gl < here, on_m = gm < here && pm < PM, on_n = gn < here && pn < PN;

    T xq[NQ], x2[NQ], yv[NV], zv[NV];

    // axis l: lane (n,m) owns the NQ consecutive words [e][n][m][0..NQ-1] of M and P
    if (on_l) {
        const long long unit = batch * G + gl;
        const long long e = unit / 3;
        const int c = (int)(unit - 3 * e);
        T mq[NQ];
        load_words<(HINT & 1) != 0>(Mq + (size_t)e * QC + (size_t)(pl * NQ), mq);
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
            const size_t cube = ((size_t)(c * 3 + dir) * (size_t)num_elems + (size_t)e) * QC;
            load_words<(HINT & 1) != 0>(Pq + cube + (size_t)(pl * NQ), xq);
#pragma unroll
            for (int l = 0; l < NQ; ++l) xq[l] *= mq[l];
            if (dir == 2) {
#pragma unroll
                for (int l = 0; l < NQ; ++l) x2[l] = xq[l];
            } else {
                matrix_product<T, NV, NQ, false, SB>(dir == 0 ? Dm : Im, xq, yv);
                T *dst = lds + (2 * gl + dir) * CUBE;
                const int nn = pl / NQ, mm = pl - nn * NQ;
#pragma unroll
                for (int i = 0; i < NV; ++i) dst[nn * PA + mm * PB + i] = yv[i];
            }
        }
    }
    __syncthreads();

    // axis m, first two terms merged: lane (n,i)
    T *c0 = lds + 2 * gm * CUBE, *c1 = c0 + CUBE;
    const int bn = pm / NV, bi = pm - bn * NV;
    if (on_m) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c0[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c1[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Dm, xq, zv);
    }
    __syncthreads();                                    // every pencil of cubes 0 and 1 has been read
    if (on_m) {
#pragma unroll
        for (int j = 0; j < NV; ++j) c0[bn * PA + j * PB + bi] = yv[j] + zv[j];
    }
    // axis l of the third term, into the freed cube 1: lane (n,m)
    if (on_l) {
        T *dst = lds + (2 * gl + 1) * CUBE;
        const int nn = pl / NQ, mm = pl - nn * NQ;
        matrix_product<T, NV, NQ, false, SB>(Im, x2, yv);
#pragma unroll
        for (int i = 0; i < NV; ++i) dst[nn * PA + mm * PB + i] = yv[i];
    }
    __syncthreads();
    // axis m of the third term: lane (n,i)
    if (on_m) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) xq[m] = c1[bn * PA + m * PB + bi];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int j = 0; j < NV; ++j) c1[bn * PA + j * PB + bi] = yv[j];   // the lane's own pencil
    }
    __syncthreads();

    // axis n: lane (j,i); stores are consecutive over lanes
    if (on_n) {
        const T *d0 = lds + 2 * gn * CUBE, *d1 = d0 + CUBE;
        const int jj = pn / NV, ii = pn - jj * NV;
#pragma unroll
        for (int n = 0; n < NQ; ++n) xq[n] = d0[n * PA + jj * PB + ii];
        matrix_product<T, NV, NQ, false, SB>(Im, xq, yv);
#pragma unroll
        for (int n = 0; n < NQ; ++n) xq[n] = d1[n * PA + jj * PB + ii];
        matrix_product<T, NV, NQ, false, SB>(Dm, xq, zv);
        const long long unit = batch * G + gn;
        const long long e = unit / 3;
        const size_t out = ((size_t)(unit - 3 * e) * (size_t)num_elems + (size_t)e) * VC;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            gstore<(HINT & 2) != 0>(F + out + (size_t)(k * NV * NV + pn), yv[k] + zv[k]);
    }
}

// Units per workgroup by lane utilisation: with at most 512 threads and 56 KB of LDS.
template <typename T, int NV, int NQ>
constexpr int convection_rect_group()
{
    int best = 1;
    long best_num = 0, best_den = 1;
    for (int g = 1; g <= 64; ++g) {
        const int p = g * ConvRectShape<T, NV, NQ, 1>::L;
        const int nt = ((p + 63) / 64) * 64;
        const long lds = (long)g * (long)ConvRectShape<T, NV, NQ, 1>::LDS_BYTES;
        if (g > 1 && (nt > 512 || lds > 56 * 1024)) break;
        if ((long)p * best_den > best_num * nt) {
            best = g;
            best_num = p;
            best_den = nt;
        }
    }
    return best;
}

// The utilisation rule's group and the first form, or the second form with a row's settings: the best of a
// sweep on MI355X over {1, 2, 3, 4, 6, 8, 12} units, the rule's group and both lane numberings, 2 GB per
// call, kept where it gains 2 % or more.  us per call on 2.5 GB, rule / row: fp64 (8,10) 523 / 441, (8,12) 515 / 486,
// (10,12) 529 / 472, (11,12) 648 / 479; fp32 (3,4) 492 / 454, (10,12) 527 / 498, (11,13) 546 / 510, (9,14) 517 / 473;
// with buffers in turns fp32 (6,8), (10,11) 0.97, (12,13) 0.93 .. 0.98 of the time.
// These serve the batches past the rows of ConvRectFirstTable.
// `from`: MiB of fields from which the row is the faster one.
//   0: on small batches too, mostly because it takes the smaller workgroups of the two (150 MB: fp64 (8,10) 31.3 /
//   25.9, (11,12) 45.9 / 33.6).  Larger groups lose there, where a launch is a few rounds of workgroups (2 MB:
//   fp64 (6,8) 3.8 / 5.9, (7,11) 5.6 / 7.2).
//   256: once the fields pass the last-level cache.
//   320: up to there the fields are cached in part and the smaller workgroups lead (row over rule at 275 .. 310 MB:
//   fp64 (6,8) 1.05, (7,8) 1.05, (7,9) 1.06, (9,11) 1.06; fp32 (2,3) 1.02 .. 1.10, (3,4) 1.02 .. 1.05).
//   60: fp32 (9,11) 0.93 .. 0.98 up to 200 MB, 1.00 .. 1.02 below.
//   26: fp32 (6,9) 0.95 .. 0.98 up to 300 MB; below 1.05 .. 1.12 at 11 .. 16 and 22 .. 24 MB, 0.84 .. 0.98 between.
struct ConvRectRow { int nv, nq, g, compact, from; };
template <typename T> struct ConvRectTable;
template <> struct ConvRectTable<double> {
    static constexpr ConvRectRow row[] = {
        {2, 4, 6, 1, 256},   {3, 4, 6, 0, 256},  {6, 8, 8, 1, 320},  {7, 8, 8, 0, 320}, {7, 9, 6, 0, 320},
        {7, 11, 4, 1, 256},  {8, 10, 1, 0, 0},   {8, 12, 3, 1, 256}, {9, 10, 1, 0, 0},  {9, 11, 2, 0, 320},
        {9, 14, 2, 1, 0},    {10, 12, 1, 0, 0},  {11, 12, 1, 0, 0},
    };
};
template <> struct ConvRectTable<float> {
    static constexpr ConvRectRow row[] = {
        {2, 3, 12, 1, 320},  {2, 4, 12, 0, 256},  {3, 4, 8, 1, 320},   {3, 5, 8, 1, 256}, {4, 5, 8, 1, 256},
        {5, 8, 6, 0, 256},   {6, 8, 6, 1, 256},   {6, 9, 4, 1, 26},    {8, 10, 3, 1, 0},  {8, 12, 2, 1, 0},
        {9, 11, 2, 1, 60},   {9, 14, 2, 1, 0},    {10, 11, 2, 0, 256}, {10, 12, 2, 1, 256}, {11, 13, 3, 1, 256},
        {12, 13, 3, 1, 256},
    };
};
template <typename T>
constexpr ConvRectRow convection_rect_row(int nv, int nq)
{
    for (const ConvRectRow &r : ConvRectTable<T>::row)
        if (r.nv == nv && r.nq == nq) return r;
    return {nv, nq, 0, 0, 0};           // no row: the first form at every batch size
}

constexpr long long kConvectionCachedBytes = 256LL << 20;
// Elements whose ten input and three output cubes take up `bytes`.
template <typename T, int NV, int NQ>
constexpr long long convection_elems(long long bytes)
{
    return bytes / ((10LL * NQ * NQ * NQ + 3LL * NV * NV * NV) * (long long)sizeof(T));
}

template <typename T, int NV, int NQ, int G, bool LARGE, bool COMPACT, int SB = convection_batch_words<T, NV, NQ>()>
struct ConvectionRectLauncherT {
    using Sh = ConvRectShape<T, NV, NQ, G>;
    static constexpr size_t LDS = Sh::LDS_BYTES;
    static constexpr int HINT = 2;
    static constexpr bool XCD = G % 3 != 0;

    static constexpr int CODE = setting_code(G, HINT, XCD, LARGE + COMPACT, SB);

    static constexpr auto kernel()
    {
        if constexpr (LARGE) return &convection_rect_large_kernel<T, NV, NQ, G, HINT, XCD, COMPACT, SB>;
        else return &convection_rect_kernel<T, NV, NQ, G, HINT, XCD, SB>;
    }

    static hipError_t launch(const ConvectionArgs &a)
    {
        const long long blocks = convection_grid<XCD>((3 * a.num_elems + G - 1) / G);
        if (blocks <= 0 || blocks > 0x7fffffffLL) return kGridTooLarge;
        drop_stale_error();
        hipLaunchKernelGGL(kernel(), dim3((unsigned)blocks), dim3(Sh::NT), LDS, a.stream,
                           (const T *)a.p, (const T *)a.m, (const T *)a.d_vq, (const T *)a.i_vq,
                           (T *)a.f, a.num_elems);
        return hipGetLastError();
    }

    static hipError_t prepare()
    {
        if (LDS <= 48 * 1024) return hipSuccess;
        return hipFuncSetAttribute((const void *)kernel(),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS);
    }
};

template <typename T, int NV, int NQ>
struct ConvectionRectLauncher {
    static constexpr ConvRectRow R = convection_rect_row<T>(NV, NQ);
    static constexpr int RULE_G = convection_rect_group<T, NV, NQ>();
    // No batch leaves the row: see takes_large().
    static constexpr bool ROW_ONLY = R.g != 0 && R.from == 0 && (R.g == 1 || R.g >= RULE_G);
    using Rule = ConvectionRectLauncherT<T, NV, NQ, RULE_G, false, false>;
    using Row = ConvectionRectLauncherT<T, NV, NQ, R.g != 0 ? R.g : 1, true, R.compact != 0>;
    // The batches that fit a row of ConvRectFirstTable, and whether those cover every batch that takes_large() refuses.
    static constexpr long long FIRST_END = convection_elems<T, NV, NQ>((long long)convection_rect_first_end<T>(NV, NQ) << 20);
    static constexpr int CUS = 256;
    static constexpr bool COVERED = R.g != 0 && FIRST_END >= convection_elems<T, NV, NQ>((long long)R.from << 20) &&
                                    FIRST_END * 3 >= CUS * RULE_G;
    using Small = std::conditional_t<ROW_ONLY || COVERED, Row, Rule>;
    using Large = std::conditional_t<R.g != 0, Row, Rule>;
    // A shape has at most three rows of ConvRectFirstTable; a last one with mib = 0 leaves nothing to the two settings.
    template <int K> static constexpr ConvRectFirst first_row = convection_rect_first<T>(NV, NQ, K);
    template <int K> static constexpr bool is_row = first_row<K>.g != 0;
    template <int K> static constexpr bool every = is_row<K> && first_row<K>.mib == 0;
    static_assert(!is_row<3>, "launch() looks at three rows");
    static constexpr bool FIRST_ONLY = every<0> || every<1> || every<2>;
    template <int K> using First = ConvectionRectLauncherT<T, NV, NQ, first_row<K>.g, first_row<K>.form != 0,
                                                           first_row<K>.form == 2, first_row<K>.sb>;

    // f(Use<the launcher of the setting that a batch takes>)
    template <typename F>
    static void with_setting(long long num_elems, F &&f)
    {
        if constexpr (is_row<0>) if (convection_rect_fits<T>(first_row<0>, num_elems)) return f(Use<First<0>>{});
        if constexpr (is_row<1>) if (convection_rect_fits<T>(first_row<1>, num_elems)) return f(Use<First<1>>{});
        if constexpr (is_row<2>) if (convection_rect_fits<T>(first_row<2>, num_elems)) return f(Use<First<2>>{});
        if constexpr (!FIRST_ONLY) {
            if (takes_large(num_elems)) f(Use<Large>{});
            else f(Use<Small>{});
        }
    }
    static hipError_t launch(const ConvectionArgs &a)
    {
        hipError_t rc = kGridTooLarge;
        with_setting(a.num_elems, [&](auto s) { rc = decltype(s)::type::launch(a); });
        return rc;
    }
    static int setting(long long num_elems)
    {
        int code = -1;
        with_setting(num_elems, [&](auto s) { code = decltype(s)::type::CODE; });
        return code;
    }
    // Of the two settings past the rows.
    static bool takes_large(long long num_elems)
    {
        if (ROW_ONLY) return true;
        if (R.g == 0 || num_elems <= convection_elems<T, NV, NQ>((long long)R.from << 20)) return false;
        // While the rule's larger workgroups still are one per CU and the row's are not, the rule's lead (row
        // over rule: fp32 (8,10) 1.03 .. 1.07 at 12 .. 18 MB, (8,12) 1.08 .. 1.10 at 13 .. 19 MB; 0.75 .. 0.90 on both
        // sides of that).  One unit per workgroup is ahead all the same (fp64 (8,10) 0.92 .. 0.96).
        return num_elems * 3 <= CUS * R.g || num_elems * 3 > CUS * RULE_G;
    }
    static hipError_t prepare()
    {
        hipError_t rc = hipSuccess;
        if constexpr (is_row<0>) rc = First<0>::prepare();
        if constexpr (is_row<1>) if (rc == hipSuccess) rc = First<1>::prepare();
        if constexpr (is_row<2>) if (rc == hipSuccess) rc = First<2>::prepare();
        if constexpr (!FIRST_ONLY) {
            if (rc == hipSuccess) rc = Large::prepare();
            if (rc == hipSuccess) rc = Small::prepare();
        }
        return rc;
    }
};

struct ConvectionRectEntry {
    int n_v, n_q;
    ConvectionEntry entry;
};
#define TPO_CONVECTION_RECT_ENTRY(T, NV, NQ)                                              \
    ConvectionRectEntry { NV, NQ, ConvectionEntry { &ConvectionRectLauncher<T, NV, NQ>::launch, \
                                                    &ConvectionRectLauncher<T, NV, NQ>::prepare, \
                                                    &ConvectionRectLauncher<T, NV, NQ>::setting } }

// Square shapes.  ConvectionTune: units per workgroup by lane utilisation, SPLIT by size, and in fp32 from n = 9 on the
// 4x4x1 matrix-core form (the vector-FMA form is bound by FMA issue there, as for the operator).  A sweep of units x
// SPLIT x form x order of the loads x HINT over 0.5 MB .. 2.5 GB on MI355X, with buffers that take turns, found better
// settings for the n below (time over ConvectionTune's at 400 MB / 2.5 GB: fp64 n = 6 0.97 / 0.98; fp32 n = 10
// 0.92 / 0.97, 14 0.86 / 0.98; fp64 n = 7, 10 and fp32 n = 7 from an earlier sweep: 430 / 454, 432 / 484,
// 446 / 462 us on 2.5 GB), and for smaller batches the rows of SquareConvectionRows.  fp32 n = 8 in the matrix-core
// form: 0.83 .. 0.95 of the time on 9 .. 200 MB, the same elsewhere.  ConvectionLargeTune pays only once the fields
// pass the last-level cache (2.5 GB: fp64 n = 3 525 / 499, 9 460 / 444; fp32 n = 3 567 / 516, 5 486 / 468,
// 11 502 / 466 us).
template <typename T, int N> struct ConvectionTune {
    static constexpr int G = convection_group<T, N>(), HINT = 2;
    static constexpr bool SPLIT = convection_split<T, N>();
    static constexpr bool MM = sizeof(T) == 4 && N >= 9, LOADS_FIRST = MM && N >= 13;
    static constexpr int SB = convection_batch_words<T, N>();
};
template <typename T, int N, int GG, bool S, bool M, bool L = (M && N >= 13)> struct ConvectionSet : ConvectionTune<T, N> {
    static constexpr int G = GG;
    static constexpr bool SPLIT = S, MM = M, LOADS_FIRST = L;
};
template <typename T, int N> struct ConvectionBase : ConvectionTune<T, N> {};
template <> struct ConvectionBase<double, 6> : ConvectionSet<double, 6, 1, false, false> {};
template <> struct ConvectionBase<double, 7> : ConvectionSet<double, 7, 1, false, false> {};
template <> struct ConvectionBase<double, 10> : ConvectionSet<double, 10, 1, true, false> {};
template <> struct ConvectionBase<float, 7> : ConvectionSet<float, 7, 1, true, true> {};
template <> struct ConvectionBase<float, 8> : ConvectionSet<float, 8, 1, true, true> {};
template <> struct ConvectionBase<float, 9> : ConvectionSet<float, 9, 3, true, true> {};
template <> struct ConvectionBase<float, 10> : ConvectionSet<float, 10, 2, false, true, true> {};
template <> struct ConvectionBase<float, 12> : ConvectionSet<float, 12, 3, true, true> {};
template <> struct ConvectionBase<float, 14> : ConvectionSet<float, 14, 2, false, true> {};
template <typename T, int N> struct ConvectionLargeTune : ConvectionBase<T, N> {
    // fp64 on large batches (3 GB, with / without: n = 11 527 / 551 us, 12 569 / 582,
    // 13 584 / 622, 14 632 / 672, 15 716 / 772, 16 703 / 750; n = 10 524 / 521, 9 544 / 534, 8 529 / 527,
    // 6 527 / 519), where the wait for memory outweighs the registers; cached ones lose 2 to 9 %
    // (n = 11, 150 MB: 38.4 / 35.2).
    static constexpr bool LOADS_FIRST = ConvectionBase<T, N>::LOADS_FIRST || (sizeof(T) == 8 && N >= 11);
};
template <> struct ConvectionLargeTune<double, 3> : ConvectionSet<double, 3, 16, false, false> {};
template <> struct ConvectionLargeTune<double, 9> : ConvectionSet<double, 9, 3, true, false> {};
template <> struct ConvectionLargeTune<float, 3> : ConvectionSet<float, 3, 16, false, false> {};
template <> struct ConvectionLargeTune<float, 5> : ConvectionSet<float, 5, 8, false, false> {};
template <> struct ConvectionLargeTune<float, 11> : ConvectionSet<float, 11, 2, true, true> {};

template <typename T, int N, typename Tune>
struct ConvectionLauncherT {
    static constexpr int G = Tune::G, HINT = Tune::HINT;
    using Sh = PencilShape<T, N, G>;
    static constexpr size_t LDS = (size_t)(Tune::SPLIT ? 2 : 3) * G * Sh::CUBE * sizeof(T);
    // Non-temporal stores are worth 3 to 8 %, non-temporal loads halve the rate (the per-lane runs
    // share cache lines).
    static constexpr bool XCD = G % 3 != 0;    // with G a multiple of 3 an element stays in one workgroup
    static constexpr int CODE = setting_code(G, HINT, XCD, Tune::MM + 2 * Tune::SPLIT + 4 * Tune::LOADS_FIRST, Tune::MM ? 0 : Tune::SB);

    static constexpr auto kernel()
    {
        if constexpr (Tune::MM) return &convection_mm_kernel<N, G, HINT, XCD, Tune::SPLIT, Tune::LOADS_FIRST>;
        else return &convection_pencil_kernel<T, N, G, HINT, XCD, Tune::SPLIT, Tune::LOADS_FIRST, Tune::SB>;
    }

    static hipError_t launch(const ConvectionArgs &a)
    {
        const long long blocks = convection_grid<XCD>((3 * a.num_elems + G - 1) / G);
        if (blocks <= 0 || blocks > 0x7fffffffLL) return kGridTooLarge;
        drop_stale_error();
        hipLaunchKernelGGL(kernel(), dim3((unsigned)blocks), dim3(Sh::NT), LDS, a.stream,
                           (const T *)a.p, (const T *)a.m, (const T *)a.d_vq, (const T *)a.i_vq,
                           (T *)a.f, a.num_elems);
        return hipGetLastError();
    }

    static hipError_t prepare()
    {
        if (LDS <= 48 * 1024) return hipSuccess;
        return hipFuncSetAttribute((const void *)kernel(),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS);
    }
};

template <typename T, int N>
struct ConvectionLauncher {
    // All loads first at n = 11, 12 costs until the fields are some times the cache (275 .. 430 MB: n = 11 1.02
    // .. 1.09 of the time, n = 12 0.99 .. 1.02; 600 MB 1.00, 0.99; 1.2 GB 0.96, 0.97).
    static constexpr long long FROM = sizeof(T) == 8 && (N == 11 || N == 12) ? 1LL << 30 : kConvectionCachedBytes;
    using Large = ConvectionLauncherT<T, N, ConvectionLargeTune<T, N>>;
    using Cached = std::conditional_t<((long long)batch_rows_end(SquareConvectionRows<T>::rows, N) << 20) >= FROM, Large,
                                      ConvectionLauncherT<T, N, ConvectionBase<T, N>>>;
    template <int K> using Row = ConvectionLauncherT<T, N, ConvectionBatchTune<SquareConvectionRows<T>::rows, N, K>>;
    // f(Use<the launcher of the setting that a batch takes>)
    template <typename F>
    static void with_setting(long long num_elems, F &&f)
    {
        if (for_batch_row<SquareConvectionRows<T>::rows, N>(num_elems, 13LL * N * N * N * (long long)sizeof(T),
                                                            [&](auto k) { f(Use<Row<decltype(k)::value>>{}); }))
            return;
        if (takes_large(num_elems)) f(Use<Large>{});
        else f(Use<Cached>{});
    }
    static hipError_t launch(const ConvectionArgs &a)
    {
        hipError_t rc = hipSuccess;
        with_setting(a.num_elems, [&](auto s) { rc = decltype(s)::type::launch(a); });
        return rc;
    }
    static int setting(long long num_elems)
    {
        int code = 0;
        with_setting(num_elems, [&](auto s) { code = decltype(s)::type::CODE; });
        return code;
    }
    // Of the two settings past the rows.
    static bool takes_large(long long num_elems) { return num_elems > convection_elems<T, N, N>(FROM); }
    static hipError_t prepare()
    {
        hipError_t rc = Cached::prepare();
        if (rc == hipSuccess) rc = Large::prepare();
        for_each_batch_row<SquareConvectionRows<T>::rows, N>([&](auto k) {
            if (rc == hipSuccess) rc = Row<decltype(k)::value>::prepare();
        });
        return rc;
    }
};

#define TPO_CONVECTION_ENTRY(T, N) \
    ConvectionEntry { &ConvectionLauncher<T, N>::launch, &ConvectionLauncher<T, N>::prepare, \
                      &ConvectionLauncher<T, N>::setting }

}  // namespace tpo
