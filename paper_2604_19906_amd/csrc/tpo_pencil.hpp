// Register-blocked vector-FMA kernel family ("pencil" kernels) for the batched
// inverse-Helmholtz tensor-product operator on gfx950.
//
// One lane owns one pencil: the n values of the cube along the axis being contracted, for
// fixed values of the other two indices.  A mode product is then n*n FMAs on registers:
// the lane's n inputs, n accumulators, and the n*n matrix entries, which are uniform over
// the wavefront and are read through the scalar data path (s_load + SGPR operand of
// v_fma), so they cost neither VGPRs nor LDS bandwidth.  Between axes the cube is
// re-distributed through LDS.  A workgroup processes G whole elements at a time (G*n*n
// pencils, padded to a multiple of 64 lanes); all six mode products and the diagonal scale
// run on chip, HBM sees u_e and D_e once (coalesced reads) and v_e once (coalesced store).
//
// Order of the six products (mode products along different axes commute):
//   forward axis 0 (from global, lanes consecutive along (b,c): coalesced)
//   forward axis 1, forward axis 2, scale by D_e, backward axis 2 (same registers),
//   backward axis 1, backward axis 0 (to global, coalesced).
// D_e either arrives in its axis-2 pencil layout (each lane loads the n consecutive words of
// its pencil) or coalesced like u_e and parked in LDS until the scale, or is evaluated in the
// kernel from its separable form; see the template parameters of ihelm_pencil_kernel.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "tpo_batch_rows.hpp"
#include "tpo_internal.h"

namespace tpo {

#define TPO_CONSTANT __attribute__((address_space(4)))

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// 1/x for the separable diagonal.  EXACT: IEEE division.  Otherwise the hardware reciprocal,
// in fp64 followed by two Newton steps (v_rcp_f64 delivers about single precision): within
// 2 ulp for normal x, a third of the instructions of the IEEE sequence.
template <bool EXACT>
__device__ __forceinline__ double recip_(double x)
{
    if constexpr (EXACT) return 1.0 / x;
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
template <bool EXACT>
__device__ __forceinline__ float recip_(float x)
{
    if constexpr (EXACT) return 1.0f / x;
    return __builtin_amdgcn_rcpf(x);
}

template <typename T, int N, int G>
struct PencilShape {
    static constexpr int P = N * N;                         // pencils per element
    static constexpr int NT = ((G * P + 63) / 64) * 64;     // threads per workgroup
    // LDS pitches (in words): row pitch odd, plane pitch odd, so that the three access
    // patterns (lanes consecutive along c, along c with a in the high part, along b)
    // spread over the banks.
    static constexpr int PB = (N & 1) ? N : N + 1;
    static constexpr int PA = ((N * PB) & 1) ? N * PB : N * PB + 1;
    static constexpr int CUBE = N * PA;
    static constexpr size_t LDS_BYTES = (size_t)2 * G * CUBE * sizeof(T);
};

// Number of elements per workgroup: the G (1..64) with the best lane utilisation among
// those with at most 512 threads and at most ~53 KB of LDS (three workgroups per CU);
// G = 1 if nothing fits.
template <typename T, int N>
constexpr int pencil_group()
{
    int best = 1;
    long best_num = 0, best_den = 1;  // utilisation = num/den
    for (int g = 1; g <= 64; ++g) {
        const int p = g * N * N;
        const int nt = ((p + 63) / 64) * 64;
        const int pb = (N & 1) ? N : N + 1;
        const int pa = ((N * pb) & 1) ? N * pb : N * pb + 1;
        const long lds = 2L * g * N * pa * (long)sizeof(T);
        if (nt > 512 || lds > 53 * 1024) break;
        if ((long)p * best_den > best_num * nt) {
            best = g;
            best_num = p;
            best_den = nt;
        }
    }
    return best;
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, K - 1>)
template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// Product with a matrix S of R rows and C columns (row-major), read through the constant address
// space so that its entries arrive in SGPRs:
//   FWD : y[c] = sum_r S[r][c] * x[r]   (the transpose of the stored matrix is applied)
//   !FWD: y[r] = sum_c S[r][c] * x[c]
//
// What bounds it with few wavefronts on a SIMD is the scalar loads: they come back in any order, so that
// a wavefront can only wait for all of them, and left to itself the compiler issues one right before that
// wait: 16 FMAs (64 cycles), then the whole latency of a load, 13 times a product at fp64 n = 14.  Matrices
// of more than 2 * SB words therefore come in batches of SB words in two buffers: wait for batch b, issue
// the loads of batch b + 1, then the FMAs of batch b; the fences hold that order.  Time over the unbatched
// product's (MI355X, fp64): 0.5 MB a call, n = 8 0.86, 11 0.83, 14 0.78, 16 0.72; 200 MB 0.97, 0.93, 0.93,
// 0.91; 2.5 GB n <= 11 1.00, 12 0.92, 13 0.96, 14 0.95, 16 0.94; square convection n = 15, 16 0.86, 0.80 at
// 2.5 GB.  Batches of 16 / 24 / 40 words: 1.03 .. 1.30 at 60 MB / 0.87 .. 0.97 at all sizes / ahead by 2 .. 12 % at
// 60 and 200 MB for n >= 11, behind by 3 .. 8 % at 2.5 GB (with 40 the compiler spills 30 .. 50 scalars into lanes of vector
// registers, 70 .. 140 instructions of a wavefront; operator n = 9 65 registers instead of 64).  In fp32 they reach the anisotropic
// kernels, for axes of nine points and more: 0.91 of the time at 4 MB, 0.98 at 16, 1.00 at 36 .. 90, 1.01 .. 1.02 from 130 MB on.  Matrices of up to two batches fit the SGPRs at
// once and lose up to 12 % by the fences (convection n <= 8 in fp32, 4 and 5 in fp64, at 60 and 200 MB).
// SB = 0 leaves the order to the compiler, for the kernels that are slower with batches.
constexpr int kScalarBatch = 32;
template <typename T, int R, int C, bool FWD, int SB = kScalarBatch>
__device__ __forceinline__ void matrix_product(const TPO_CONSTANT T *S, const T (&x)[FWD ? R : C],
                                               T (&y)[FWD ? C : R])
{
    // Make the pointer opaque per product: otherwise two products with the same matrix share
    // one set of scalar loads, all entries stay live across both and spill out of the
    // SGPR file.
    asm volatile("" : "+s"(S));
    constexpr int NE = R * C;                                   // entries
    constexpr int B = (SB & 255) * 4 / (int)sizeof(T);          // entries per batch
    if constexpr (B == 0 || NE <= 2 * B) {
        if constexpr (FWD) {
#pragma unroll
            for (int c = 0; c < C; ++c) y[c] = S[c] * x[0];
#pragma unroll
            for (int r = 1; r < R; ++r) {
#pragma unroll
                for (int c = 0; c < C; ++c) y[c] = fma_(S[r * C + c], x[r], y[c]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                T acc = S[r * C] * x[0];
#pragma unroll
                for (int c = 1; c < C; ++c) acc = fma_(S[r * C + c], x[c], acc);
                y[r] = acc;
            }
        }
    } else {
        T buf[2][B];
        auto load = [&](int b) {
#pragma unroll
            for (int k = 0; k < B; ++k)
                if (b * B + k < NE) buf[b & 1][k] = S[b * B + k];
        };
        auto term = [&](int b, int k) {
            const int q = b * B + k;
            if (q >= NE) return;
            const int r = q / C, c = q - r * C;
            const int i = FWD ? c : r, l = FWD ? r : c;
            y[i] = l == 0 ? buf[b & 1][k] * x[0] : fma_(buf[b & 1][k], x[l], y[i]);
        };
        load(0);
        for_each_index([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            term(b, 0);                                 // waits for batch b
            __builtin_amdgcn_sched_barrier(0);
            load(b + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 1; k < B; ++k) term(b, k);
            __builtin_amdgcn_sched_barrier(0);
        }, std::make_integer_sequence<int, (NE + B - 1) / B>{});
    }
}

// Settings with kWarm in SB (launches of about one workgroup per CU at most): every 64-byte line of the matrices is touched right after
// the wavefront has asked for its first words of the fields, by scalar loads that all go out before one wait per matrix (a second and
// third one only where they differ: the registers of all three do not fit).  There the matrices are in no scalar cache yet, and every
// batch of a product misses, one wait after the other; on larger launches the workgroups before have brought them in, and the touching only
// costs (1.01 .. 1.05).  Time with / without, fp64, up to the rows' ends: halves n = 12 0.90 .. 0.97, 13 0.86 .. 0.96, 14 and 15 0.88 ..
// 0.92, 16 0.72 .. 0.80; convection n = 10 .. 13 0.89 .. 0.92, 14 0.89 .. 0.98, 15 0.86 .. 0.92, 16 0.88 .. 0.90, (8,12) and (9,14) 0.91 ..
// 0.98; operator n = 9 0.93 .. 1.00 (three matrices; one 0.99), 10 0.87 .. 0.88 (0.99), with one matrix 11 0.96 .. 0.97, 13 .. 15 0.93 .. 0.97
// (with three they run in the tiles); separable n = 9, 10 0.89 .. 0.92.  Smaller matrices gain nothing (0.98 .. 1.05).  Touched in groups of
// eight with a wait after each, as the compiler has it where one register collects the words: halves 1.02 .. 1.06 of this time,
// convection 1.00 .. 1.03, operator and separable form 1.00 .. 1.02.
template <int SB, int WORDS, typename T, typename... M>
__device__ __forceinline__ void warm_scalar_cache(const TPO_CONSTANT T *first, M... more)
{
    if constexpr ((SB & kWarm) != 0) {
        constexpr int LINES = (WORDS * (int)sizeof(T) + 63) / 64 + 1;       // and the last word, which may lie in a line of its own
        auto touch = [&](const TPO_CONSTANT T *S) {
            const TPO_CONSTANT unsigned *w = (const TPO_CONSTANT unsigned *)S;
            unsigned t[LINES];
#pragma unroll
            for (int k = 0; k < LINES - 1; ++k) t[k] = w[16 * k];
            t[LINES - 1] = w[WORDS * (int)sizeof(T) / 4 - 1];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < LINES; ++k) asm volatile("" :: "s"(t[k]));
        };
        __builtin_amdgcn_sched_barrier(0);
        touch(first);
        ((more != first ? touch(more) : void()), ...);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The square product of the operators: y[i] = sum_l S[l][i] * x[l] (FWD), sum_l S[i][l] * x[l] (!FWD).
template <typename T, int N, bool FWD, int SB = kScalarBatch>
__device__ __forceinline__ void mode_product(const TPO_CONSTANT T *S, const T (&x)[N], T (&y)[N])
{
    matrix_product<T, N, N, FWD, SB>(S, x, y);
}

// Global accesses with or without the non-temporal hint (streamed once, never re-read).
template <bool NT, typename T>
__device__ __forceinline__ T gload(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void gstore(T *p, T x)
{
    if constexpr (NT) __builtin_nontemporal_store(x, p);
    else *p = x;
}

// K consecutive words of type T from/to global memory at word alignment, as the widest
// accesses the hardware takes at that alignment (vectors of 2 and 4 words declared with the
// alignment of one word become dwordx2 / dwordx4 instructions).
template <typename T, int W> struct WordVec {
    typedef T type __attribute__((ext_vector_type(W), aligned(sizeof(T))));
};
template <bool NT, typename T, int K>
__device__ __forceinline__ void load_words(const T *p, T (&out)[K])
{
    typedef typename WordVec<T, 4>::type v4;
    typedef typename WordVec<T, 2>::type v2;
    int q = 0;
#pragma unroll
    for (; q + 4 <= K; q += 4) {
        const v4 *pv = reinterpret_cast<const v4 *>(p + q);
        v4 t;
        if constexpr (NT) t = __builtin_nontemporal_load(pv); else t = *pv;
        out[q] = t[0]; out[q + 1] = t[1]; out[q + 2] = t[2]; out[q + 3] = t[3];
    }
    if (q + 2 <= K) {
        const v2 *pv = reinterpret_cast<const v2 *>(p + q);
        v2 t;
        if constexpr (NT) t = __builtin_nontemporal_load(pv); else t = *pv;
        out[q] = t[0]; out[q + 1] = t[1];
        q += 2;
    }
    if (q < K) out[q] = gload<NT>(p + q);
}
template <bool NT, typename T, int K>
__device__ __forceinline__ void store_words(T *p, const T (&in)[K])
{
    typedef typename WordVec<T, 4>::type v4;
    typedef typename WordVec<T, 2>::type v2;
    int q = 0;
#pragma unroll
    for (; q + 4 <= K; q += 4) {
        v4 t = {in[q], in[q + 1], in[q + 2], in[q + 3]};
        v4 *pv = reinterpret_cast<v4 *>(p + q);
        if constexpr (NT) __builtin_nontemporal_store(t, pv); else *pv = t;
    }
    if (q + 2 <= K) {
        v2 t = {in[q], in[q + 1]};
        v2 *pv = reinterpret_cast<v2 *>(p + q);
        if constexpr (NT) __builtin_nontemporal_store(t, pv); else *pv = t;
        q += 2;
    }
    if (q < K) gstore<NT>(p + q, in[q]);
}

// HINT bit 0: non-temporal coalesced loads (u, and D_e when it is loaded coalesced); bit 1:
// non-temporal stores of v; bit 2: non-temporal loads of D_e's per-lane runs (DDIRECT).
// DDIRECT = 0    : D_e is loaded coalesced with u_e and parked in LDS until the scale.
// DDIRECT = 1    : every lane loads, at kernel start, the n consecutive words of D_e that
//                  belong to its axis-2 pencil (no LDS for D_e: half the LDS per workgroup).
// XCD = true : workgroups are renumbered so that each of the 8 accelerator dies (workgroups
//              are dealt to them round-robin) works on one contiguous eighth of the elements;
//              cache lines shared by neighbouring elements then stay within one L2.
//              The grid must be pencil_grid<XCD>(number of batches).
template <bool XCD>
__host__ __device__ inline long long pencil_grid(long long nbatch)
{
    return XCD ? 8 * ((nbatch + 7) / 8) : nbatch;
}
template <bool XCD>
__device__ __forceinline__ long long pencil_batch(long long nbatch)
{
    if constexpr (XCD) {
        const long long per = (nbatch + 7) / 8;
        return (long long)(blockIdx.x & 7) * per + (long long)(blockIdx.x >> 3);
    } else {
        return blockIdx.x;
    }
}

// The first argument of a kernel whose setting has kHeld.  The build has arguments preloaded into scalar registers up to the first one that is a
// struct: none of them here.  (A struct of one member is passed as that member.)
template <typename T> struct HeldArgument {
    const T *p;
    const void *nothing;
    __host__ __device__ operator const T *() const { return p; }
};
template <typename T, bool HELD> using KernelField = std::conditional_t<HELD, HeldArgument<T>, const T *>;
template <typename FIELD, typename T> FIELD kernel_field(const T *p)
{
    if constexpr (std::is_pointer_v<FIELD>) return p;
    else return {p, nullptr};
}

// SEP != 0 : D_e is not read; it is evaluated where it is used from the separable form
//            D_e[a][b][c] = 1 / (lam_x[a] + lam_y[b] + lam_z[c] + mu[e])
//            (sum left to right; SEP = 1: IEEE division, SEP = 2: recip_<false>); D is ignored
//            and may be null.
// SB: see matrix_product.
// DDIRECT = 2    : the same words, asked for after the forward products along axes 0 and 1: half the
//                  words on their way at a time, for launches that LDS_MIN holds at few workgroups.
template <typename T, int N, int G, int HINT, int DDIRECT = 0, bool XCD = false,
          int SEP = 0, int SB = kScalarBatch>
__global__ void __launch_bounds__((PencilShape<T, N, G>::NT))
ihelm_pencil_kernel(KernelField<T, (SB & kHeld) != 0> u_, const T *Sx_, const T *Sy_, const T *Sz_,
                    const T *__restrict__ D, T *v, long long num_elems,
                    const T *__restrict__ lam_x, const T *__restrict__ lam_y,
                    const T *lam_z_, const T *__restrict__ mu)
{
    using Sh = PencilShape<T, N, G>;
    constexpr int P = Sh::P, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *cube_all = reinterpret_cast<T *>(tpo_lds);
    T *dpark_all = cube_all + G * CUBE;

    const T *u = u_;
    const TPO_CONSTANT T *Sx = (const TPO_CONSTANT T *)Sx_;
    const TPO_CONSTANT T *Sy = (const TPO_CONSTANT T *)Sy_;
    const TPO_CONSTANT T *Sz = (const TPO_CONSTANT T *)Sz_;

    const int tid = threadIdx.x;
    const int g = tid / P;          // element slot inside the workgroup
    const int p = tid - g * P;      // pencil id inside the element
    const int hi = p / N;
    const int lo = p - hi * N;
    const long long nbatch = (num_elems + G - 1) / G;
    const long long batch = pencil_batch<XCD>(nbatch);
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const long long e = batch * G + g;
    const bool on = (tid < G * P) && (e < num_elems);

    T *cube = cube_all + (g < G ? g : 0) * CUBE;
    T *dpark = dpark_all + (g < G ? g : 0) * CUBE;
    const size_t base = (size_t)(on ? e : 0) * (size_t)(N * N * N);

    T x[N], y[N];

    // forward, axis 0: lane (b,c) = (hi,lo); global reads are consecutive over lanes
    T dd[N];
    T sep_ab = T(0), sep_mu = T(0);     // lam_x[a] + lam_y[b] of the lane's axis-2 pencil, mu[e]
    if (on) {
#pragma unroll
        for (int l = 0; l < N; ++l) x[l] = gload<(HINT & 1) != 0>(u + base + (size_t)(l * P + p));
        if constexpr (SEP != 0) {
            sep_ab = lam_x[hi] + lam_y[lo];
            sep_mu = mu[e];
        } else if constexpr (DDIRECT == 1) {
            load_words<(HINT & 4) != 0>(D + base + (size_t)(p * N), dd);   // D_e[a][b][0..n-1]
        } else if constexpr (DDIRECT == 0) {
#pragma unroll
            for (int l = 0; l < N; ++l) dd[l] = gload<(HINT & 1) != 0>(D + base + (size_t)(l * P + p));
        }
        warm_scalar_cache<SB, N * N>(Sx, Sy, Sz);
        mode_product<T, N, true, SB>(Sx, x, y);
#pragma unroll
        for (int i = 0; i < N; ++i) cube[i * PA + hi * PB + lo] = y[i];
        if constexpr (!DDIRECT && SEP == 0) {
#pragma unroll
            for (int l = 0; l < N; ++l) dpark[l * PA + hi * PB + lo] = dd[l];
        }
    }
    __syncthreads();

    // forward, axis 1: lane (a,c) = (hi,lo)
    if (on) {
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = cube[hi * PA + m * PB + lo];
        mode_product<T, N, true, SB>(Sy, x, y);
        if constexpr (DDIRECT == 2 && SEP == 0) {
            __builtin_amdgcn_sched_barrier(0);
            load_words<(HINT & 4) != 0>(D + base + (size_t)(p * N), dd);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) cube[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // forward axis 2, diagonal scale, backward axis 2: lane (a,b) = (hi,lo)
    if (on) {
#pragma unroll
        for (int q = 0; q < N; ++q) x[q] = cube[hi * PA + lo * PB + q];
        mode_product<T, N, true, SB>(Sz, x, y);
        if constexpr (SEP != 0) {       // after the product: the reciprocals would hold N registers through it
            const TPO_CONSTANT T *lam_z = (const TPO_CONSTANT T *)lam_z_;
#pragma unroll
            for (int k = 0; k < N; ++k) dd[k] = recip_<SEP == 1>((sep_ab + lam_z[k]) + sep_mu);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) y[k] *= (DDIRECT || SEP != 0) ? dd[k] : dpark[hi * PA + lo * PB + k];
        mode_product<T, N, false, SB>(Sz, y, x);
#pragma unroll
        for (int k = 0; k < N; ++k) cube[hi * PA + lo * PB + k] = x[k];
    }
    __syncthreads();

    // backward, axis 1: lane (a,c) = (hi,lo)
    if (on) {
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = cube[hi * PA + m * PB + lo];
        mode_product<T, N, false, SB>(Sy, x, y);
#pragma unroll
        for (int j = 0; j < N; ++j) cube[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // backward, axis 0: lane (b,c) = (hi,lo); global stores are consecutive over lanes
    if (on) {
#pragma unroll
        for (int l = 0; l < N; ++l) x[l] = cube[l * PA + hi * PB + lo];
        mode_product<T, N, false, SB>(Sx, x, y);
#pragma unroll
        for (int i = 0; i < N; ++i) gstore<(HINT & 2) != 0>(v + base + (size_t)(i * P + p), y[i]);
    }
}

// Per (type, n): elements per workgroup G, hint bits, how D_e is brought in (1: straight into
// its pencil layout, half the LDS; 0: coalesced and parked in LDS), and whether the workgroups
// are renumbered per accelerator die.  One row per n = 1..16: the best of a sweep on MI355X over
// G in {1,2,3,4,6,8,12,16,32} x hint bits x D mode x renumbering on 1 GiB fields; n = 8, 11
// (fp64) and 13 (fp32) are the sweeps at the sizes of the named workloads, re-checked on the
// named workloads' own data (n = 8: D_e in per-lane runs 0.2501-0.2506 ms against 0.2523-0.2550
// parked in LDS, at 4 elements per workgroup with non-temporal accesses).  n = 1 keeps the
// lane-utilisation rule (G = 0 in the table).
struct PencilRow { int g, hint, ddirect, xcd; };
template <typename T> struct PencilTable;
template <> struct PencilTable<double> {
    static constexpr PencilRow row[TPO_MAX_N + 1] = {
        {0, 2, 1, 0},
        {0, 2, 1, 1},  {16, 2, 1, 0}, {32, 0, 1, 0}, {4, 3, 0, 0},  {16, 0, 1, 0}, {1, 3, 1, 0},
        {1, 3, 1, 0},  {4, 3, 1, 0},  {3, 1, 1, 0},  {1, 3, 1, 0},  {1, 0, 1, 1},  {3, 3, 1, 0},
        {3, 0, 1, 0},  {1, 0, 1, 0},  {1, 0, 1, 0},  {1, 3, 1, 1},
    };
};
template <> struct PencilTable<float> {
    static constexpr PencilRow row[TPO_MAX_N + 1] = {
        {0, 2, 1, 0},
        {0, 2, 1, 1},  {16, 2, 1, 0}, {24, 2, 1, 0}, {8, 2, 1, 0},  {8, 2, 1, 0}, {12, 0, 1, 0},
        {1, 3, 1, 1},  {2, 3, 1, 0},  {3, 0, 1, 0},  {2, 0, 1, 0},  {2, 0, 1, 0},  {3, 2, 1, 0},
        {3, 0, 1, 0},  {2, 0, 1, 0},  {2, 0, 1, 0},  {1, 3, 1, 0},
    };
};
template <typename T, int N>
struct PencilTune {
    static constexpr PencilRow R = PencilTable<T>::row[N];
    static constexpr int G = R.g > 0 ? R.g : pencil_group<T, N>();
    static constexpr int HINT = R.hint;
    static constexpr bool DDIRECT = R.ddirect != 0;
    static constexpr bool XCD = R.xcd != 0;
    static constexpr size_t LDS_MIN = 0;    // LDS requested at least (caps workgroups per CU)
    static constexpr int SB = kScalarBatch; // words per batch of scalar loads (matrix_product)
};
// n = 11: two elements per workgroup (242 of 256 lanes), non-temporal loads of u_e, D_e asked for late
// (DDIRECT 2), and an LDS request of 36 KB (20.8 KB are used), which holds the CU at 4 workgroups = 8
// elements instead of 14.  Bound by memory in one-shot bursts: a kernel of the same loads and stores alone
// runs at 6.28 TB/s with 85 KB asked for per CU and at 5.7 TB/s with 213 KB.  Against D_e at once with 28 KB
// (5 workgroups) 0.98 .. 0.99 of the time at 1.8 .. 8.4 GB and 0.975 .. 0.99 up to 29 GB, one matrix and three, the same
// fields and three sets in turn (50 calls of 15 alternating rounds, all below 1); the named workload 1437 -> 1420 us (1431 ->
// 1418 and 1436 -> 1420 on another box), less than what two boxes differ by
// (32 and 40 KB the same within 1 %; late D_e at 24 and 28 KB 0.99 .. 1.00; D_e at once with 32 .. 40 KB
// 1.02 .. 1.05; D_e after the product along axis 0 instead, 32 .. 40 KB, 1.01 .. 1.03).  Requests of
// 32 / 32 / 40 KB at n = 9, 15, 16 give 0.97 .. 1.03: not taken.  The first choice was made on the named workload
// (E = 262144, full-mantissa values; the settings rank differently on low-entropy data, where
// the clock runs higher), alternating libraries on one box, ms per launch: D_e at once with 28 KB 1.421-
// 1.424; the same with cached u_e loads 1.450-1.452; 26 KB / 30 KB requests 1.465 / 1.421-1.430;
// one element per workgroup with 18 KB (the earlier choice) 1.441-1.462, with 14 KB 1.469;
// three / four elements per workgroup 1.518 / 1.472.  Scalars in batches: 1.444 against 1.435 here (the rows by batch
// size, which serve everything up to 1650 MiB, take them; the other n keep them, 0.99 of the time before them at 4 and 8 GB,
// geometric mean, no call above 1.045).
template <> struct PencilTune<double, 11> {
    static constexpr int G = 2, HINT = 1, DDIRECT = 2;
    static constexpr bool XCD = true;
    static constexpr size_t LDS_MIN = 36 * 1024;
    static constexpr int SB = 0;
};

// Tuning of the separable-diagonal form: as the D form unless measured otherwise.  Without the
// D_e stream a workgroup has half the loads in flight, so the D form's occupancy cap at n = 11
// and its four elements per workgroup at n = 8 no longer pay (n = 11: 1.27 against 1.35 ms;
// n = 8: 0.202 against 0.215 ms).
template <typename T, int N>
struct PencilSepTune : PencilTune<T, N> {};
template <> struct PencilSepTune<double, 11> : PencilTune<double, 11> {
    static constexpr int G = 1, HINT = 0;
    static constexpr size_t LDS_MIN = 0;
    static constexpr int SB = kScalarBatch;
};
template <> struct PencilSepTune<double, 8> : PencilTune<double, 8> {
    static constexpr int G = 1;
};
// n = 12: with batches of scalar loads 1.06 .. 1.12 of the time at 100 MB .. 2.5 GB (0.82 .. 0.94 up to 25 MB)
template <> struct PencilSepTune<double, 12> : PencilTune<double, 12> {
    static constexpr int SB = 0;
};

// Settings of a pencil kernel spelled out.
template <int GG, int H, bool X> struct PencilSet {
    static constexpr int G = GG, HINT = H;
    static constexpr bool DDIRECT = true, XCD = X;
    static constexpr size_t LDS_MIN = 0;
    static constexpr int SB = kScalarBatch;
};
// Separable form on batches whose two fields pass the last-level cache, where a sweep over 1 .. 32
// elements per workgroup x hints x renumbering on 2 GB per call found 4 % or more against the D form's
// settings (us per call on 2.5 GB, before / now): fp64 n = 3 578 / 544, 5 530 / 464,
// 6 566 / 483, 9 550 / 522; fp32 n = 3 691 / 620, 4 456 / 443, 5 580 / 563, 6 580 / 551.  On smaller batches
// the gains are larger (600 MB: fp64 n = 6 136 / 115, fp32 n = 6 144 / 123); while the fields stay in the
// cache there are none to be had.
constexpr long long kPencilCachedBytes = 256LL << 20;
template <typename T, int N>
struct PencilSepLargeTune : PencilSepTune<T, N> {};
template <> struct PencilSepLargeTune<double, 3> : PencilSet<24, 0, false> {};
template <> struct PencilSepLargeTune<double, 5> : PencilSet<2, 2, false> {};
template <> struct PencilSepLargeTune<double, 6> : PencilSet<3, 0, false> {};
template <> struct PencilSepLargeTune<double, 9> : PencilSet<3, 0, false> {};
template <> struct PencilSepLargeTune<float, 3> : PencilSet<24, 2, false> {};
template <> struct PencilSepLargeTune<float, 4> : PencilSet<4, 2, false> {};
template <> struct PencilSepLargeTune<float, 5> : PencilSet<2, 0, true> {};
template <> struct PencilSepLargeTune<float, 6> : PencilSet<6, 2, false> {};

// SEP: 0 = D read from memory, 1 / 2 = separable diagonal (IEEE division / fast reciprocal).
template <typename T, int N, typename Tune, int SEP>
struct PencilLauncherT {
    static constexpr int G = Tune::G;
    using Sh = PencilShape<T, N, G>;
    static constexpr int DDIRECT = SEP != 0 ? 1 : (int)Tune::DDIRECT;       // no D_e in LDS either way
    static constexpr size_t LDS_USED = DDIRECT ? Sh::LDS_BYTES / 2 : Sh::LDS_BYTES;
    static constexpr size_t LDS = LDS_USED > Tune::LDS_MIN ? LDS_USED : Tune::LDS_MIN;
    static constexpr int CODE = setting_code(G, Tune::HINT, Tune::XCD, 0, Tune::SB);

    static constexpr auto kernel()
    {
        return &ihelm_pencil_kernel<T, N, G, Tune::HINT, DDIRECT, Tune::XCD, SEP, Tune::SB>;
    }
    using Field = KernelField<T, (Tune::SB & kHeld) != 0>;

    static hipError_t launch(const ApplyArgs &a)
    {
        const long long blocks = pencil_grid<Tune::XCD>((a.num_elems + G - 1) / G);
        if (blocks <= 0 || blocks > 0x7fffffffLL) return kGridTooLarge;
        drop_stale_error();
        hipLaunchKernelGGL(kernel(), dim3((unsigned)blocks), dim3(Sh::NT), LDS, a.stream,
                           kernel_field<Field>((const T *)a.u), (const T *)a.sx, (const T *)a.sy, (const T *)a.sz,
                           (const T *)a.d, (T *)a.v, a.num_elems, (const T *)a.lam_x,
                           (const T *)a.lam_y, (const T *)a.lam_z, (const T *)a.mu);
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
struct PencilLauncher {
    using Plain = PencilLauncherT<T, N, PencilTune<T, N>, 0>;
    using SepLarge = PencilLauncherT<T, N, PencilSepLargeTune<T, N>, 2>;     // fast reciprocal
    using Sep = std::conditional_t<((long long)batch_rows_end(PencilSepRows<T>::rows, N) << 20) >= kPencilCachedBytes, SepLarge,
                                   PencilLauncherT<T, N, PencilSepTune<T, N>, 2>>;
    template <int K> using Row = PencilLauncherT<T, N, BatchTune<PencilRows<T>::rows, N, K>, 0>;
    template <int K> using SepRow = PencilLauncherT<T, N, BatchTune<PencilSepRows<T>::rows, N, K>, 2>;
    static constexpr long long FIELD = (long long)N * N * N * (long long)sizeof(T);

    // f(Use<the launcher of the setting that a batch takes>)
    template <typename F>
    static void with_setting(long long num_elems, F &&f)
    {
        if (!for_batch_row<PencilRows<T>::rows, N>(num_elems, 3 * FIELD, [&](auto k) { f(Use<Row<decltype(k)::value>>{}); }))
            f(Use<Plain>{});
    }
    template <typename F>
    static void with_sep_setting(long long num_elems, F &&f)
    {
        if (for_batch_row<PencilSepRows<T>::rows, N>(num_elems, 2 * FIELD, [&](auto k) { f(Use<SepRow<decltype(k)::value>>{}); }))
            return;
        if (num_elems <= kPencilCachedBytes / (2 * FIELD)) f(Use<Sep>{});
        else f(Use<SepLarge>{});
    }
    static hipError_t launch(const ApplyArgs &a)
    {
        hipError_t rc = hipSuccess;
        with_setting(a.num_elems, [&](auto s) { rc = decltype(s)::type::launch(a); });
        return rc;
    }
    static hipError_t launch_sep(const ApplyArgs &a)
    {
        hipError_t rc = hipSuccess;
        with_sep_setting(a.num_elems, [&](auto s) { rc = decltype(s)::type::launch(a); });
        return rc;
    }
    static int setting(long long num_elems, bool sep)
    {
        int code = 0;
        auto get = [&](auto s) { code = decltype(s)::type::CODE; };
        if (sep) with_sep_setting(num_elems, get);
        else with_setting(num_elems, get);
        return code;
    }
    static hipError_t prepare()
    {
        hipError_t rc = Plain::prepare();
        if (rc == hipSuccess) rc = Sep::prepare();
        if (rc == hipSuccess) rc = SepLarge::prepare();
        auto also = [&](hipError_t (*f)()) { if (rc == hipSuccess) rc = f(); };
        for_each_batch_row<PencilRows<T>::rows, N>([&](auto k) { also(&Row<decltype(k)::value>::prepare); });
        for_each_batch_row<PencilSepRows<T>::rows, N>([&](auto k) { also(&SepRow<decltype(k)::value>::prepare); });
        return rc;
    }
};

#define TPO_PENCIL_ENTRY(T, N)                                                        \
    KernelEntry { &PencilLauncher<T, N>::launch, &PencilLauncher<T, N>::launch_sep, \
                  &PencilLauncher<T, N>::prepare, &PencilLauncher<T, N>::setting }

}  // namespace tpo
