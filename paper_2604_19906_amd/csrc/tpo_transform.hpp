// One half of the operator on its own: the three-dimensional transform
//   forward   t[i,j,k] = sum_l sum_m sum_q  S_x[l,i] * S_y[m,j] * S_z[q,k] * u[l,m,q]
//   backward  t[i,j,k] = sum_l sum_m sum_q  S_x[i,l] * S_y[j,m] * S_z[k,q] * u[l,m,q]
// evaluated as three one-dimensional mode products (the forward one is the worked example of
// reduction lifting in Sec. 5.2 of the paper).  Same building blocks as the pencil kernels
// (tpo_pencil.hpp): one pencil per lane, matrix entries in SGPRs, the cube re-distributed
// through LDS between axes.  Order: axis 2 first, on the n consecutive words each lane loads
// straight from global memory (lane (a,b)), then axis 1, then axis 0, whose outputs leave as
// coalesced stores (lanes consecutive along (b,c)).  Two barriers.
#pragma once
#include <hip/hip_runtime.h>

#include "tpo_pencil.hpp"
#include "tpo_pencil_mm.hpp"

namespace tpo {

template <typename T, int N, int G, int HINT, bool XCD, bool FWD, int SB>
__global__ void __launch_bounds__((PencilShape<T, N, G>::NT))
transform_pencil_kernel(KernelField<T, (SB & (FWD ? kHeldForward : kHeldBackward)) != 0> u_, const T *Sx_, const T *Sy_, const T *Sz_, T *t,
                        long long num_elems)
{
    using Sh = PencilShape<T, N, G>;
    constexpr int P = Sh::P, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *cube_all = reinterpret_cast<T *>(tpo_lds);

    const T *u = u_;
    const TPO_CONSTANT T *Sx = (const TPO_CONSTANT T *)Sx_;
    const TPO_CONSTANT T *Sy = (const TPO_CONSTANT T *)Sy_;
    const TPO_CONSTANT T *Sz = (const TPO_CONSTANT T *)Sz_;

    const int tid = threadIdx.x;
    const int g = tid / P;
    const int p = tid - g * P;
    const int hi = p / N;
    const int lo = p - hi * N;
    const long long nbatch = (num_elems + G - 1) / G;
    const long long batch = pencil_batch<XCD>(nbatch);
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const long long e = batch * G + g;
    const bool on = (tid < G * P) && (e < num_elems);
    T *cube = cube_all + (g < G ? g : 0) * CUBE;
    const size_t base = (size_t)(on ? e : 0) * (size_t)(N * N * N);

    T x[N], y[N];

    // axis 2: lane (a,b) = (hi,lo) owns u[a][b][0..n-1], contiguous in memory
    if (on) {
        load_words<(HINT & 1) != 0>(u + base + (size_t)(p * N), x);
        warm_scalar_cache<SB, N * N>(Sz, Sy, Sx);
        mode_product<T, N, FWD, SB>(Sz, x, y);
#pragma unroll
        for (int k = 0; k < N; ++k) cube[hi * PA + lo * PB + k] = y[k];
    }
    __syncthreads();

    // axis 1: lane (a,c) = (hi,lo)
    if (on) {
#pragma unroll
        for (int m = 0; m < N; ++m) x[m] = cube[hi * PA + m * PB + lo];
        mode_product<T, N, FWD, SB>(Sy, x, y);
#pragma unroll
        for (int j = 0; j < N; ++j) cube[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // axis 0: lane (b,c) = (hi,lo); stores are consecutive over lanes
    if (on) {
#pragma unroll
        for (int l = 0; l < N; ++l) x[l] = cube[l * PA + hi * PB + lo];
        mode_product<T, N, FWD, SB>(Sx, x, y);
#pragma unroll
        for (int i = 0; i < N; ++i) gstore<(HINT & 2) != 0>(t + base + (size_t)(i * P + p), y[i]);
    }
}

// fp32 form with the mode products issued as 4x4x1 matrix-core outer products (tpo_pencil_mm.hpp):
// same data movement, same order of the sums, bit-identical results.  The table of axis 2 goes
// straight into registers, those of axes 1 and 0 are built once per workgroup and parked in LDS
// until the barrier before their use.  Idle lanes shadow pencil 0 of the batch's first element and
// never store (the matrix instructions read their coefficients from active lanes).
// What bounds it: the vector-FMA form issues 3 n^2 FMAs of 4 cycles per pencil, half as many cycles
// here; what is left is the memory system (a plain copy in the same pieces runs at 5.75 TB/s).  On
// 3 GB, us per call against the vector-FMA form: n = 12 539 / 551, 13 538 / 555, 14 623 / 622, 15
// 593 / 627, 16 519 / 569; n = 8 485 / 483, 9 520 / 524, 10 568 / 548, 11 539 / 535.  While both
// fields stay in the last-level cache (256 MB) the cycles count for more, and n = 8 .. 11 gain
// too (150 MB: 22.1 / 23.7, 24.4 / 25.3, 26.8 / 28.2, 26.3 / 27.5; 40 MB: 5.2 / 6.2, 8.3 / 8.6, 9.3 /
// 10.1, 9.2 / 10.2; 600 MB: 96 / 89, 105 / 105, 116 / 110, 111 / 107); n = 4 .. 7 do not.
template <int N, int G, int HINT, bool XCD, bool FWD>
__global__ void __launch_bounds__((PencilShape<float, N, G>::NT))
__attribute__((amdgpu_waves_per_eu(mm_waves_per_simd<N>())))
transform_mm_kernel(const float *u, const float *__restrict__ Sx, const float *__restrict__ Sy,
                    const float *__restrict__ Sz, float *t, long long num_elems)
{
    using Sh = PencilShape<float, N, G>;
    using M = MmShape<N>;
    constexpr int P = Sh::P, PA = Sh::PA, PB = Sh::PB, CUBE = Sh::CUBE, N3 = N * N * N;
    constexpr int NWAVES = Sh::NT / 64, ROWS = 2 * M::NTAB, PER_WAVE = (ROWS + NWAVES - 1) / NWAVES;
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    float *cube_all = reinterpret_cast<float *>(tpo_lds);
    float *tabs = cube_all + G * CUBE;                  // [axis 1, axis 0][register][lane]

    const int tid = threadIdx.x, lane = tid & 63;
    const long long nbatch = (num_elems + G - 1) / G;
    const long long batch = pencil_batch<XCD>(nbatch);
    if (XCD && batch >= nbatch) return;                 // whole workgroup: no barrier is skipped
    const int g_ = tid / P;
    const bool on = (tid < G * P) && (batch * G + g_ < num_elems);
    const int g = on ? g_ : 0;
    const int p = on ? tid - g_ * P : 0;
    const int hi = p / N, lo = p - hi * N;
    float *cube = cube_all + g * CUBE;
    const size_t wg_base = (size_t)(batch * G) * (size_t)N3;

    float x[N], y[M::NY], tab[M::NTAB];

    // axis 2: lane (a,b) = (hi,lo) owns u[a][b][0..n-1], contiguous in memory
    // From n = 13 on u is asked for before the table (4 GB: n = 13 714 against 758 us, 14 816 / 859, 15 800
    // / 837; n = 12 735 / 724).
    constexpr bool U_FIRST = N >= 13;
    auto load_u = [&]() { load_words<(HINT & 1) != 0>(u + wg_base + (unsigned)(g * N3 + p * N), x); };
    if constexpr (U_FIRST) {
        load_u();
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < M::NTAB; ++r) tab[r] = mm_coef<N>(Sz, FWD, r, lane);
    if constexpr (!U_FIRST) load_u();
    {
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        float val[PER_WAVE];
#pragma unroll
        for (int k = 0; k < PER_WAVE; ++k) {
            const int r = wave + k * NWAVES < ROWS ? wave + k * NWAVES : ROWS - 1;
            val[k] = r < M::NTAB ? mm_coef<N>(Sy, FWD, r, lane) : mm_coef<N>(Sx, FWD, r - M::NTAB, lane);
        }
#pragma unroll
        for (int k = 0; k < PER_WAVE; ++k) {
            const int r = wave + k * NWAVES < ROWS ? wave + k * NWAVES : ROWS - 1;
            tabs[r * 64 + lane] = val[k];
        }
    }
    mode_product_mm<N, FWD>(tab, (const TPO_CONSTANT float *)Sz, x, y);
    if (on) {
#pragma unroll
        for (int k = 0; k < N; ++k) cube[hi * PA + lo * PB + k] = y[k];
    }
    __syncthreads();

    // axis 1: lane (a,c) = (hi,lo)
    mm_fetch_table<N>(tabs, 1, lane, tab);
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = cube[hi * PA + m * PB + lo];
    mode_product_mm<N, FWD>(tab, (const TPO_CONSTANT float *)Sy, x, y);
    if (on) {
#pragma unroll
        for (int j = 0; j < N; ++j) cube[hi * PA + j * PB + lo] = y[j];
    }
    __syncthreads();

    // axis 0: lane (b,c) = (hi,lo); stores are consecutive over lanes
    mm_fetch_table<N>(tabs, 2, lane, tab);
#pragma unroll
    for (int l = 0; l < N; ++l) x[l] = cube[l * PA + hi * PB + lo];
    mode_product_mm<N, FWD>(tab, (const TPO_CONSTANT float *)Sx, x, y);
    if (on) {
        float *tb = t + wg_base + (unsigned)(g * N3 + p);
#pragma unroll
        for (int i = 0; i < N; ++i) gstore<(HINT & 2) != 0>(tb + i * P, y[i]);
    }
}

// Elements per workgroup and die renumbering as for the separable-diagonal operator kernels
// (same traffic: one field in, one out); cached loads, since each lane's n-word run shares its
// cache lines with its neighbours' runs.  The matrix-core form has its own rows: the best of 1 .. 3
// elements per workgroup x non-temporal stores x renumbering (swept before the coefficient tables took their
// present layout and u went first from n = 13 on; the settings were not swept again).
template <typename T, int N> struct TransformTune {
    using Tune = PencilSepTune<T, N>;
    static constexpr int G = Tune::G, HINT = Tune::HINT & 2;
    static constexpr bool XCD = Tune::XCD, MM = false;
    static constexpr int SB = kScalarBatch;
    static constexpr long long FROM = kPencilCachedBytes;       // of the settings for large batches
};
template <int GG, int H, bool X, bool M, long long MB = 256, int S = kScalarBatch> struct TransformSet {
    static constexpr int G = GG, HINT = H, SB = S;
    static constexpr bool XCD = X, MM = M;
    static constexpr long long FROM = MB << 20;
};
template <typename T> struct TransformTune<T, 2> : TransformSet<16, 0, false, false> {};
template <> struct TransformTune<float, 13> : TransformSet<3, 0, true, true> {};
template <> struct TransformTune<float, 14> : TransformSet<2, 0, false, true> {};
template <> struct TransformTune<float, 15> : TransformSet<1, 0, false, true> {};
template <> struct TransformTune<float, 16> : TransformSet<1, 2, false, true> {};
// While both fields stay in the last-level cache: the matrix-core form from n = 8 on.
template <> struct TransformTune<float, 8> : TransformSet<2, 2, false, true> {};
template <> struct TransformTune<float, 9> : TransformSet<3, 0, false, true> {};
template <> struct TransformTune<float, 10> : TransformSet<2, 0, false, true> {};
template <> struct TransformTune<float, 11> : TransformSet<2, 0, false, true> {};
// Beyond: the vector-FMA form for those, and settings from a sweep over 1 .. 32 elements per workgroup
// x stores x renumbering on 2 GB per call where it found 4 % or more (us per call on 2.5
// GB, before / now): fp64 n = 3 460 / 434, 4 427 / 384, 7 452 / 427, 9 450 / 433, 10 476 / 439, 12 454 /
// 435, 13 480 / 450; fp32 n = 3 569 / 531, 5 491 / 450.  Some begin later, in MiB: fp64 n = 7, 10 only past 1 GB
// (600 MB 101 / 108, 110 / 114), 9 too (340 .. 500 MB 1.01 .. 1.04 of the time), 13 at 512 (275 .. 430 MB 0.99 .. 1.03), 3 at 272
// (275 MB 1.05 .. 1.08, 290 MB 0.92).  Where the rows by batch size go further (n = 7, 10, 13) these sizes decide nothing.
// fp32 n = 12, matrix-core form: non-temporal stores leave the cache to the input until the fields are well
// past it (time over the vector-FMA form's with / without, forward: 60 MB 0.78 / 1.02, 100 MB 0.79 / 0.83, 290 MB 0.91 /
// 1.01 .. 1.07, 380 MB 0.91 / 1.05 .. 1.09, 600 MB 0.91 / 0.94, 1.2 GB 0.97 / 0.92; backward 290 MB 0.80 / 0.98).
template <typename T, int N> struct TransformLargeTune : TransformTune<T, N> {};
template <int N> struct TransformVectorTune {
    using Tune = PencilSepTune<float, N>;
    static constexpr int G = Tune::G, HINT = Tune::HINT & 2;
    static constexpr bool XCD = Tune::XCD, MM = false;
    static constexpr int SB = kScalarBatch;
    static constexpr long long FROM = kPencilCachedBytes;
};
template <> struct TransformLargeTune<float, 8> : TransformVectorTune<8> {};
template <> struct TransformLargeTune<float, 9> : TransformVectorTune<9> {};
template <> struct TransformLargeTune<float, 10> : TransformVectorTune<10> {};
template <> struct TransformLargeTune<float, 11> : TransformVectorTune<11> {};
template <> struct TransformLargeTune<float, 3> : TransformSet<24, 2, false, false> {};
template <> struct TransformLargeTune<float, 5> : TransformSet<2, 0, true, false> {};
template <> struct TransformLargeTune<float, 12> : TransformSet<3, 0, true, true, 640> {};
template <> struct TransformLargeTune<double, 3> : TransformSet<24, 0, true, false, 272> {};
template <> struct TransformLargeTune<double, 4> : TransformSet<2, 2, false, false> {};
template <> struct TransformLargeTune<double, 7> : TransformSet<6, 0, true, false, 1024> {};
template <> struct TransformLargeTune<double, 9> : TransformSet<4, 0, true, false, 1024> {};
template <> struct TransformLargeTune<double, 10> : TransformSet<3, 0, true, false, 1024> {};
template <> struct TransformLargeTune<double, 12> : TransformSet<2, 2, true, false> {};
template <> struct TransformLargeTune<double, 13> : TransformSet<2, 0, true, false, 512> {};

template <typename T, int N, bool FWD, typename Tune>
struct TransformLauncherT {
    static constexpr int G = Tune::G;
    using Sh = PencilShape<T, N, G>;
    static constexpr size_t LDS = Sh::LDS_BYTES / 2 + (Tune::MM ? 2 * MmShape<N>::NTAB * 256 : 0);
    static constexpr int CODE = setting_code(G, Tune::HINT, Tune::XCD, Tune::MM, Tune::MM ? 0 : Tune::SB);

    static constexpr auto kernel()
    {
        if constexpr (Tune::MM) return &transform_mm_kernel<N, G, Tune::HINT, Tune::XCD, FWD>;
        else return &transform_pencil_kernel<T, N, G, Tune::HINT, Tune::XCD, FWD, Tune::SB>;
    }
    using Field = KernelField<T, !Tune::MM && (Tune::SB & (FWD ? kHeldForward : kHeldBackward)) != 0>;

    static hipError_t launch(const TransformArgs &a)
    {
        const long long blocks = pencil_grid<Tune::XCD>((a.num_elems + G - 1) / G);
        if (blocks <= 0 || blocks > 0x7fffffffLL) return kGridTooLarge;
        drop_stale_error();
        hipLaunchKernelGGL(kernel(), dim3((unsigned)blocks), dim3(Sh::NT), LDS, a.stream,
                           kernel_field<Field>((const T *)a.u), (const T *)a.sx, (const T *)a.sy, (const T *)a.sz,
                           (T *)a.t, a.num_elems);
        return hipGetLastError();
    }

    static hipError_t prepare()
    {
        if (LDS <= 48 * 1024) return hipSuccess;
        return hipFuncSetAttribute((const void *)kernel(),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS);
    }
};

template <typename T, int N, bool FWD>
struct TransformLauncher {
    using Large = TransformLauncherT<T, N, FWD, TransformLargeTune<T, N>>;
    using Cached = std::conditional_t<((long long)batch_rows_end(TransformRows<T>::rows, N) << 20) >= TransformLargeTune<T, N>::FROM, Large,
                                      TransformLauncherT<T, N, FWD, TransformTune<T, N>>>;
    template <int K> using Row = TransformLauncherT<T, N, FWD, BatchTune<TransformRows<T>::rows, N, K>>;
    static constexpr long long BYTES = 2LL * N * N * N * (long long)sizeof(T);
    // f(Use<the launcher of the setting that a batch takes>)
    template <typename F>
    static void with_setting(long long num_elems, F &&f)
    {
        if (for_batch_row<TransformRows<T>::rows, N>(num_elems, BYTES, [&](auto k) { f(Use<Row<decltype(k)::value>>{}); })) return;
        if (takes_large(num_elems)) f(Use<Large>{});
        else f(Use<Cached>{});
    }
    static hipError_t launch(const TransformArgs &a)
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
    static bool takes_large(long long num_elems) { return num_elems > TransformLargeTune<T, N>::FROM / BYTES; }
    static hipError_t prepare()
    {
        hipError_t rc = Cached::prepare();
        if (rc == hipSuccess) rc = Large::prepare();
        for_each_batch_row<TransformRows<T>::rows, N>([&](auto k) {
            if (rc == hipSuccess) rc = Row<decltype(k)::value>::prepare();
        });
        return rc;
    }
};

#define TPO_TRANSFORM_ENTRY(T, N)                                                          \
    TransformEntry { &TransformLauncher<T, N, true>::launch, &TransformLauncher<T, N, false>::launch, \
                     &TransformLauncher<T, N, true>::prepare, &TransformLauncher<T, N, false>::prepare,   \
                     &TransformLauncher<T, N, true>::setting }

}  // namespace tpo
