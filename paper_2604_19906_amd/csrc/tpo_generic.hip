// Kernel of the inverse-Helmholtz operator for anisotropic elements: nx, ny, nz points along
// axes 0, 1, 2, all runtime values in 1 .. 16.  It stands behind tpo_ihelm_apply_aniso for the
// shapes that are not cubic (cubic shapes go to the tuned families), except the fp32 calls for which
// slice_kernel_pays() chooses the slice kernel (tpo_slice_f32.hip).
//
// Same scheme as the pencil kernels: a workgroup takes g whole elements, the cube lives in LDS,
// every lane owns one pencil per mode product, the matrix entries arrive in SGPRs.  What makes
// it work for runtime sizes is that a mode product only needs the size of ITS axis at compile
// time (for the unrolled FMAs and the batched scalar loads of the matrix); the other two sizes
// only enter pencil counts and strides, which may be runtime values.  So every product is a
// uniform switch over the size of its axis, and the kernel is compiled once per size class
// (largest of the three sizes at most 4, 8, 12 or 16, in fp64 also 10, in fp32 6: the class bounds the registers; with
// the class of 10 fp64 shapes of 9 and 10 points keep six wavefronts per SIMD instead of five, 0.94 .. 0.98 of
// the time; a class of 14 changes nothing, four wavefronts per SIMD either way, and five cost spills, 1.05 .. 1.20).
//
// Order of the products, as in the pencil kernels: axis 0 first, on words read coalesced from
// u_e (for a fixed index along axis 0 the lanes of that pass are consecutive words), axis 1,
// then axis 2 forward, the scale and axis 2 backward on the lane's registers (each lane asked
// for the nz consecutive words of D_e it needs when the kernel started), axis 1, and axis 0
// last, stored coalesced to v_e.  Four barriers.
//
// What the runtime sizes cost is integer work: divisions (20 instructions, five of them at a quarter of the rate) for the place of a
// lane in each pass, 64-bit address sums per word, and products for LDS addresses, 20 .. 40 % of a wavefront's vector
// instructions with three axes of 5 .. 7 points, 16 .. 23 % at 8 .. 16.  They are reciprocals in 24 bits, one uniform base that moves
// along the axis with a 32-bit offset per lane, and one addition per LDS word now; the stores leave in ascending order, which
// the 128-byte lines that two of them share need (in the compiler's order fp32 (5,5,6) wrote 1.20 of its bytes at 2.4 GB).  Time over
// the kernels before, arguments in scalar registers and cached stores included, geometric means over 120 shapes per type at 1 / 8 / 24 / 60 / 100 /
// 300 MB / 1 / 2.4 GB: fp64 .91 .90 .88 .91 .90 .88 .89 .89 (one turn), turns .90 .. .92 from 100 MB on; fp32 .90 .84 .83 .88 .87 .85 .88
// .88, turns .89 .. .90.  One of 1920 calls is slower by more than 2 % (fp64 (2,2,6) at 300 MB, 1.04).  Vector registers fall by 2 .. 8, scalars
// spilled to them rise in some classes: one turn fp64 class 12 from none to 16, 16 from 6 to 12; in turns fp64 class 14 from 61 to 72, fp32 class
// 10 from 19 to 30, the others fall or stay.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tpo_internal.h"
#include "tpo_pencil.hpp"

namespace tpo {

namespace {

constexpr int ANISO_MAX_NT = 256;
constexpr int kMaxPencils = TPO_MAX_N * TPO_MAX_N;          // of one element in one pass
constexpr size_t kTurnsLds = 48 * 1024;                     // of a workgroup of the turns kernel, at most
// Hints and die renumbering: non-temporal stores of v_e and workgroups renumbered per die, or (STREAM) non-temporal
// loads of u_e as well and no renumbering.  STREAM over the other in fp64, geometric means over 120 shapes: 0.93 at 52 and 60 MB,
// 0.98 at 150, 0.96 at 300, 0.97 at 800 MB; 1.00 .. 1.02 with maxima of 1.09 at 100 and 130 MB (fields that the
// last-level cache holds in part) and at 2.5 GB, 1.0 .. 1.1 at 30 MB, up to 1.07 on elements of less than 128 points and at 50 MB
// of less than 300.  In fp32 1.00, up to 1.24 on faces of a dozen points: not there.
// CACHED: v_e stored without the hint.  Thin faces that fill no whole 128-byte lines (below 192 bytes): the stores of two indices along axis 0
// share most lines, and past the last-level cache the hint writes a line out before its second part comes.  But stores without it take the
// cache from what the next call on the same fields finds there: all three fields up to 256 MiB of them, u_e and D_e up to 384, D_e alone up to
// 768 where u_e is streamed.  Cached over non-temporal, the same fields / three sets in turn, 14 sizes from 200 MB to 2.4 GB.
// fp64 in turns (35 shapes), u_e streamed: 340 and 400 MB 0.85 .. 1.01 / 0.86 .. 1.02, from 850 MB on 0.79 .. 1.02 / 0.80 .. 1.02; 430 .. 700 MB faces
// of 9 and 15 words 0.90 .. 1.04 / 0.88 .. 0.93, 8, 10 and 12 .. 14 0.91 .. 1.10 / 0.86 .. 0.99, 18 .. 22 0.97 .. 1.14 / 0.92 .. 1.02; not
// streamed: 340 and 400 MB 1.01 .. 1.14 / 0.85 .. 1.00 ((12,10,1), (8,1,14)), from 460 MB on 0.84 .. 1.01 / 0.83 .. 1.01.  Faces of 16 and 24
// words 1.00 .. 1.08.
// One turn, fp64, elements of at most eight points along every axis and of less than 128 in all (24 shapes): 250 MB 0.89 .. 1.01 / 0.95 .. 1.01, 280
// .. 430 MB 0.99 .. 1.45 / 0.91 .. 1.01, from 460 MB on 0.92 .. 1.02 / 0.91 .. 1.01; faces of 8 and 16 words 1.00 .. 1.06, 1.02 with one or two
// points along axis 0.  fp32, at most six points along every axis (19 shapes): 200 and 250 MB 0.88 .. 1.02 / 0.87 .. 1.00, 280 .. 400 MB 1.19 .. 1.51 /
// 0.79 .. 1.00, from 430 MB on 0.83 .. 1.02 / 0.84 .. 1.00; faces of 8, 12 and 16 words 1.01 .. 1.03, in turns 0.93 .. 1.07.
constexpr int aniso_hint(bool stream, bool cached) { return (stream ? 1 : 0) | (cached ? 0 : 2); }
constexpr bool aniso_xcd(bool stream) { return !stream; }
template <typename T>
bool aniso_stream(const AnisoArgs &a, bool turns)
{
    const int points = a.nx * a.ny * a.nz;
    const long long mib = 3LL * a.num_elems * points * (long long)sizeof(T) >> 20;
    if (sizeof(T) == 4) return false;
    if (!turns && mib >= 48 && mib < 80) return points >= 300;
    return points >= 128 && mib >= 144 && mib < 1536;
}
template <typename T>
bool aniso_cached_stores(const AnisoArgs &a, bool turns)
{
    const int face = a.ny * a.nz, points = a.nx * face;
    const long long mib = 3LL * a.num_elems * points * (long long)sizeof(T) >> 20;
    const auto all_up_to = [&](int n) { return a.nx <= n && a.ny <= n && a.nz <= n; };
    if (sizeof(T) == 4)
        return !turns && a.nx >= 3 && a.ny > 1 && a.nz > 1 && all_up_to(6) && face < 12 && face % 4 != 0
               && ((mib >= 184 && mib < 244) || mib >= 408);
    if (turns) {
        if (face >= 24 || face == 16 || mib < 320) return false;
        if (!aniso_stream<T>(a, true)) return mib >= 440;
        return mib < 384 || mib >= 784 || face == 9 || face == 15;
    }
    return a.nx >= 3 && all_up_to(8) && !all_up_to(4) && points < 128 && face < 24 && face % 8 != 0
           && ((mib >= 224 && mib < 244) || mib >= 440);
}

// f(integral_constant<int, n>) for the runtime n in 1 .. MAXN (uniform over the workgroup).
template <int MAXN, typename F>
__device__ __forceinline__ void dispatch_size(int n, F &&f)
{
#define TPO_SIZE_CASE(K)                                                       \
    case K:                                                                    \
        if constexpr (K <= MAXN) f(std::integral_constant<int, K>{});          \
        break;
    switch (n) {
        TPO_SIZE_CASE(1) TPO_SIZE_CASE(2) TPO_SIZE_CASE(3) TPO_SIZE_CASE(4)
        TPO_SIZE_CASE(5) TPO_SIZE_CASE(6) TPO_SIZE_CASE(7) TPO_SIZE_CASE(8)
        TPO_SIZE_CASE(9) TPO_SIZE_CASE(10) TPO_SIZE_CASE(11) TPO_SIZE_CASE(12)
        TPO_SIZE_CASE(13) TPO_SIZE_CASE(14) TPO_SIZE_CASE(15) TPO_SIZE_CASE(16)
    default: break;
    }
#undef TPO_SIZE_CASE
}

// LDS pitches: odd row pitch and odd plane pitch (in words) against bank conflicts.
__host__ __device__ inline int aniso_pz(int nz) { return nz | 1; }
__host__ __device__ inline int aniso_pyz(int ny, int nz) { return (ny * aniso_pz(nz)) | 1; }

// a * b and a * b + c for a, b < 2^24, b uniform: one instruction at the full rate.  Left to itself the compiler takes
// 32-bit products (a quarter of the rate) where it cannot see the bounds.
__device__ __forceinline__ unsigned mul24(unsigned a, unsigned b)
{
    unsigned r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "s"(b), "v"(a));
    return r;
}
__device__ __forceinline__ unsigned mad24(unsigned a, unsigned b, unsigned c)
{
    unsigned r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// Upper 32 bits of a * b.
__device__ __forceinline__ unsigned mulhi24(unsigned a, unsigned b)
{
    unsigned r;
    asm("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(r) : "s"(b), "v"(a));
    return r;
}

// N words of LDS a runtime number of bytes apart, from byte address `at` on.  The address moves by one addition per word;
// opaque, since the compiler would rather multiply (v_mad_u64_u32, a quarter of the rate) than keep the chain.
typedef __attribute__((address_space(3))) unsigned char lds_byte;
template <typename T, int N, typename F>
__device__ __forceinline__ void each_word(unsigned at, unsigned step, F &&f)
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        f(i, *reinterpret_cast<__attribute__((address_space(3))) T *>(reinterpret_cast<lds_byte *>(at)));
        at += step;
        asm("" : "+v"(at));
    }
}
template <typename T, int N>
__device__ __forceinline__ void lds_read(unsigned at, unsigned step, T (&x)[N])
{
    each_word<T, N>(at, step, [&](int i, const __attribute__((address_space(3))) T &w) { x[i] = w; });
}
template <typename T, int N>
__device__ __forceinline__ void lds_write(unsigned at, unsigned step, const T (&x)[N])
{
    each_word<T, N>(at, step, [&](int i, __attribute__((address_space(3))) T &w) { w = x[i]; });
}
__device__ __forceinline__ unsigned lds_address(const void *p)
{
    return (unsigned)(unsigned long long)reinterpret_cast<const lds_byte *>((const __attribute__((address_space(3))) void *)p);
}

// A uniform value as it stands in a scalar register (k * NT + lane would become a v_mad_u64_u32).
__device__ __forceinline__ unsigned scalar(unsigned s)
{
    asm("" : "+s"(s));
    return s;
}

// N words of HBM a runtime number of bytes apart: the uniform base moves (scalar additions, kept next to their access: hoisted
// out of the turns they spill), the lane's 32-bit offset stays.  The base has to be a pointer to global memory by its type: behind
// the asm the compiler no longer sees where a generic one came from and takes FLAT accesses, which have no form with a scalar base (a 64-bit sum
// per word) and are waited for together with LDS and scalar loads (a product waits for its last word before it starts on the first):
// 1.01 .. 1.03 of the time, geometric means over 75 shapes per type at 1 MB .. 2.4 GB.
typedef __attribute__((address_space(1))) char global_byte;
template <bool NT, typename T, int N>
__device__ __forceinline__ void global_read(const global_byte *base, unsigned step, unsigned off, T (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto *p = reinterpret_cast<const __attribute__((address_space(1))) T *>(base + off);
        if constexpr (NT) x[i] = __builtin_nontemporal_load(p);
        else x[i] = *p;
        base += step;
        asm("" : "+s"(base));
    }
}
template <bool NT, typename T, int N>
__device__ __forceinline__ void global_write(global_byte *base, unsigned step, unsigned off, const T (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        auto *p = reinterpret_cast<__attribute__((address_space(1))) T *>(base + off);
        if constexpr (NT) __builtin_nontemporal_store(x[i], p);
        else *p = x[i];
        base += step;
        asm("" : "+s"(base));
    }
}

// Arguments of a call's shape, one word each so that the kernel finds them in scalar registers when it starts (the build has the
// first 14 words of the arguments preloaded; a struct is not): the three sizes in one word, the elements per workgroup, and
// reciprocals of the pencil counts of the passes and of two sizes.  (At most 2^31 - 1 elements.)
#define TPO_ANISO_SHAPE unsigned num_elems, unsigned groups, unsigned sizes, unsigned g, \
                        unsigned by_yz, unsigned by_xz, unsigned by_xy, unsigned by_y, unsigned by_z
constexpr unsigned packed_sizes(int nx, int ny, int nz) { return (unsigned)(nx | ny << 8 | nz << 16); }
template <bool XCD>
__device__ __forceinline__ unsigned aniso_batch(unsigned groups)        // pencil_batch in 32 bits
{
    return XCD ? (blockIdx.x & 7) * ((groups + 7) / 8) + (blockIdx.x >> 3) : blockIdx.x;
}

constexpr unsigned lane_reciprocal(int d) { return (65536u + d - 1) / d; }
// t / d for a lane t and d pencils, m = lane_reciprocal(d): m d exceeds 65536 by r < d, so t m / 65536 exceeds t / d by less than
// 1 / d while t r < 65536.
constexpr bool lane_reciprocals_exact()
{
    for (unsigned d = 1; d <= kMaxPencils; ++d)
        for (unsigned t = 0; t < ANISO_MAX_NT; ++t)
            if (t * lane_reciprocal((int)d) >> 16 != t / d) return false;
    return true;
}
static_assert(lane_reciprocals_exact());
__device__ __forceinline__ unsigned lane_quotient(unsigned t, unsigned m) { return mul24(t, m) >> 16; }

// HINT bits as in the pencil kernels: 1 non-temporal loads of u_e, 2 non-temporal stores of v_e,
// 4 non-temporal loads of D_e.  XCD: workgroups renumbered per accelerator die (the grid must be
// pencil_grid<XCD>(number of groups)).
template <typename T, int MAXN, int HINT, bool XCD>
__global__ void __launch_bounds__(ANISO_MAX_NT)
ihelm_aniso_kernel(const T *u, const T *__restrict__ D, TPO_ANISO_SHAPE,
                   const T *Sx_, const T *Sy_, const T *Sz_, T *v)
{
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *cube = reinterpret_cast<T *>(tpo_lds);
    const TPO_CONSTANT T *Sx = (const TPO_CONSTANT T *)Sx_;
    const TPO_CONSTANT T *Sy = (const TPO_CONSTANT T *)Sy_;
    const TPO_CONSTANT T *Sz = (const TPO_CONSTANT T *)Sz_;
    const int nx = sizes & 255, ny = sizes >> 8 & 255, nz = sizes >> 16;

    const unsigned tid = threadIdx.x;
    const unsigned batch = aniso_batch<XCD>(groups);
    if (batch >= groups) return;                           // padding workgroup of the renumbering
    const unsigned e0 = batch * g, left = num_elems - e0;
    const unsigned here = left < g ? left : g;             // elements of this workgroup
    const unsigned pz = aniso_pz(nz), pyz = aniso_pyz(ny, nz);
    const unsigned cube_words = nx * pyz, face = ny * nz, total = nx * face;
    // addresses in HBM: one base per workgroup and index along the axis (uniform) plus a 32-bit byte offset per lane
    constexpr unsigned W = sizeof(T);
    const global_byte *ub = (const global_byte *)(u + (size_t)e0 * total);
    const char *db = reinterpret_cast<const char *>(D + (size_t)e0 * total);
    global_byte *vb = (global_byte *)(v + (size_t)e0 * total);

    // the lane's place in a pass with `pencils` pencils per element: element ge, pencil p
    auto place = [&](unsigned pencils, unsigned by, unsigned &ge, unsigned &p) {
        ge = lane_quotient(tid, by);
        p = tid - mul24(ge, pencils);
        return ge < here;
    };

    unsigned ge2, p2;
    const bool act2 = place(nx * ny, by_xy, ge2, p2);    // lane (a, b): a pencil along axis 2
    // D_e in the layout of the axis-2 pass, asked for before anything else
    T dreg[MAXN];
    if (act2)
        dispatch_size<MAXN>(nz, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T t[N];
            const unsigned off = mad24(ge2, total, mul24(p2, N)) * W;
            load_words<(HINT & 4) != 0, T, N>(reinterpret_cast<const T *>(db + off), t);
#pragma unroll
            for (int k = 0; k < N; ++k) dreg[k] = t[k];
        });
    const unsigned a2 = lane_quotient(p2, by_y), b2 = p2 - mul24(a2, ny);
    T *row2 = cube + mad24(ge2, cube_words, mad24(a2, pyz, mul24(b2, pz)));

    unsigned ge1, p1;
    const bool act1 = place(nx * nz, by_xz, ge1, p1);    // lane (a, c): a pencil along axis 1
    const unsigned a1 = lane_quotient(p1, by_z), c1 = p1 - mul24(a1, nz);
    const unsigned col1 = lds_address(cube) + mad24(ge1, cube_words, mad24(a1, pyz, c1)) * W, step1 = pz * W;

    unsigned ge0, p0;
    const bool act0 = place(face, by_yz, ge0, p0);       // lane (b, c): a pencil along axis 0
    const unsigned b0 = lane_quotient(p0, by_z);
    const unsigned col0 = lds_address(cube) + mad24(ge0, cube_words, mad24(b0, pz - nz, p0)) * W, step0 = pyz * W;
    const unsigned off0 = mad24(ge0, total, p0) * W, face_bytes = face * W;

    // forward, axis 0, from global memory
    if (act0)
        dispatch_size<MAXN>(nx, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T x[N], y[N];
            global_read<(HINT & 1) != 0>(ub, face_bytes, off0, x);
            mode_product<T, N, true>(Sx, x, y);
            lds_write(col0, step0, y);
        });
    __syncthreads();
    // forward, axis 1, in place
    if (act1)
        dispatch_size<MAXN>(ny, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T x[N], y[N];
            lds_read(col1, step1, x);
            mode_product<T, N, true>(Sy, x, y);
            lds_write(col1, step1, y);
        });
    __syncthreads();
    // axis 2: forward, scale by D_e, backward, in place
    if (act2)
        dispatch_size<MAXN>(nz, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T x[N], y[N];
#pragma unroll
            for (int k = 0; k < N; ++k) x[k] = row2[k];
            mode_product<T, N, true>(Sz, x, y);
#pragma unroll
            for (int k = 0; k < N; ++k) y[k] *= dreg[k];
            mode_product<T, N, false>(Sz, y, x);
#pragma unroll
            for (int k = 0; k < N; ++k) row2[k] = x[k];
        });
    __syncthreads();
    // backward, axis 1, in place
    if (act1)
        dispatch_size<MAXN>(ny, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T x[N], y[N];
            lds_read(col1, step1, x);
            mode_product<T, N, false>(Sy, x, y);
            lds_write(col1, step1, y);
        });
    __syncthreads();
    // backward, axis 0, to global memory
    if (act0)
        dispatch_size<MAXN>(nx, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            T x[N], y[N];
            lds_read(col0, step0, x);
            mode_product<T, N, false>(Sx, x, y);
            global_write<(HINT & 2) != 0>(vb, face_bytes, off0, y);
        });
}

// The same passes with more elements per workgroup than its lanes can hold pencils: a pass runs in turns of
// one pencil per lane.  For shapes whose passes differ much in their number of pencils: there the kernel
// above sizes the workgroup by the largest pass, and in the others most of the lanes idle.  What bounds it then is
// the loads: u_e and D_e are asked for by few lanes, so few bytes are on their way (fp64 (3,9,16) 34 KB per CU against
// 216 KB here).  us per call on 800 MB, kernel above / this one: fp64 (3,9,16) 329 / 155, (16,9,3) 279 / 157, (13,3,12)
// 267 / 157, (10,7,13) 192 / 161; fp32 (3,9,15) 438 / 184, (14,4,3) 279 / 190, (8,15,6) 225 / 189 (both since 5 .. 10 % faster).
// With one turn per pass it is the slower one by 3 .. 15 % (quotients, loops).
// t / d for t < 2^15 (24 bits hold t << 9) and d pencils, with m = turn_reciprocal(d): m d exceeds 2^23 by r < d, so t m / 2^23 exceeds
// t / d by less than 1 / d while t r < 2^23.  A workgroup's pencils are fewer than its words in LDS.
constexpr unsigned turn_reciprocal(int d) { return ((1u << 23) + d - 1) / d; }
constexpr bool turn_reciprocals_exact()
{
    // the excess grows with t and shows first on the word before a multiple of d: the last such word, and the multiple
    constexpr unsigned long long words = kTurnsLds / sizeof(float);
    for (unsigned long long d = 1; d <= kMaxPencils; ++d)
        for (unsigned long long q = words / d, t = q * d - 1; t <= q * d; ++t)
            if (((t << 9) * turn_reciprocal((int)d)) >> 32 != t / d || (t << 9) >> 24 != 0 || turn_reciprocal((int)d) >> 24 != 0) return false;
    return true;
}
static_assert(turn_reciprocals_exact());
__device__ __forceinline__ unsigned quotient(unsigned t, unsigned m) { return mulhi24(t << 9, m); }

template <typename T, int MAXN, int HINT, bool XCD>
__global__ void __launch_bounds__(ANISO_MAX_NT)
ihelm_aniso_turns_kernel(const T *u, const T *__restrict__ D, TPO_ANISO_SHAPE,
                         const T *Sx_, const T *Sy_, const T *Sz_, T *v)
{
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    T *cube = reinterpret_cast<T *>(tpo_lds);
    const TPO_CONSTANT T *Sx = (const TPO_CONSTANT T *)Sx_;
    const TPO_CONSTANT T *Sy = (const TPO_CONSTANT T *)Sy_;
    const TPO_CONSTANT T *Sz = (const TPO_CONSTANT T *)Sz_;
    const int nx = sizes & 255, ny = sizes >> 8 & 255, nz = sizes >> 16;

    const unsigned tid = threadIdx.x;
    const unsigned NT = blockDim.x;
    const unsigned batch = aniso_batch<XCD>(groups);
    if (batch >= groups) return;                           // padding workgroup of the renumbering
    const unsigned e0 = batch * g, left = num_elems - e0;
    const unsigned here = left < g ? left : g;             // elements of this workgroup
    const unsigned pz = aniso_pz(nz), pyz = aniso_pyz(ny, nz);
    const unsigned cube_words = nx * pyz;
    const unsigned face = ny * nz, side = nx * nz, base = nx * ny, total = nx * face;
    constexpr unsigned W = sizeof(T);
    const global_byte *ub = (const global_byte *)(u + (size_t)e0 * total);
    const char *db = reinterpret_cast<const char *>(D + (size_t)e0 * total);
    global_byte *vb = (global_byte *)(v + (size_t)e0 * total);
    const unsigned lds = lds_address(cube), step0 = pyz * W, step1 = pz * W, face_bytes = face * W;

    // Pencil t of a pass with `limit` of them goes to lane t % NT in turn t / NT; the wavefront takes part in a
    // turn if its first lane has a pencil, lanes past the end shadow the last one and do not store.
    const unsigned first = __builtin_amdgcn_readfirstlane(tid & ~63u);
    // LDS address of pencil (b, c) along axis 0 and of pencil (a, c) along axis 1
    auto column0 = [&](unsigned q, unsigned p) {
        return lds + mad24(q, cube_words, mad24(quotient(p, by_z), pz - nz, p)) * W;
    };
    auto column1 = [&](unsigned q, unsigned p) {            // p = a nz + c: a pyz + c
        return lds + mad24(q, cube_words, mad24(quotient(p, by_z), pyz - nz, p)) * W;
    };

    // D_e in the layout of the axis-2 pass (pencils (a, b), nz consecutive words), asked for before anything else
    T dreg[MAXN];
    dispatch_size<MAXN>(nz, [&](auto nc) {
        constexpr int N = decltype(nc)::value, K = MAXN / N;
        const unsigned limit = here * base;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const unsigned turn = scalar(k * NT);
            if (first + turn < limit) {
                const unsigned t = min(tid + turn, limit - 1);
                T w[N];
                load_words<(HINT & 4) != 0, T, N>(reinterpret_cast<const T *>(db + mul24(t, N * W)), w);
#pragma unroll
                for (int i = 0; i < N; ++i) dreg[k * N + i] = w[i];
            }
        }
    });

    // forward, axis 0, from global memory: pencils (b, c)
    dispatch_size<MAXN>(nx, [&](auto nc) {
        constexpr int N = decltype(nc)::value, K = MAXN / N;
        const unsigned limit = here * face;
        T x[K][N];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const unsigned turn = scalar(k * NT);
            if (first + turn < limit) {
                const unsigned t = min(tid + turn, limit - 1);
                const unsigned off = mad24(quotient(t, by_yz), total - face, t) * W;
                global_read<(HINT & 1) != 0>(ub, face_bytes, off, x[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const unsigned t = tid + scalar(k * NT);
            if (t < limit) {
                const unsigned q = quotient(t, by_yz);
                T y[N];
                mode_product<T, N, true>(Sx, x[k], y);
                lds_write(column0(q, t - mul24(q, face)), step0, y);
            }
        }
    });
    __syncthreads();
    // axis 1, in place: pencils (a, c)
    auto axis1 = [&](auto fwd) {
        dispatch_size<MAXN>(ny, [&](auto nc) {
            constexpr int N = decltype(nc)::value;
            for (unsigned t = tid; t < here * side; t += NT) {
                const unsigned q = quotient(t, by_xz), at = column1(q, t - mul24(q, side));
                T x[N], y[N];
                lds_read(at, step1, x);
                mode_product<T, N, decltype(fwd)::value>(Sy, x, y);
                lds_write(at, step1, y);
            }
        });
    };
    axis1(std::integral_constant<bool, true>{});
    __syncthreads();
    // axis 2 forward, scale, axis 2 backward, in place
    dispatch_size<MAXN>(nz, [&](auto nc) {
        constexpr int N = decltype(nc)::value, K = MAXN / N;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const unsigned t = tid + scalar(k * NT);
            if (t < here * base) {
                const unsigned q = quotient(t, by_xy), p = t - mul24(q, base);
                const unsigned a = quotient(p, by_y), b = p - mul24(a, ny);
                T *row = cube + mad24(q, cube_words, mad24(a, pyz, mul24(b, pz)));
                T x[N], y[N];
#pragma unroll
                for (int i = 0; i < N; ++i) x[i] = row[i];
                mode_product<T, N, true>(Sz, x, y);
#pragma unroll
                for (int i = 0; i < N; ++i) y[i] *= dreg[k * N + i];
                mode_product<T, N, false>(Sz, y, x);
#pragma unroll
                for (int i = 0; i < N; ++i) row[i] = x[i];
            }
        }
    });
    __syncthreads();
    axis1(std::integral_constant<bool, false>{});
    __syncthreads();
    // backward, axis 0, to global memory
    dispatch_size<MAXN>(nx, [&](auto nc) {
        constexpr int N = decltype(nc)::value;
        for (unsigned t = tid; t < here * face; t += NT) {
            const unsigned q = quotient(t, by_yz);
            T x[N], y[N];
            lds_read(column0(q, t - mul24(q, face)), step0, x);
            mode_product<T, N, false>(Sx, x, y);
            const unsigned off = mad24(q, total - face, t) * W;
            global_write<(HINT & 2) != 0>(vb, face_bytes, off, y);
        }
    });
}

// Elements per workgroup: the g with the best lane utilisation in the pass with the most
// pencils, among those with at most 256 lanes and at most 40 KB of LDS.
template <typename T>
void aniso_shape(const AnisoArgs &a, int &g, int &nt, size_t &lds)
{
    int maxp = a.ny * a.nz;
    if (a.nx * a.nz > maxp) maxp = a.nx * a.nz;
    if (a.nx * a.ny > maxp) maxp = a.nx * a.ny;
    const size_t cube_bytes = (size_t)a.nx * aniso_pyz(a.ny, a.nz) * sizeof(T);
    g = 1;
    long best_num = 0, best_den = 1;
    for (int c = 1; c <= 256; ++c) {
        const int lanes = c * maxp;
        const int rounded = ((lanes + 63) / 64) * 64;
        if (rounded > ANISO_MAX_NT || c * cube_bytes > 40 * 1024) break;
        if ((long)lanes * best_den >= best_num * rounded) {   // ties: the larger workgroup
            g = c;
            best_num = lanes;
            best_den = rounded;
        }
    }
    nt = ((g * maxp + 63) / 64) * 64;                              // at most 256
    lds = g * cube_bytes;                                          // at most 40 KB (34 KB for g = 1)
}

constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Lane-cycles that the products of g elements need over those that nt lanes spend on them in turns.
double aniso_lane_use(int nx, int ny, int nz, int g, int nt)
{
    double need = 0, spent = 0;
    const int pencils[3] = {ny * nz, nx * nz, nx * ny}, n[3] = {nx, ny, nz};
    for (int d = 0; d < 3; ++d) {
        need += (double)g * pencils[d] * n[d] * n[d];
        spent += (double)ceil_div(g * pencils[d], nt) * nt * n[d] * n[d];
    }
    return need / spent;
}

// Register class of the turns kernel: it holds turns * n words of u_e and of D_e in that many registers.
// (Elements with at most eight points along every axis hardly take it.)
constexpr int turns_class(int n) { return n <= 8 ? 8 : (n + 1) / 2 * 2; }

// Elements and lanes per workgroup of the turns kernel: the best lane use, ties to the fewer lanes (over 46 shapes
// at 100 and 800 MB within 3 % of the best of fourteen settings on average); g = 0: none fits.
template <typename T>
void aniso_turns_shape(int nx, int ny, int nz, int &g, int &nt)
{
    int most = nx > ny ? nx : ny;
    if (nz > most) most = nz;
    const int regs = turns_class(most);
    const size_t cube_bytes = (size_t)nx * aniso_pyz(ny, nz) * sizeof(T);
    g = nt = 0;
    double best = 0;
    for (int lanes = 64; lanes <= ANISO_MAX_NT; lanes += 64)
        for (int c = 1; c <= 64 && c * cube_bytes <= kTurnsLds; ++c) {
            if (ceil_div(c * ny * nz, lanes) * nx > regs || ceil_div(c * nx * ny, lanes) * nz > regs) break;
            const double use = aniso_lane_use(nx, ny, nz, c, lanes);
            if (use > best + 1e-9) {
                best = use;
                g = c;
                nt = lanes;
            }
        }
}

// Whether the turns kernel is the faster one, given the lane use q of the one-turn kernel over its own.  From the times
// of 140 shapes at 4 .. 800 MB: turns / one turn in fp32 0.51 .. 0.73 for q <= 0.4 and 0.68 .. 0.93 for q <= 0.8 at 800 MB, 0.60 .. 0.82
// and 0.79 .. 1.02 at 100 MB, 0.68 .. 0.93 for q <= 0.4 at 40 MB; in fp64, q <= 0.4: 0.47 .. 0.98 at 800 MB, 0.61 .. 1.06 at 100 MB;
// q <= 0.6 where an axis has more than 12 points (four wavefronts per SIMD in the one-turn kernel) 0.83 .. 0.97 at 800 MB,
// elsewhere 0.9 .. 1.06.  On smaller batches a launch is a few rounds of workgroups and the turns are only a longer chain: 0.9 .. 1.5.
// Elements of 108 points and fewer stay ((12,3,3) 1.05, (3,12,3) 1.08), and in fp64 those of less than 300 until 256 MiB
// ((14,4,4) 1.05 at 100 MB, 0.92 at 300).
template <typename T>
bool turns_pay(const AnisoArgs &a, int g1, int nt1, int &g, int &nt)
{
    const int points = a.nx * a.ny * a.nz;
    const long long mib = 3LL * a.num_elems * points * (long long)sizeof(T) >> 20;
    if (points < 112 || mib < (sizeof(T) == 4 ? 32 : points < 300 ? 256 : 64)) return false;
    aniso_turns_shape<T>(a.nx, a.ny, a.nz, g, nt);
    if (g == 0) return false;
    const double q = aniso_lane_use(a.nx, a.ny, a.nz, g1, nt1) / aniso_lane_use(a.nx, a.ny, a.nz, g, nt);
    if (q <= 0.4) return true;
    const bool wide = a.nx > 12 || a.ny > 12 || a.nz > 12;
    if (sizeof(T) == 8) return wide && q <= 0.6 && mib >= 256;
    return q <= 0.8 && mib >= 96;
}

template <typename T, int MAXN, bool STREAM, bool CACHED = false>
hipError_t launch_turns_as(const AnisoArgs &a, int g, int nt)
{
    const long long groups = (a.num_elems + g - 1) / g;
    drop_stale_error();
    hipLaunchKernelGGL((ihelm_aniso_turns_kernel<T, MAXN, aniso_hint(STREAM, CACHED), aniso_xcd(STREAM)>),
                       dim3((unsigned)pencil_grid<aniso_xcd(STREAM)>(groups)), dim3(nt),
                       (size_t)g * a.nx * aniso_pyz(a.ny, a.nz) * sizeof(T), a.stream,
                       (const T *)a.u, (const T *)a.d, (unsigned)a.num_elems, (unsigned)groups, packed_sizes(a.nx, a.ny, a.nz),
                       (unsigned)g, turn_reciprocal(a.ny * a.nz), turn_reciprocal(a.nx * a.nz), turn_reciprocal(a.nx * a.ny),
                       turn_reciprocal(a.ny), turn_reciprocal(a.nz), (const T *)a.sx, (const T *)a.sy, (const T *)a.sz, (T *)a.v);
    return hipGetLastError();
}

template <typename T, int MAXN>
hipError_t launch_turns(const AnisoArgs &a, int g, int nt)
{
    if constexpr (sizeof(T) == 8) {
        const bool stream = aniso_stream<T>(a, true);
        if (aniso_cached_stores<T>(a, true)) {
            if constexpr (MAXN > 8)                         // class of 8: no shape of 128 points with such a face runs in turns
                if (stream) return launch_turns_as<T, MAXN, true, true>(a, g, nt);
            return launch_turns_as<T, MAXN, false, true>(a, g, nt);
        }
        if (stream) return launch_turns_as<T, MAXN, true>(a, g, nt);
    }
    return launch_turns_as<T, MAXN, false>(a, g, nt);
}

template <typename T, int MAXN, bool STREAM, bool CACHED = false>
hipError_t launch_bound_as(const AnisoArgs &a, int g, int nt, size_t lds)
{
    const long long groups = (a.num_elems + g - 1) / g;
    drop_stale_error();
    hipLaunchKernelGGL((ihelm_aniso_kernel<T, MAXN, aniso_hint(STREAM, CACHED), aniso_xcd(STREAM)>),
                       dim3((unsigned)pencil_grid<aniso_xcd(STREAM)>(groups)), dim3(nt), lds, a.stream,
                       (const T *)a.u, (const T *)a.d, (unsigned)a.num_elems, (unsigned)groups, packed_sizes(a.nx, a.ny, a.nz),
                       (unsigned)g, lane_reciprocal(a.ny * a.nz), lane_reciprocal(a.nx * a.nz), lane_reciprocal(a.nx * a.ny),
                       lane_reciprocal(a.ny), lane_reciprocal(a.nz), (const T *)a.sx, (const T *)a.sy, (const T *)a.sz, (T *)a.v);
    return hipGetLastError();
}

template <typename T, int MAXN>
hipError_t launch_bound(const AnisoArgs &a, int g, int nt, size_t lds)
{
    if constexpr (sizeof(T) == 8 && MAXN > 4)            // STREAM needs 128 points
        if (aniso_stream<T>(a, false)) return launch_bound_as<T, MAXN, true>(a, g, nt, lds);
    if constexpr (MAXN <= 6 ? sizeof(T) == 4 : sizeof(T) == 8 && MAXN == 8)
        if (aniso_cached_stores<T>(a, false)) return launch_bound_as<T, MAXN, false, true>(a, g, nt, lds);
    return launch_bound_as<T, MAXN, false>(a, g, nt, lds);
}

template <typename T>
hipError_t launch_generic(const AnisoArgs &a)
{
    if (a.num_elems <= 0 || a.num_elems > 0x7fffffffLL) return kGridTooLarge;
    int n = a.nx > a.ny ? a.nx : a.ny;
    if (a.nz > n) n = a.nz;
    int g, nt, gt, ntt;
    size_t lds;
    aniso_shape<T>(a, g, nt, lds);
    if (sizeof(T) == 4 && slice_kernel_pays(a.nx, a.ny, a.nz, a.num_elems, g, nt / 64))
        return launch_ihelm_slice(a);
    if (turns_pay<T>(a, g, nt, gt, ntt)) {
        switch (turns_class(n)) {
        case 8: return launch_turns<T, 8>(a, gt, ntt);
        case 10: return launch_turns<T, 10>(a, gt, ntt);
        case 12: return launch_turns<T, 12>(a, gt, ntt);
        case 14: return launch_turns<T, 14>(a, gt, ntt);
        default: return launch_turns<T, 16>(a, gt, ntt);
        }
    }
    if (n <= 4) return launch_bound<T, 4>(a, g, nt, lds);
    if constexpr (sizeof(T) == 4)
        if (n <= 6) return launch_bound<T, 6>(a, g, nt, lds);
    if (n <= 8) return launch_bound<T, 8>(a, g, nt, lds);
    if constexpr (sizeof(T) == 8)
        if (n <= 10) return launch_bound<T, 10>(a, g, nt, lds);
    if (n <= 12) return launch_bound<T, 12>(a, g, nt, lds);
    return launch_bound<T, 16>(a, g, nt, lds);
}

}  // namespace

hipError_t launch_ihelm_generic(const AnisoArgs &a, int dtype)
{
    return dtype == TPO_F64 ? launch_generic<double>(a) : launch_generic<float>(a);
}

}  // namespace tpo

extern "C" int tpo_internal_aniso_takes_slice(int nx, int ny, int nz, int dtype, long long num_elems)
{
    if (dtype != TPO_F32) return 0;
    tpo::AnisoArgs a = {};
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    int g, nt;
    size_t lds;
    tpo::aniso_shape<float>(a, g, nt, lds);
    return tpo::slice_kernel_pays(nx, ny, nz, num_elems, g, nt / 64);
}

// 0: one turn per pass (or the slice kernel); else 1000 * elements + lanes per workgroup of the turns kernel.
extern "C" int tpo_internal_aniso_turns(int nx, int ny, int nz, int dtype, long long num_elems)
{
    tpo::AnisoArgs a = {};
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.num_elems = num_elems;
    int g, nt, gt = 0, ntt = 0;
    size_t lds;
    bool turns;
    if (dtype == TPO_F64) {
        tpo::aniso_shape<double>(a, g, nt, lds);
        turns = tpo::turns_pay<double>(a, g, nt, gt, ntt);
    } else {
        tpo::aniso_shape<float>(a, g, nt, lds);
        turns = !tpo::slice_kernel_pays(nx, ny, nz, num_elems, g, nt / 64) && tpo::turns_pay<float>(a, g, nt, gt, ntt);
    }
    return turns ? 1000 * gt + ntt : 0;
}

extern "C" int tpo_internal_aniso_streams(int nx, int ny, int nz, int dtype, long long num_elems)
{
    tpo::AnisoArgs a = {};
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.num_elems = num_elems;
    return dtype == TPO_F64 && tpo::aniso_stream<double>(a, tpo_internal_aniso_turns(nx, ny, nz, dtype, num_elems) != 0);
}

extern "C" int tpo_internal_aniso_caches(int nx, int ny, int nz, int dtype, long long num_elems)
{
    tpo::AnisoArgs a = {};
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.num_elems = num_elems;
    const bool turns = tpo_internal_aniso_turns(nx, ny, nz, dtype, num_elems) != 0;
    return dtype == TPO_F64 ? tpo::aniso_cached_stores<double>(a, turns) : tpo::aniso_cached_stores<float>(a, turns);
}
