// fp32 slice kernel of the inverse-Helmholtz operator for anisotropic elements: one wavefront per
// element, no barriers, both axes of a slice in matrix instructions without touching memory in
// between.
//
// The cube is taken as n_x slices (b, c) of at most 16 x 16 points, and a slice goes through its
// two mode products as two chained 16x16x4 matrix products in registers: the accumulator of one
// product is, unchanged, the A operand of the next.  With lane = 16 g + x the instruction takes
// A[m][k] from lane (x = m, g = k), B[k][n] from lane (x = n, g = k) and leaves D[m][n], m = 4g+r,
// in register r of lane (x = n, g).  D as the A operand of the next product therefore contracts
// over m and has n as its rows:
//
//   forward   t1[c][j] = sum_b u[b][c] Sy[b][j]      A = u (from LDS),             B = Sy
//             t2[j][k] = sum_c t1[c][j] Sz[c][k]     A = t1,                       B = Sz
//   axis 0    every lane now holds, for its columns (j, k), all n_x slices: the two axis-0
//             products and the scale by D_e are pencil products on the lane's own registers
//             (4x4x1 matrix products, tpo_pencil_mm.hpp)
//   backward  t3[k][b] = sum_j g[j][k] Sy[b][j]      A = g (as columns k),         B = Sy^T
//             v[b][c]  = sum_k t3[k][b] Sz[c][k]     A = t3,                       B = Sz^T
//
// Index maps.  Which index a lane x stands for, and which one register r of group g does, is free
// as long as producer and consumer agree:
//   * b and j: index 4s + g in register (k-step) s of group g, so that KSB = ceil(n_y/4) registers
//     and k-steps are enough; the lanes x of the operand that becomes these rows stand for
//     4 (x % 4) + x / 4;
//   * c and k: lane x stands for KSC (x / 4) + x % 4 with the lanes x % 4 >= KSC idle,
//     KSC = ceil(n_z/4): register r of group g is then KSC g + r and KSC k-steps are enough.
// Only KSB, KSC and n_x are compile-time: one kernel serves every n_y, n_z of its class.  Lanes and
// registers past the slice repeat its last row or column as free indices (they store what that
// one stores) and are zeroed in the data before they enter a sum (not only in the coefficients:
// zero times an infinity is not zero).
//
// Memory.  u_e and D_e come flat, 1 KB per instruction, straight into LDS (global_load_lds_dwordx4),
// v_e leaves through LDS as flat 16-byte stores, OUT slices at a time.  A wavefront walks over a few
// consecutive elements: the next u_e is on its way from the end of the forward products on, the
// next D_e from the end of the scale on.
//
// What bounds it: at (12,12,16) issue of the matrix instructions, 7104 cycles per element: they hold a
// SIMD 65 % of the launch and the other vector instructions 7 %, at a clock that falls to 1.8 GHz,
// with seven wavefronts per CU (21 KB of LDS each) to cover loads and LDS.  Other shapes take 4 to 32 KB of
// LDS per wavefront, half of them less than 13 KB; there registers set the number of wavefronts, two
// per SIMD from n_x KSB = 33 on, one for n_x >= 15 with KSB = 4.  Against the runtime-size pencil
// kernel, GB/s of algorithmic traffic on 6 GB: (12,12,16) 4980 against 3820, (11,11,14) 4520 / 3630, (9,14,15)
// 4750 / 3070, (12,16,16) 4850 / 3770, (13,13,12) 4190 / 3730.
// One element per wavefront instead of a walk over eight: 4150 instead of 4400 at (12,16,16); a
// grid of resident wavefronts that divide the batch among them: the same at eight wavefronts per CU,
// slower where the LDS allows five to seven (they load the four SIMDs unevenly).
#pragma once
#include <hip/hip_runtime.h>

#include "tpo_internal.h"
#include "tpo_mfma.hpp"
#include "tpo_pencil.hpp"
#include "tpo_pencil_mm.hpp"

namespace tpo {

// 16 (x4) or 4 (x1) bytes per lane from memory straight to LDS, lane L to lds + 16 L (4 L); lds is
// uniform.  Counted by vmcnt; the caller waits.  The address goes through m0, as an operand, so that the
// compiler knows what m0 holds; the s_nop is the wait state that such a load needs behind a write of m0.
__device__ __forceinline__ void lds_load_x4(const void *src, unsigned lds)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "{m0}"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(src) : "memory");
}
__device__ __forceinline__ void lds_load_x1(const void *src, unsigned lds)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %1, off"
                 :: "{m0}"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(src) : "memory");
}
// A field of one element (whole words, word aligned) as a flat copy in LDS: 16-byte chunks, then
// one instruction for the up to three words past the last whole chunk.
__host__ __device__ constexpr int stage_bytes(int bytes) { return (bytes + 15) / 16 * 16; }
__device__ __forceinline__ void stage_field(const float *src, unsigned lds, int bytes, int lane)
{
    const char *p = reinterpret_cast<const char *>(src);
    const int chunks = bytes / 16, full = chunks / 64;
    for (int i = 0; i < full; ++i) lds_load_x4(p + (i * 1024 + lane * 16), lds + i * 1024);
    if (lane < chunks % 64) lds_load_x4(p + (full * 1024 + lane * 16), lds + full * 1024);
    if (lane < bytes % 16 / 4) lds_load_x1(p + (chunks * 16 + lane * 4), lds + chunks * 16);
}
// Waits until at most N of the wavefront's loads and stores (they complete in order) are
// outstanding; the counter holds 63.
template <int N>
__device__ __forceinline__ void wait_outstanding()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N < 63 ? N : 63) : "memory");
}
// The wavefront's LDS reads have returned: what they read may be overwritten by a load to LDS.
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int NX, int KSB, int KSC>
struct SliceShape {
    // Slices per group of stores.  Four fill the 1 KB store instructions better, two need less LDS:
    // GB/s with four / two on 6 GB, (12,12,16) 4980 / 4510, (11,11,14) 4520 / 4520, (12,16,16)
    // 4850 / 5020, (13,14,14) 4190 / 4365, (15,15,16) 3960 / 4330.  By n_x alone, although what four
    // slices cost goes with n_y n_z: (12,16,16) has the slower one of the two.
    static constexpr int OUT = NX <= 12 ? 4 : 2;
    // LDS of one workgroup (one wavefront): both stages and the slices on their way out.
    static size_t lds_bytes(int ny, int nz)
    {
        return (size_t)2 * stage_bytes(NX * ny * nz * 4) + (size_t)OUT * ny * nz * 4;
    }
    // Memory instructions of one element, lower bounds over the class (smallest n_y, n_z): loads of
    // one field, stores.
    static constexpr int FACE_MIN = (4 * KSB - 3) * (4 * KSC - 3);
    static constexpr int N_IN = (NX * FACE_MIN / 4 + 63) / 64;
    static constexpr int N_ST = NX / OUT * (OUT * FACE_MIN / 4 / 64);
    // 512 registers per SIMD: two wavefronts on each while the n_x slices leave room.
    static constexpr int WAVES = NX <= 14 ? 2 : 1;
};

// Each workgroup (one wavefront) takes `walk` consecutive elements.  Workgroups are numbered per
// accelerator die as in pencil_batch<true>; the grid is a multiple of 8.
template <int NX, int KSB, int KSC>
__global__ void __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu((SliceShape<NX, KSB, KSC>::WAVES))))
ihelm_slice_kernel(const float *u, const float *__restrict__ Sx, const float *__restrict__ Sy,
                   const float *__restrict__ Sz, const float *__restrict__ D, float *v, int ny, int nz,
                   int walk, long long num_elems)
{
    using Sh = SliceShape<NX, KSB, KSC>;
    using MM = MmShape<NX>;
    using M = Mfma<float>;
    using acc_t = M::acc_t;
    constexpr int OUT = Sh::OUT, NSL = 2;        // NSL slices share a run of matrix instructions
    static_assert(OUT % NSL == 0, "a group of stores is whole runs");
    extern __shared__ __align__(16) unsigned char tpo_lds[];
    const int face = ny * nz;
    const int cube_bytes = NX * face * 4;
    float *us = reinterpret_cast<float *>(tpo_lds);
    float *ds = reinterpret_cast<float *>(tpo_lds + stage_bytes(cube_bytes));
    float *os = reinterpret_cast<float *>(tpo_lds + 2 * stage_bytes(cube_bytes));
    const unsigned us_at = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)tpo_lds;
    const unsigned ds_at = us_at + stage_bytes(cube_bytes);

    const int lane = threadIdx.x & 63;
    const int x = lane & 15, g = lane >> 4;
    long long e = ((long long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * walk;
    if (e >= num_elems) return;
    auto field = [&](const float *f, long long el) { return f + (size_t)el * (size_t)(NX * face); };

    const int xm = 4 * (x & 3) + (x >> 2);                             // lane x along the middle axis
    const int xf = (x & 3) < KSC ? KSC * (x >> 2) + (x & 3) : 16;      // ... along the fastest axis
    const bool col = xf < nz;
    const int xfc = col ? xf : nz - 1;

    // ---- coefficient operands, for the products over b, c, j, k --------------------------------
    float cb[KSB], cc[KSC], cj[KSB], ck[KSC];
#pragma unroll
    for (int s = 0; s < KSB; ++s) {
        const bool ok = 4 * s + g < ny;
        const int k = ok ? 4 * s + g : 0, n = xm < ny ? xm : ny - 1;
        const float f = Sy[k * ny + n], b = Sy[n * ny + k];
        cb[s] = ok ? f : 0.0f;
        cj[s] = ok ? b : 0.0f;
    }
#pragma unroll
    for (int s = 0; s < KSC; ++s) {
        const bool ok = KSC * g + s < nz;
        const int k = ok ? KSC * g + s : 0;
        const float f = Sz[k * nz + xfc], b = Sz[(x < nz ? x : nz - 1) * nz + k];
        cc[s] = ok ? f : 0.0f;
        ck[s] = ok ? b : 0.0f;
    }
    const TPO_CONSTANT float *Sxc = (const TPO_CONSTANT float *)Sx;
    float tab_f[MM::NTAB], tab_b[MM::NTAB];
#pragma unroll
    for (int r = 0; r < MM::NTAB; ++r) {
        tab_f[r] = mm_coef<NX>(Sx, true, r, lane);
        tab_b[r] = mm_coef<NX>(Sx, false, r, lane);
    }

    // Register r: word (row 4r+g, column xf) of a slice on its way in, (row 4r+g, column x) on its
    // way out, and whether the former lies in the slice.
    int o_in[KSB], o_out[KSB];
    bool in_slice[KSB];
#pragma unroll
    for (int r = 0; r < KSB; ++r) {
        const int row = 4 * r + g < ny ? 4 * r + g : ny - 1;
        o_in[r] = row * nz + xfc;
        o_out[r] = row * nz + (x < nz ? x : nz - 1);
        in_slice[r] = col && 4 * r + g < ny;
    }

    // Two chained products on the NSL slices from a0 on (those past the last one are skipped): over
    // the middle axis with cm, over the fastest with cf.
    auto chain = [&](int a0, const float (&w)[NSL][KSB], const float (&cm)[KSB], const float (&cf)[KSC],
                     acc_t (&out)[NSL]) {
        acc_t acc[NSL];
#pragma unroll
        for (int q = 0; q < NSL; ++q) acc[q] = out[q] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KSB; ++s)
#pragma unroll
            for (int q = 0; q < NSL; ++q)
                if (a0 + q < NX) acc[q] = M::mma(w[q][s], cm[s], acc[q]);
#pragma unroll
        for (int s = 0; s < KSC; ++s)
#pragma unroll
            for (int q = 0; q < NSL; ++q)
                if (a0 + q < NX) out[q] = M::mma(acc[q][s], cf[s], out[q]);
    };

    stage_field(field(u, e), us_at, cube_bytes, lane);
    stage_field(field(D, e), ds_at, cube_bytes, lane);
    for (bool first = true;; first = false) {
        const long long next = e + 1;
        const bool more = --walk > 0 && next < num_elems;
        float *ve = v + (size_t)e * (size_t)(NX * face);
        float t[NX][KSB];

        // ---- forward, axes 1 and 2, slice by slice ---------------------------------------------
        // issued after this u_e: D_e, and the stores of the element before
        if (first) wait_outstanding<Sh::N_IN>(); else wait_outstanding<Sh::N_IN + Sh::N_ST>();
#pragma unroll
        for (int a0 = 0; a0 < NX; a0 += NSL) {
            float w[NSL][KSB];
#pragma unroll
            for (int q = 0; q < NSL; ++q)
#pragma unroll
                for (int s = 0; s < KSB; ++s)
                    if (a0 + q < NX) {
                        const float word = us[(a0 + q) * face + o_in[s]];
                        w[q][s] = in_slice[s] ? word : 0.0f;
                    }
            acc_t out[NSL];
            chain(a0, w, cb, cc, out);
#pragma unroll
            for (int q = 0; q < NSL; ++q)
#pragma unroll
                for (int r = 0; r < KSB; ++r)
                    if (a0 + q < NX) t[a0 + q][r] = out[q][r];
        }
        wait_lds_reads();
        if (more) stage_field(field(u, next), us_at, cube_bytes, lane);

        // ---- axis 0 forward, scale, axis 0 backward, pencil by pencil --------------------------
        // issued after this D_e: the stores of the element before, the next u_e
        if (!more) wait_outstanding<0>();
        else if (first) wait_outstanding<Sh::N_IN>();
        else wait_outstanding<Sh::N_ST + Sh::N_IN>();
#pragma unroll
        for (int r = 0; r < KSB; ++r) {
            float p[NX], y[MM::NY], d[NX];
#pragma unroll
            for (int a = 0; a < NX; ++a) {
                p[a] = t[a][r];
                d[a] = ds[a * face + o_in[r]];
            }
            mode_product_mm<NX, true>(tab_f, Sxc, p, y);
#pragma unroll
            for (int a = 0; a < NX; ++a) p[a] = in_slice[r] ? y[a] * d[a] : 0.0f;
            mode_product_mm<NX, false>(tab_b, Sxc, p, y);
#pragma unroll
            for (int a = 0; a < NX; ++a) t[a][r] = y[a];
        }
        wait_lds_reads();
        if (more) stage_field(field(D, next), ds_at, cube_bytes, lane);

        // ---- backward, axes 1 and 2; OUT slices at a time leave through LDS --------------------
#pragma unroll
        for (int b0 = 0; b0 < NX; b0 += OUT) {
#pragma unroll
            for (int a0 = b0; a0 < b0 + OUT && a0 < NX; a0 += NSL) {
                float w[NSL][KSB];
#pragma unroll
                for (int q = 0; q < NSL; ++q)
#pragma unroll
                    for (int s = 0; s < KSB; ++s)
                        if (a0 + q < NX) w[q][s] = t[a0 + q][s];
                acc_t out[NSL];
                chain(a0, w, cj, ck, out);
#pragma unroll
                for (int q = 0; q < NSL; ++q)
#pragma unroll
                    for (int r = 0; r < KSB; ++r)
                        if (a0 + q < NX) os[(a0 - b0 + q) * face + o_out[r]] = out[q][r];
            }
            // LDS operations of a wavefront run in order; the fences keep the compiler to it (words
            // written, vectors read)
            asm volatile("" ::: "memory");
            typedef WordVec<float, 4>::type vec;
            const int words = (NX - b0 < OUT ? NX - b0 : OUT) * face;
            float *dst = ve + b0 * face;
#pragma unroll
            for (int i = 0; i < (OUT * 16 * KSB * KSC / 4 + 63) / 64; ++i) {
                const int c = i * 64 + lane;
                if (4 * c + 4 <= words)
                    __builtin_nontemporal_store(*reinterpret_cast<const vec *>(os + 4 * c),
                                                reinterpret_cast<vec *>(dst + 4 * c));
            }
            if (lane < words % 4) dst[words / 4 * 4 + lane] = os[words / 4 * 4 + lane];
            asm volatile("" ::: "memory");
        }
        if (!more) break;
        e = next;
    }
}

template <int NX, int KSB, int KSC>
hipError_t launch_slice(const AnisoArgs &a)
{
    // Elements per wavefront: eight (the next element's loads and the coefficients are then shared
    // out) while that leaves four rounds of the wavefronts the chip holds, fewer below.
    const long long resident = 256 * 8;
    long long walk = a.num_elems / (4 * resident);
    walk = walk < 1 ? 1 : (walk > 8 ? 8 : walk);
    const long long blocks = pencil_grid<true>((a.num_elems + walk - 1) / walk);
    drop_stale_error();
    hipLaunchKernelGGL((ihelm_slice_kernel<NX, KSB, KSC>), dim3((unsigned)blocks), dim3(64),
                       (SliceShape<NX, KSB, KSC>::lds_bytes(a.ny, a.nz)), a.stream, (const float *)a.u,
                       (const float *)a.sx, (const float *)a.sy, (const float *)a.sz, (const float *)a.d,
                       (float *)a.v, a.ny, a.nz, (int)walk, a.num_elems);
    return hipGetLastError();
}

}  // namespace tpo
