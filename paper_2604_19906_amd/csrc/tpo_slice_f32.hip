// Instantiations of the fp32 slice kernel (tpo_slice.hpp) and the rule that says which anisotropic
// calls take it instead of the runtime-size pencil kernel (tpo_generic.hip).
#include "tpo_slice.hpp"

namespace tpo {

namespace {

constexpr int NX_MIN = 5, NX_MAX = 16, KSB_MIN = 2, KSC_MIN = 3;

typedef hipError_t (*SliceLaunch)(const AnisoArgs &);
// Null for the classes that no shape of slice_kernel_pays() is in.
template <int NX, int KSB, int KSC>
constexpr SliceLaunch slice_entry()
{
    if constexpr (KSB == 2 && KSC == 3 && (NX == 7 || NX == 8 || NX == 10)) return nullptr;
    else if constexpr (KSB == 4 && KSC == 3 && NX >= 15) return nullptr;
    else return &launch_slice<NX, KSB, KSC>;
}
#define TPO_SLICE_NX(NX)                                  \
    {{slice_entry<NX, 2, 3>(), slice_entry<NX, 2, 4>()},  \
     {slice_entry<NX, 3, 3>(), slice_entry<NX, 3, 4>()},  \
     {slice_entry<NX, 4, 3>(), slice_entry<NX, 4, 4>()}}
const SliceLaunch kSlice[NX_MAX - NX_MIN + 1][3][2] = {
    TPO_SLICE_NX(5),  TPO_SLICE_NX(6),  TPO_SLICE_NX(7),  TPO_SLICE_NX(8),
    TPO_SLICE_NX(9),  TPO_SLICE_NX(10), TPO_SLICE_NX(11), TPO_SLICE_NX(12),
    TPO_SLICE_NX(13), TPO_SLICE_NX(14), TPO_SLICE_NX(15), TPO_SLICE_NX(16),
};

// Issue cycles of an element's products on a SIMD: n_x slices, KSB + KSC instructions of 32 cycles
// each way, and KSB pencils of 4x4x1 products (8 cycles for four rows; a single left-over row as
// vector FMAs, 4 cycles each) each way.
long slice_cycles(int nx, int ksb, int ksc)
{
    const bool rem = nx % 4 == 1;
    const int pencil = nx * (rem ? nx / 4 : (nx + 3) / 4) * 8 + (rem ? 4 * nx : 0);
    return (long)nx * (ksb + ksc) * 64 + (long)ksb * 2 * pencil;
}

// Two counts for a workgroup of the pencil kernel, whose six passes issue n^2 FMAs of 4 cycles on every
// wavefront that has pencils: what it issues, and what it would issue if none of its `waves`
// wavefronts sat a pass out (they hold their places on the SIMD while they do).
long pencil_issued(int nx, int ny, int nz, int g)
{
    auto pass = [&](int n, int pencils) { return (long)n * n * ((g * pencils + 63) / 64); };
    return 8 * (pass(nx, ny * nz) + pass(ny, nx * nz) + pass(nz, nx * ny));
}
long pencil_held(int nx, int ny, int nz, int waves) { return 8L * (nx * nx + ny * ny + nz * nz) * waves; }

}  // namespace

// The lines are measured on all shapes with 5 <= n_x, n_y and 9 <= n_z at batches of 8 MB to 2.5 GB, time of
// the slice kernel over that of the pencil kernel (9134 calls):
//   * slice/held <= 0.8 and slice/issued <= 1.36: 0.40 .. 1.06, nine in ten below 1.0.  `held` alone takes in
//     shapes with a short pass, (16,7,9) 1.22, (13,6,10) 1.11, (12,5,11) 1.15 (slice/issued 1.45 to 1.9).
//   * n_y and n_x large enough for two wavefronts per SIMD (n_x >= 13, KSB >= 3): slice/issued <= 1.05; from
//     1.05 to 1.2 0.95 .. 1.12, (13,9,13) 1.11.
//   * one wavefront per SIMD (n_x >= 15, KSB = 4): only with slice/issued <= 0.625 and from 24576 elements
//     on, where a wavefront walks over three or more: 0.79 .. 0.97.  Below 24576 elements 0.97 .. 1.17, with
//     slice/issued 0.65 .. 1.05 1.0 .. 1.5 at every batch.
//   * Shapes with n_z <= 8 do not keep to the counts (0.57: 1.28, 0.7: 1.47) and stay with the pencil kernel.
//   * On small batches one wavefront per element has fewer wavefronts to hide its latency behind: from
//     1024 elements on slice/held <= 0.625 and n_x <= 14 (0.43 .. 0.96), with n_x >= 13 and KSB >= 3 from 2048
//     (1024 .. 2047: 0.88 .. 1.19).  Below 1024 elements the two leapfrog.
bool slice_kernel_pays(int nx, int ny, int nz, long long num_elems, int elems_per_wg, int waves_per_wg)
{
    const int ksb = (ny + 3) / 4, ksc = (nz + 3) / 4;
    if (nx < NX_MIN || nx > NX_MAX || ksb < KSB_MIN || ksc < KSC_MIN) return false;
    const long slice = slice_cycles(nx, ksb, ksc) * elems_per_wg;
    const long issued = pencil_issued(nx, ny, nz, elems_per_wg);
    const long held = pencil_held(nx, ny, nz, waves_per_wg);
    if (nx >= 15 && ksb == 4) return num_elems >= 24576 && 8 * slice <= 5 * issued;
    const bool two_waves = nx >= 13 && ksb >= 3;
    if (two_waves ? 20 * slice > 21 * issued : 25 * slice > 34 * issued) return false;
    if (num_elems >= 12288) return 5 * slice <= 4 * held;
    return num_elems >= (two_waves ? 2048 : 1024) && nx <= 14 && 8 * slice <= 5 * held;
}

hipError_t launch_ihelm_slice(const AnisoArgs &a)
{
    return kSlice[a.nx - NX_MIN][(a.ny + 3) / 4 - KSB_MIN][(a.nz + 3) / 4 - KSC_MIN](a);
}

bool slice_class_built(int nx, int ksb, int ksc)
{
    if (nx < NX_MIN || nx > NX_MAX || ksb < KSB_MIN || ksb > 4 || ksc < KSC_MIN || ksc > 4) return false;
    return kSlice[nx - NX_MIN][ksb - KSB_MIN][ksc - KSC_MIN] != nullptr;
}

}  // namespace tpo

extern "C" int tpo_internal_slice_class_built(int nx, int ksb, int ksc)
{
    return tpo::slice_class_built(nx, ksb, ksc);
}
