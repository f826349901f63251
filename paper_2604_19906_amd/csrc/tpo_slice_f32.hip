// Instantiations of the fp32 slice kernel (tpo_slice.hpp) and the rule that says which anisotropic
// calls take it instead of the runtime-size pencil kernel (tpo_generic.hip).
#include "tpo_slice.hpp"

namespace tpo {

namespace {

constexpr int NX_MIN = 5, NX_MAX = 16, KSB_MIN = 2, KSC_MIN = 3;

typedef hipError_t (*SliceLaunch)(const AnisoArgs &);
#define TPO_SLICE_NX(NX)                                      \
    {{&launch_slice<NX, 2, 3>, &launch_slice<NX, 2, 4>},      \
     {&launch_slice<NX, 3, 3>, &launch_slice<NX, 3, 4>},      \
     {&launch_slice<NX, 4, 3>, &launch_slice<NX, 4, 4>}}
const SliceLaunch kSlice[NX_MAX - NX_MIN + 1][3][2] = {
    TPO_SLICE_NX(5),  TPO_SLICE_NX(6),  TPO_SLICE_NX(7),  TPO_SLICE_NX(8),
    TPO_SLICE_NX(9),  TPO_SLICE_NX(10), TPO_SLICE_NX(11), TPO_SLICE_NX(12),
    TPO_SLICE_NX(13), TPO_SLICE_NX(14), TPO_SLICE_NX(15), TPO_SLICE_NX(16),
};

// Issue cycles of an element's products on a SIMD.  Slice kernel: n_x slices, KSB + KSC
// instructions of 32 cycles each way, and KSB pencils of 4x4x1 products (8 cycles for four rows; a
// single left-over row as vector FMAs, 4 cycles each) each way.  Pencil kernel: in each of its six
// passes every wavefront of the workgroup issues n^2 FMAs of 4 cycles.
long slice_cycles(int nx, int ksb, int ksc)
{
    const bool rem = nx % 4 == 1;
    const int pencil = nx * (rem ? nx / 4 : (nx + 3) / 4) * 8 + (rem ? 4 * nx : 0);
    return (long)nx * (ksb + ksc) * 64 + (long)ksb * 2 * pencil;
}

}  // namespace

bool slice_kernel_pays(int nx, int ny, int nz, long long num_elems, int elems_per_wg, int waves_per_wg)
{
    const int ksb = (ny + 3) / 4, ksc = (nz + 3) / 4;
    if (nx < NX_MIN || nx > NX_MAX || ksb < KSB_MIN || ksc < KSC_MIN) return false;
    const long slice = slice_cycles(nx, ksb, ksc) * elems_per_wg;
    const long pencil = 2L * (nx * nx + ny * ny + nz * nz) * 4 * waves_per_wg;
    // Measured on 90 shapes of 5 .. 16 points per axis, 3 GB a call: every shape with
    // slice/pencil <= 0.8 is as fast or faster (0.23: 0.46 of the pencil kernel's time, 0.5: 0.7-0.8,
    // 0.63: 0.75-0.85, 0.8: 0.91-1.0), above that most are slower (0.92: 1.12, 1.2: 1.25).  The
    // shapes with n_z <= 8 do not keep to the line (0.57: 1.28, 0.7: 1.47) and stay with the pencil
    // kernel.  On small batches one wavefront per element has fewer wavefronts to hide its
    // latency behind: E = 1000 .. 6000: ratio 0.54-0.62 0.81-0.87 of the time, 0.76 1.05, n_x >= 15
    // 0.94-1.06; below about a thousand elements the two leapfrog (0.77-1.2).
    if (num_elems >= 12288) return 5 * slice <= 4 * pencil;
    return num_elems >= 1024 && nx <= 14 && 8 * slice <= 5 * pencil;
}

hipError_t launch_ihelm_slice(const AnisoArgs &a)
{
    return kSlice[a.nx - NX_MIN][(a.ny + 3) / 4 - KSB_MIN][(a.nz + 3) / 4 - KSC_MIN](a);
}

}  // namespace tpo
