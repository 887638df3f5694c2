// Shared by the translation units of the fp32 weight-gradient kernels with seven to sixteen block offsets (the largest fully
// unrolled kernels of the library: split over several units so that they compile side by side).
#pragma once
#include "dwconv_host.hip.h"

namespace dwhost {

// fp32, seven to sixteen block offsets (K up to 226): the LDS-direct kernel on ordinary rows.
template <int ND, int W>
int launch_dw_partial_wide_ndw(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                               int dmin, hipStream_t st)
{
    constexpr size_t lds = dwconv::dw_direct_lds_bytes(ND, W);
    if constexpr (lds > kMaxLdsBytes) {
        return -1;
    } else {
        auto kernel = dwconv::dw_partial_direct_kernel<ND, W, false>;
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                           static_cast<const float *>(x), static_cast<const float *>(dy), part,
                           static_cast<float *>(dw_out), s.B, s.C, s.L, s.K, s.pad, dmin, p.tiles_per_row, p.rows.map);
        return launch_status();
    }
}

// The units: four-wave workgroups on ordinary rows and on virtual rows, whole-channel workgroups of five, eight and sixteen
// waves.
int launch_dw_wide_w4_f32(int nd, const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                          int dmin, hipStream_t st);
int launch_dw_wide_rows_f32(int nd, const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                            int dmin, hipStream_t st);
int launch_dw_wide_multi_f32(int nd, const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                             int dmin, hipStream_t st);

}  // namespace dwhost
