// Weight-gradient stage-1 kernels, fp32, four-wave workgroups on the virtual rows of short rows: seven to sixteen block offsets
// (which of them go to dw_band_kernel instead: dw_takes_band).
#include "dwconv_launch_dw_wide.hip.h"

namespace dwhost {

template <int ND>
static int launch_rows_nd(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p, int dmin,
                          hipStream_t st)
{
    constexpr int W = 4;
    constexpr size_t lds = dwconv::dw_direct_lds_bytes(ND, W);
    static_assert(lds <= kMaxLdsBytes, "LDS budget");
    auto kernel = dwconv::dw_partial_direct_kernel<ND, W, true>;
    if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
    hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st, static_cast<const float *>(x),
                       static_cast<const float *>(dy), part, static_cast<float *>(dw_out), 1, s.C, s.L, s.K, s.pad, dmin,
                       p.tiles_per_row, p.rows.map);
    return launch_status();
}

int launch_dw_wide_rows_f32(int nd, const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                            int dmin, hipStream_t st)
{
    if (p.wpb != 4) return -1;
    switch (nd) {
    case 7: return launch_rows_nd<7>(x, dy, part, dw_out, s, p, dmin, st);
    case 8: return launch_rows_nd<8>(x, dy, part, dw_out, s, p, dmin, st);
    case 9: return launch_rows_nd<9>(x, dy, part, dw_out, s, p, dmin, st);
    case 10: return launch_rows_nd<10>(x, dy, part, dw_out, s, p, dmin, st);
    case 11: return launch_rows_nd<11>(x, dy, part, dw_out, s, p, dmin, st);
    case 12: return launch_rows_nd<12>(x, dy, part, dw_out, s, p, dmin, st);
    case 13: return launch_rows_nd<13>(x, dy, part, dw_out, s, p, dmin, st);
    case 14: return launch_rows_nd<14>(x, dy, part, dw_out, s, p, dmin, st);
    case 15: return launch_rows_nd<15>(x, dy, part, dw_out, s, p, dmin, st);
    case 16: return launch_rows_nd<16>(x, dy, part, dw_out, s, p, dmin, st);
    default: return -1;
    }
}

}  // namespace dwhost
