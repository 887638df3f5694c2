// Rows of 132 to 512 positions with filters of the order of the row length, f32 storage: stage 1 of the
// weight gradient on the sixteen-row kernels of dwconv_rowtall.hip.h.
#include "dwconv_host.hip.h"

namespace dwhost {

namespace {

dwconv::RowTallGeom rowtall_geom(const Shape &s, int pad)
{
    dwconv::RowTallGeom g;
    int dmin, nd;
    rows_batch_offsets(s.L, s.K, pad, &dmin, &nd);
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K;
    g.pad = pad;
    g.dmin = dmin; g.dmax = dmin + nd - 1;
    g.m = (s.L + 15) / 16;
    g.n_units = 0; g.win = 0;
    g.lg_recip = (unsigned)((1ull << 32) / (unsigned long long)((s.L + 3) / 4)) + 1u;
    return g;
}

}  // namespace

int launch_dw_rowtall_f32(const void *x, const void *dy, float *part, const Shape &s, const DwPlan &p, hipStream_t st)
{
    typedef float T;
    dwconv::RowTallGeom g = rowtall_geom(s, s.pad);
    g.n_units = (s.B + 3) / 4;
    const int nwin = (g.dmax - g.dmin + 1 + dwconv::kRtWindow - 1) / dwconv::kRtWindow;
    if (nwin != p.tall_windows || p.S % nwin != 0 || p.S / nwin > 65535) return -1;
    g.win = (g.dmax - g.dmin + 1 + nwin - 1) / nwin;                  // windows of equal size
    auto kernel = dwconv::dw_rowtall_kernel<T>;
    const size_t lds = dwconv::rt_dw_lds_bytes(g.m);
    if (lds > kMaxLdsBytes) return -1;
    if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
    hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)(p.S / nwin), (unsigned)nwin), dim3(64 * dwconv::kRtWaves), lds, st,
                       static_cast<const T *>(x), static_cast<const T *>(dy), part, g);
    return launch_status();
}

}  // namespace dwhost
