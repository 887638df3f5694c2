// Stage 1 of the weight gradient for filters of hundreds of taps and more (dwconv_dw_toep.hip.h), both storage types: the
// launchers.
#include "dwconv_dw_toep.hip.h"
#include "dwconv_host.hip.h"

namespace dwhost {

// Pieces of lags per launch: 8192 fill the chip as well as 65535, and a test reaches the second launch (23 million lags, 11280 pieces).
constexpr int kMaxGridPieces = 8192;

template <typename E>
static int launch_dw_toep(const void *x, const void *dy, float *part, void *dw_out, const DwToepPlan &p, int slices, hipStream_t st)
{
    auto go = [&](auto kernel) -> int {
        if (p.lds > 64 * 1024 && !allow_large_lds(kernel)) return DWCONV_ERR_LAUNCH;
        // (a grid holds fewer than 2^32 threads along channels and 65536 pieces: what is beyond in launches of their own)
        dwconv::DwToepGeom g = p.g;
        for (g.piece0 = 0; g.piece0 < g.npiece; g.piece0 += kMaxGridPieces) {
            const int nz = g.npiece - g.piece0 < kMaxGridPieces ? g.npiece - g.piece0 : kMaxGridPieces;
            for (int c0 = 0; c0 < g.C; c0 += kMaxGridChannels) {
                const int n = g.C - c0 < kMaxGridChannels ? g.C - c0 : kMaxGridChannels;
                const size_t row = (size_t)c0 * (size_t)g.L, taps = (size_t)c0 * (size_t)g.K;
                hipLaunchKernelGGL(kernel, dim3((unsigned)n, (unsigned)p.S, (unsigned)nz), dim3(dwconv::kToepThreads), p.lds, st,
                                   static_cast<const E *>(x) + row, static_cast<const E *>(dy) + row, part + taps,
                                   dw_out ? static_cast<E *>(dw_out) + taps : nullptr, g, slices);
            }
        }
        return launch_status();
    };
    return p.T == 1 ? go(dwconv::dw_toep_kernel<E, 1>) : go(dwconv::dw_toep_kernel<E, 2>);
}

int launch_dw_toep_f32(const void *x, const void *dy, float *part, void *dw_out, const DwToepPlan &p, int slices, hipStream_t st)
{
    return launch_dw_toep<float>(x, dy, part, dw_out, p, slices, st);
}
int launch_dw_toep_bf16(const void *x, const void *dy, float *part, void *dw_out, const DwToepPlan &p, int slices, hipStream_t st)
{
    return launch_dw_toep<bf16_t>(x, dy, part, dw_out, p, slices, st);
}

}  // namespace dwhost
