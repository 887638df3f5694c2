// Stage 1 of the weight gradient for long filters (dwconv_dw_band.hip.h), both storage types: the launchers.
#include "dwconv_dw_band.hip.h"
#include "dwconv_host.hip.h"

namespace dwhost {

template <typename E>
static int launch_dw_band(const void *x, const void *dy, float *part, void *dw_out, const DwBandPlan &p, int slices, hipStream_t st)
{
    auto go = [&](auto kernel) -> int {
        if (p.lds > 64 * 1024 && !allow_large_lds(kernel)) return DWCONV_ERR_LAUNCH;
        if (p.g.nwin > 65535) return DWCONV_ERR_LAUNCH;                  // (filters of 23 million taps: dw_toep_kernel's)
        // (a grid dimension holds fewer than 2^32 threads: further channels in launches of their own)
        for (int c0 = 0; c0 < p.g.C; c0 += kMaxGridChannels) {
            const int n = p.g.C - c0 < kMaxGridChannels ? p.g.C - c0 : kMaxGridChannels;
            const size_t row = (size_t)c0 * (size_t)p.g.L, taps = (size_t)c0 * (size_t)p.g.K;
            hipLaunchKernelGGL(kernel, dim3((unsigned)n, (unsigned)p.S, (unsigned)p.g.nwin), dim3(dwconv::kDwBandThreads), p.lds, st,
                               static_cast<const E *>(x) + row, static_cast<const E *>(dy) + row, part + taps,
                               dw_out ? static_cast<E *>(dw_out) + taps : nullptr, p.g, slices);
        }
        return launch_status();
    };
    auto form = [&](auto nd, auto dg) -> int {
        constexpr int ND = decltype(nd)::value, DG = decltype(dg)::value;
        if constexpr (std::is_same<E, float>::value) {
            if (p.g.chain > 0) return p.split ? go(dwconv::dw_band_kernel<E, ND, DG, true, true>) : go(dwconv::dw_band_kernel<E, ND, DG, false, true>);
        }
        return p.split ? go(dwconv::dw_band_kernel<E, ND, DG, true>) : go(dwconv::dw_band_kernel<E, ND, DG, false>);
    };
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    constexpr std::integral_constant<int, 4> c4{};
    switch (8 * p.ND + p.g.dg_log) {
    case 8: return form(c1, c1);
    case 16: return form(c2, c1);
    case 17: return form(c2, c2);
    case 18: return form(c2, c4);
    case 24: return form(c3, c1);
    case 25: return form(c3, c2);
    case 26: return form(c3, c4);
    default:
        if constexpr (std::is_same<E, float>::value) return DWCONV_ERR_LAUNCH;       // (never planned)
        else return form(c4, c4);
    }
}

int launch_dw_band_f32(const void *x, const void *dy, float *part, void *dw_out, const DwBandPlan &p, int slices, hipStream_t st)
{
    return launch_dw_band<float>(x, dy, part, dw_out, p, slices, st);
}
int launch_dw_band_bf16(const void *x, const void *dy, float *part, void *dw_out, const DwBandPlan &p, int slices, hipStream_t st)
{
    return launch_dw_band<bf16_t>(x, dy, part, dw_out, p, slices, st);
}

}  // namespace dwhost
