// Launchers of the forward / input-gradient kernels for long filters (dwconv_band.hip.h), both storage types.
#include "dwconv_band.hip.h"
#include "dwconv_host.hip.h"

namespace dwhost {

// Returns -1 when no geometry fits.
template <typename E>
static int launch_corr_band(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    constexpr int NL = dwconv::Limbs<E>::N;
    BandPlan p;
    if (!plan_corr_band(s, pad_eff, reverse, &p)) return -1;
    auto go = [&](auto kernel) -> int {
        if (p.lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        // (a grid dimension holds fewer than 2^32 threads: further channels in launches of their own)
        for (int c0 = 0; c0 < s.C; c0 += kMaxGridChannels) {
            const int n = s.C - c0 < kMaxGridChannels ? s.C - c0 : kMaxGridChannels;
            hipLaunchKernelGGL(kernel, dim3((unsigned)n, (unsigned)p.gy), dim3(dwconv::kBandThreads), p.lds, st,
                               static_cast<const E *>(in) + (size_t)c0 * (size_t)s.L, static_cast<const E *>(f) + (size_t)c0 * (size_t)s.K,
                               static_cast<E *>(out) + (size_t)c0 * (size_t)s.L, p.g);
        }
        return launch_status();
    };
    switch (p.T) {
    case 1:
        if constexpr (NL == 3) {
            if (p.g.F < s.K) return go(dwconv::corr_band_kernel<E, 1, true>);
        }
        return go(dwconv::corr_band_kernel<E, 1>);
    case 2:
        if constexpr (NL == 3) {
            if (p.g.F < s.K) return go(dwconv::corr_band_kernel<E, 2, true>);
            if (p.few) return go(dwconv::corr_band_kernel<E, 2, false, dwconv::kBandPrefetchF32Few>);
        }
        return go(dwconv::corr_band_kernel<E, 2>);
    default:
        if constexpr (NL == 1) return go(dwconv::corr_band_kernel<E, 4>);
        else return -1;
    }
}

int launch_corr_band_f32(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    return launch_corr_band<float>(in, f, out, s, pad_eff, reverse, st);
}
int launch_corr_band_bf16(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    return launch_corr_band<bf16_t>(in, f, out, s, pad_eff, reverse, st);
}

}  // namespace dwhost
