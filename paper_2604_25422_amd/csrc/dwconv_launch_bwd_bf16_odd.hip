// Fused backward kernel, bf16 rows that do not all start on a dword.
#include "dwconv_launch_bwd.hip.h"

namespace dwhost {

// Ordinary rows from kRaggedMinL positions on (the kernel contracts whole segments, as on other rows that are not whole granules), x, dy
// and dx on the same half of a dword; workgroups of sixteen waves or four, whatever other number the plan has.  Returns -1 when it
// does not apply.  The two separate kernels -> here, us for both gradients: B32 C256 L4097 K64 57 -> 49,
// B64 C512 L2047 K7 106 -> 91, B300 C100 L999 K50 60 -> 47, B100 C64 L1701 K33 29 -> 20, B4 C64 L1023 K16 7.8 -> 7.7.
int launch_bwd_fused_bf16_odd(const void *dy, const void *x, const void *w, void *dx, float *part, void *dw_out, bool *wrote_dw,
                              const Shape &s, const DwPlan &p, int dmin, int nd, hipStream_t st)
{
    if (p.rows.on || p.rows.batch || p.rows.tall || s.L < kRaggedMinL || (long long)s.B * s.C >= (1ll << 31) ||
        bf16_odd_small_call(s, p.rows) || aligned_to(x, 4) != aligned_to(dy, 4) || aligned_to(x, 4) != aligned_to(dx, 4))
        return -1;
    void *direct = (p.single && p.S == 1) ? dw_out : nullptr;
    auto go = [&](auto ndc, auto wc) -> int {
        constexpr int ND = decltype(ndc)::value, W = decltype(wc)::value;
        auto kernel = dwconv::bwd_fused_bf16_kernel<ND, W, false, true>;
        constexpr size_t lds = dwconv::bwd_fused_bf16_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        // (a shifted row may reach one position into a segment more)
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st, static_cast<const bf16_t *>(dy),
                           static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(w), static_cast<bf16_t *>(dx), part,
                           static_cast<bf16_t *>(direct), s.B, s.C, s.L, s.K, s.pad, dmin,
                           (s.L + 1 + dwconv::kSegLen - 1) / dwconv::kSegLen, p.rows.map, aligned_to(x, 4) ? 0 : 1);
        return launch_status();
    };
    auto waves = [&](auto ndc) -> int {
        return p.wpb == 16 ? go(ndc, std::integral_constant<int, 16>{}) : go(ndc, std::integral_constant<int, 4>{});
    };
    int rc = -1;
    switch (nd) {
    case 2: rc = waves(std::integral_constant<int, 2>{}); break;
    case 3: rc = waves(std::integral_constant<int, 3>{}); break;
    case 4: rc = waves(std::integral_constant<int, 4>{}); break;
    case 5: rc = waves(std::integral_constant<int, 5>{}); break;
    case 6: rc = waves(std::integral_constant<int, 6>{}); break;
    default: break;
    }
    if (rc == DWCONV_OK && direct) *wrote_dw = true;
    return rc;
}

}  // namespace dwhost
