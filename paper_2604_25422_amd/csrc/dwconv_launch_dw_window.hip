// Stage 1 of the weight gradient with the operands in registers (dwconv_dw_window.hip.h): plan and launcher.
#include "dwconv_dw_window.hip.h"
#include "dwconv_host.hip.h"

namespace dwhost {

// Depends on the shape only.  False: the kernel does not apply.  slices: those of the workspace, at least as many as the plan uses.
bool plan_dw_window(const Shape &s, int slices, DwWinPlan *p)
{
    dwconv::DwWinGeom &g = p->g;
    // (byte offsets inside a unit stay below the out-of-row marker)
    if (s.dtype != DWCONV_F32 || s.L <= dwconv::kRbMaxL || s.L > kMfmaMaxL || 64ll * s.C * s.L >= (1ll << 30)) return false;
    const int nb32 = (s.L + 31) / 32;
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K; g.pad = s.pad;
    g.dmin = std::max(-(int)((s.pad + 31ll) / 32), -(nb32 - 1));
    g.nd = std::min((int)((s.K - 1ll - s.pad + 31) / 32), nb32 - 1) - g.dmin + 1;
    if (g.nd > dwconv::kDwWinND) return false;
    const int ND = std::max(g.nd, 4);
    p->ND = ND;
    // Pieces of a row and slices: the least of what a wave has to do in the rounds its workgroup takes (cycles).  A product takes 48 with what is
    // done beside it, a step without products 900, start and sums of a workgroup 14000, a second launch 8000.
    double best = 0.0;
    for (int np = 1; np <= 16 && np <= (s.L + 255) / 256; ++np) {
        const int P = ((s.L + np - 1) / np + 63) / 64 * 64, NP = (s.L + P - 1) / P;
        if (NP != np || (np > 1 && P < 32 * (g.nd + 2))) continue;
        const long long units = ((long long)s.B * NP + 15) / 16;
        if (units * 16 * NP >= (1ll << 32) || units > 0x3fffffff) continue;
        const int nb = NP > 1 ? P / 32 : nb32, chi = NP > 1 ? 1 << 28 : nb32 - 1;
        const int s_first = (NP > 1 ? -(ND - 1) : std::max(-(ND - 1), -g.dmin - (ND - 1))) & ~1, s_end = (std::min(nb, chi - g.dmin + 1) + 1) & ~1;
        const int with = std::min(nb, s_end) - std::max(0, s_first), without = s_end - s_first - with;
        const double unit = with * 48.0 * 6 * ND + without * 900.0;
        for (int S = 1; S <= slices && S <= units; S = S < 8 ? S + 1 : S + S / 4) {
            const long long wave = (units + (long long)dwconv::kDwWinWaves * S - 1) / ((long long)dwconv::kDwWinWaves * S);
            const long long rounds = ((long long)s.C * S + kComputeUnits - 1) / kComputeUnits;
            const double cost = (double)rounds * ((double)wave * unit + 14000.0) + (S > 1 ? 8000.0 : 0.0);
            if (best == 0.0 || cost < 0.99 * best) {
                best = cost;
                p->S = S;
                g.NP = NP; g.P = P; g.np_magic = NP > 1 ? (unsigned)((1ull << 32) / (unsigned)NP) + 1u : 0u;
                g.units = (int)units;
                g.rem = NP > 1 ? (s.L >> 5) % (P >> 5) : s.L >> 5;
            }
            if ((long long)s.C * S > 2ll * kComputeUnits) break;
        }
    }
    p->cycles = best;
    return best > 0.0;
}

int launch_dw_window_f32(const void *x, const void *dy, float *part, void *dw_out, const DwWinPlan &p, int slices, hipStream_t st)
{
    auto go = [&](auto kernel) -> int {
        if (!allow_large_lds(kernel)) return DWCONV_ERR_LAUNCH;
        hipLaunchKernelGGL(kernel, dim3((unsigned)p.g.C, (unsigned)p.S), dim3(dwconv::kDwWinThreads), (size_t)dwconv::dw_win_lds_bytes(), st,
                           static_cast<const float *>(x), static_cast<const float *>(dy), part, static_cast<float *>(dw_out), p.g, slices);
        return launch_status();
    };
    return p.ND == 4 ? go(dwconv::dw_window_kernel<4>) : go(dwconv::dw_window_kernel<5>);
}

}  // namespace dwhost
