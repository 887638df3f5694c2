// Stage 1 of the weight gradient for long filters (dwconv_dw_band.hip.h), both storage types: the plan and the launchers.
#include "dwconv_dw_band.hip.h"
#include "dwconv_host.hip.h"
#include <algorithm>

namespace dwhost {

namespace {

// floor division
int fdiv(long long a, int b) { return (int)(a >= 0 ? a / b : -((-a + b - 1) / b)); }

}  // namespace

// Depends on the shape only.  False: no geometry (rows of fewer than four positions).  slices: those of the
// workspace, at least as many as the plan uses.
bool plan_dw_band(const Shape &s, int slices, DwBandPlan *p)
{
    if (s.L < 4 || s.L > kMfmaMaxL) return false;
    dwconv::DwBandGeom &g = p->g;
    const int NL = s.dtype == DWCONV_F32 ? 3 : 1;
    const int nb32 = (s.L + 31) / 32;
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K; g.pad = s.pad;
    int dmin = -fdiv((long long)s.pad + 31, 32), dmax = fdiv((long long)s.K - 1 - s.pad + 31, 32);
    if (dmin < -(nb32 - 1)) dmin = -(nb32 - 1);
    if (dmax > nb32 - 1) dmax = nb32 - 1;
    g.dmin = dmin;
    g.nd = dmax - dmin + 1;
    // offsets per wave and offset groups: at most twelve offsets per window in fp32 (32 accumulator registers each), sixteen in
    // bf16, as few idle ones as possible
    {
        const int most = NL == 3 ? 12 : 16;
        const int nwin = g.nd <= most ? 1 : (g.nd - 1 + most - 2) / (most - 1);
        const int per = nwin == 1 ? g.nd : (g.nd - 1 + nwin - 1) / nwin + 1;
        if (per <= 3) { p->ND = per; g.dg_log = 0; }
        else if (per <= 4) { p->ND = 2; g.dg_log = 1; }
        else if (per <= 6) { p->ND = 3; g.dg_log = 1; }
        else if (per <= 8) { p->ND = 2; g.dg_log = 2; }
        else if (per <= 12) { p->ND = 3; g.dg_log = 2; }
        else { p->ND = 4; g.dg_log = 2; }
        g.ndw = p->ND << g.dg_log;
        g.nwin = g.nd <= g.ndw ? 1 : (g.nd - 1 + g.ndw - 2) / (g.ndw - 1);
    }
    // fewer than eight rows: several virtual rows per row
    g.nseg = s.B >= 5 ? 1 : 8 / s.B;
    if (g.nseg > (s.L + 127) / 128) g.nseg = (s.L + 127) / 128;
    g.Lv = 1 << 30;
    if (g.nseg > 1) {
        g.Lv = (int)((((long long)s.L + g.nseg - 1) / g.nseg + 63) / 64 * 64);
        g.nseg = (s.L + g.Lv - 1) / g.Lv;
        if (g.nseg == 1) g.Lv = 1 << 30;
    }
    g.seg_magic = 65536u / (unsigned)g.nseg + 1u;
    const int nbv = g.nseg > 1 ? g.Lv / 32 : nb32;
    const int BB = dwconv::dw_band_block_bytes(NL);
    const int blocks = (int)(kMaxLdsBytes / 2) / BB;                   // of a stage: two workgroups per compute unit
    auto x_blocks = [&](int S32) { const int n = S32 + g.ndw - 1; return g.nseg == 1 && n > nb32 + 2 ? nb32 + 2 : n; };
    // (one item per thread and tensor: at most 32 blocks of either for the four waves)
    g.S32 = (nbv + 1) / 2 * 2;
    while (g.S32 > 2 && (g.S32 + x_blocks(g.S32) > blocks || g.S32 > 32 || x_blocks(g.S32) > 32)) g.S32 -= 2;
    g.nstep = (nbv + g.S32 - 1) / g.S32;
    g.S32 = ((nbv + g.nstep - 1) / g.nstep + 1) / 2 * 2;
    const long long VR = (long long)s.B * g.nseg;
    g.rg_log = 0;
    while (g.nstep == 1 && g.rg_log < 2 && (16ll << g.rg_log) <= VR && (2 << g.rg_log) * (g.S32 + x_blocks(g.S32)) <= blocks &&
           (2 << g.rg_log) * x_blocks(g.S32) <= 32 && (2 << g.rg_log) * g.S32 <= 32) ++g.rg_log;
    p->split = g.nseg == 1 && g.nstep == 1 && g.rg_log < 2 && 8 * nb32 <= 32 * (4 >> g.rg_log) && 8 * g.S32 <= 32 * (4 >> g.rg_log);
    const long long groups = (VR + (8 << g.rg_log) - 1) / (8 << g.rg_log);
    if (groups * g.nstep > 0x3fffffff || VR > 0x3fffffff) return false;
    g.stages = (int)(groups * g.nstep);
    g.step_magic = (long long)g.stages * g.nstep < (1ll << 32) ? (unsigned)((1ull << 32) / (unsigned)g.nstep) + 1u : 0u;
    g.rev = s.pad >= s.K / 2 ? 1 : 0;
    g.fold = 4ll * s.pad < s.K || 4ll * (s.K - 1 - s.pad) < s.K ? (1 << g.dg_log) - 1 : 0;
    // slices that are used: about two rounds of two workgroups per compute unit (a workgroup's start and its diagonal sums do
    // not shrink with its stages: B8 C256 K = L = 8192 with one slice 745 us, two 837 us; bf16 232 / 286), partial sums of at
    // most 16 MiB
    long long S = (4ll * kComputeUnits + (long long)s.C * g.nwin - 1) / ((long long)s.C * g.nwin);
    S = std::min(S, (16ll << 20) / ((long long)s.C * s.K * 4));
    S = std::min(S, (long long)std::min(g.stages, slices));
    p->S = S < 1 ? 1 : (int)S;
    p->lds = dwconv::dw_band_lds_bytes(NL, 1 << g.rg_log, g.S32, x_blocks(g.S32) - g.S32 + 1, p->ND);
    return true;
}

template <typename E>
static int launch_dw_band(const void *x, const void *dy, float *part, void *dw_out, const DwBandPlan &p, int slices, hipStream_t st)
{
    auto go = [&](auto kernel) -> int {
        if (p.lds > 64 * 1024 && !allow_large_lds(kernel)) return DWCONV_ERR_LAUNCH;
        // (a grid holds fewer than 2^32 threads along channels and 65536 windows: what is beyond in launches of their own)
        dwconv::DwBandGeom g = p.g;
        for (g.win0 = 0; g.win0 < p.g.nwin; g.win0 += 65535) {
            const int nz = p.g.nwin - g.win0 < 65535 ? p.g.nwin - g.win0 : 65535;
            for (int c0 = 0; c0 < g.C; c0 += kMaxGridChannels) {
                const int n = g.C - c0 < kMaxGridChannels ? g.C - c0 : kMaxGridChannels;
                const size_t row = (size_t)c0 * (size_t)g.L, taps = (size_t)c0 * (size_t)g.K;
                hipLaunchKernelGGL(kernel, dim3((unsigned)n, (unsigned)p.S, (unsigned)nz), dim3(dwconv::kDwBandThreads), p.lds, st,
                                   static_cast<const E *>(x) + row, static_cast<const E *>(dy) + row, part + taps,
                                   dw_out ? static_cast<E *>(dw_out) + taps : nullptr, g, slices);
            }
        }
        return launch_status();
    };
    auto form = [&](auto nd, auto dg) -> int {
        constexpr int ND = decltype(nd)::value, DG = decltype(dg)::value;
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
