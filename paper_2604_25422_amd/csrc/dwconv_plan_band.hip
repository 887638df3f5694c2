// Plans of the kernels for long filters: geometry from the shape alone.  Host code only, and no kernel is named here: a test builds
// this unit for itself and follows the operand addresses of what is planned.
#include "dwconv_host.hip.h"
#include <algorithm>

namespace dwhost {

// ---- stage 1 of the weight gradient, dw_band_kernel

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

}  // namespace dwhost
