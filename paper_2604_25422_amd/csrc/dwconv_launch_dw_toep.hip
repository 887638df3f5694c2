// Stage 1 of the weight gradient for filters of hundreds of taps and more (dwconv_dw_toep.hip.h), both storage types: the plan
// and the launchers.
#include "dwconv_dw_toep.hip.h"
#include "dwconv_host.hip.h"
#include <algorithm>

namespace dwhost {

// Depends on the shape only.  False: no geometry (rows of fewer than eight positions, more pieces than a grid holds).
// slices: those of the workspace, at least as many as the plan uses.
bool plan_dw_toep(const Shape &s, int slices, DwToepPlan *p)
{
    if (s.L < 8 || s.L > kMfmaMaxL) return false;
    dwconv::DwToepGeom &g = p->g;
    const int NL = s.dtype == DWCONV_F32 ? 3 : 1;
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K; g.pad = s.pad;
    const long long first = std::max(-(long long)s.pad, -(long long)(s.L - 1)), last = std::min((long long)s.K - 1 - s.pad, (long long)s.L - 1);
    // Tiles start at the first lag or end at the last, whichever leaves less work: the lags of a tile that is not full should be the far
    // ones, which meet few positions (causal: bf16 B32 C256 L4097 K4097, four tiles and one lag, 272 -> 202 us; fp32 B6 C71 L1967 K1967 30 -> 19)
    const int tiles = (int)((last - first) / 1024) + 1;
    // products of 32 x 32 x 16 of a batch entry for tile t of those that start at lag o0
    auto tile_work = [&](long long o0, int t) {
        const long long o = o0 + 1024ll * t, from = std::max(0ll, -(o + 1023)), to = std::min((long long)s.L, s.L - o);
        return to > from ? (double)((to - from + 30) / 16 + 1) : 0.0;
    };
    const long long end = last + 1 - 1024ll * tiles;
    double from_first = 0.0, to_last = 0.0;
    for (int t = 0; t < tiles; ++t) {
        from_first += tile_work(first, t);
        to_last += tile_work(end, t);
    }
    const long long o0 = to_last < from_first ? end : first;
    g.blk0 = (int)(o0 >> 5);
    g.shift = (int)(o0 & 31);
    g.nblk = (int)((last - o0) >> 5) + 1;
    // tiles per workgroup: two while there are three workgroups per compute unit (B8 C256 K = L = 8192: 1024 workgroups of two, 2048 of
    // one: bf16 125 / 152 us, fp32 618 / 658.  Four, bf16, take the registers of a third workgroup: B16 C400 L8192 437 us with two, 470 with
    // four, B8 C768 L4096 121 / 125, B8 C1024 L4096 centred 205 / 192)
    p->T = 2;
    while (p->T > 1 && (p->T / 2 >= tiles || (long long)s.C * ((tiles + p->T - 1) / p->T) < 3 * kComputeUnits)) p->T /= 2;
    g.npiece = (tiles + p->T - 1) / p->T;
    if (g.npiece > 65535) return false;
    // chunks of equal length, as few as fit half the LDS of a compute unit (a third where registers allow a third workgroup)
    const size_t budget = kMaxLdsBytes / (size_t)dwconv::toep_waves(NL, p->T);
    const int whole = (s.L + 31) / 32 + 64;                               // blocks of X that any tile can reach
    for (int n = 1;; ++n) {
        g.F = (int)((((long long)s.L + n - 1) / n + 31) / 32 * 32);
        const int blocks = std::min(dwconv::toep_blocks(p->T, g.F), whole);
        p->lds = dwconv::dw_toep_lds_bytes(NL, blocks, g.F);
        g.tap_off = (int)dwconv::dw_toep_tap_offset(NL, blocks);
        if (4 * blocks <= dwconv::kToepX * dwconv::kToepThreads && g.F <= 8 * dwconv::kToepY * dwconv::kToepThreads && p->lds <= budget) break;
    }
    // the products of a batch entry: in all, and of the piece that has most
    double most = 0.0;
    p->work = std::min(from_first, to_last);
    for (int i = 0; i < g.npiece; ++i) {
        double piece = 0.0;
        for (int t = i * p->T; t < std::min(tiles, (i + 1) * p->T); ++t) piece += tile_work(o0, t);
        most = std::max(most, piece);
    }
    // slices: three workgroups per compute unit and none with more than its share, as far as the batch and the workspace go, where
    // that is worth a second launch (fp32 B11 C64 L4135 K4135 139 us in one slice)
    const long long wgs = (long long)s.C * g.npiece, slots = 3ll * kComputeUnits;
    const long long stages = (long long)s.B * (((long long)s.L + g.F - 1) / g.F);
    const double us = 1.2 * stages + most * s.B * (NL == 3 ? 6 : 1) * 32.0 / 4 / 2000.0;      // (of a workgroup that has its SIMDs to itself)
    long long S = 1;
    if (us > 10.0) S = std::min((long long)(us / 4.0), std::max((slots + wgs - 1) / wgs, (long long)(most * slots / (p->work * s.C) + 0.5)));
    S = std::max(1ll, std::min(S, (long long)std::min(s.B, slices)));
    g.rows = (int)((s.B + S - 1) / S);
    p->S = (s.B + g.rows - 1) / g.rows;
    // The e between two additions to the totals (four waves).  An element sums N = rows x L / 64 products of the instruction and wave; chains of
    // root N of them, and as many totals, are the shortest of two levels.
    // bf16: chains end with a stage, a break costs 5 % (B1 C544 L6988 46.4 -> 48.8 us): only few batch entries, whose error was small on
    // dw_band_kernel's virtual rows, have them inside one.  Error of the sums before they are rounded to bf16, dw_band_kernel -> here
    // without totals -> with (normal data): B8 L8192 2.3e-7, 6.7e-7, 1.9e-7, B32 L4097 3.3e-7, 9.5e-7, 1.9e-7, B1 L5952 0.91e-7, 1.9e-7,
    // 0.85e-7, B2 L1150 0.78e-7, 1.2e-7, 0.77e-7; what they cost: B8 C256 L8192 130 -> 131 us, B12 C355 L1832 43 -> 46, B2 C384 L1150 7.2 -> 8.4
    const int sets = dwconv::toep_sets(NL, p->T);
    int root = 4;
    while ((long long)(root + 1) * (root + 1) <= (long long)g.rows * s.L / (64 * sets)) ++root;
    g.chain = 4 * sets * root;
    g.run = s.B < 5 ? 4 * sets * root : 1 << 24;
    // fp32: the fewer products a gradient sums, the shorter were the chains of
    // the kernel this one replaced; with these its error against 64 bits is what it was: few rows, as long chains of products as of totals
    // (B1 L5664 1.5e-7 without a limit, 1.0e-7 with 32 and with 16, dw_band_kernel 1.0e-7); B9 L3000 1.26e-7, 1.05e-7 with 32 (1.07e-7);
    // B8 L8192 1.43e-7 without one (1.65e-7).  What they cost: B8 C256 L8192 K8192 641 us, 667 with 64, 715 with 32
    if (NL == 3) {
        int root_l = 4;
        while ((root_l + 1) * (root_l + 1) <= s.L / 64) ++root_l;
        g.run = s.B < 5 ? 4 * root_l : (long long)s.B * s.L < 65536 ? 32 : 1 << 24;
    }
    p->work *= s.B;
    return true;
}

template <typename E>
static int launch_dw_toep(const void *x, const void *dy, float *part, void *dw_out, const DwToepPlan &p, int slices, hipStream_t st)
{
    auto go = [&](auto kernel) -> int {
        if (p.lds > 64 * 1024 && !allow_large_lds(kernel)) return DWCONV_ERR_LAUNCH;
        // (a grid dimension holds fewer than 2^32 threads: further channels in launches of their own)
        for (int c0 = 0; c0 < p.g.C; c0 += kMaxGridChannels) {
            const int n = p.g.C - c0 < kMaxGridChannels ? p.g.C - c0 : kMaxGridChannels;
            const size_t row = (size_t)c0 * (size_t)p.g.L, taps = (size_t)c0 * (size_t)p.g.K;
            hipLaunchKernelGGL(kernel, dim3((unsigned)n, (unsigned)p.S, (unsigned)p.g.npiece), dim3(dwconv::kToepThreads), p.lds, st,
                               static_cast<const E *>(x) + row, static_cast<const E *>(dy) + row, part + taps,
                               dw_out ? static_cast<E *>(dw_out) + taps : nullptr, p.g, slices);
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
