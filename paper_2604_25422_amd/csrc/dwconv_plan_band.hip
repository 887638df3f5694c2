// Plans of the kernels for long filters: geometry from the shape alone.  Host code only, and no kernel is named here: a test builds
// this unit for itself and follows the operand addresses of what is planned.
#include "dwconv_host.hip.h"
#include <algorithm>

namespace dwhost {

// ---- forward and input gradient, corr_band_kernel

// False: no geometry fits.
bool plan_corr_band(const Shape &s, int pad_eff, int reverse, BandPlan *p)
{
    const int NL = s.dtype == DWCONV_F32 ? 3 : 1;
    const int nb32 = (s.L + 31) / 32;
    dwconv::BandGeom &g = p->g;
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K; g.pad = pad_eff; g.reverse = reverse;
    if (s.L < 8 || s.L > kMfmaMaxL) return false;
    const int TMAX = NL == 3 ? 2 : 4;
    int T = 1, NBk = 1, window_blocks = 0;
    long long row_groups = 1;
    // Geometry with columns of 2^nb_log blocks; false when window and taps do not fit (half the LDS of a compute unit, the
    // prefetch registers).  whole_filter: only with all taps in one chunk.
    auto fit = [&](int nb_log, bool whole_filter) -> bool {
        g.nb_log = nb_log;
        NBk = 1 << nb_log;
        g.RW = 32 >> nb_log;
        const int row_tiles = (nb32 + NBk - 1) / NBk;
        row_groups = ((long long)s.B + g.RW - 1) / g.RW;
        if (nb32 <= 32) {
            // short rows: one item is RW whole rows, a tile for every wave first
            g.TG = row_tiles >= 3 ? 4 : row_tiles;
            T = (row_tiles + g.TG - 1) / g.TG;
            if (T == 3) T = 4;
            if (T > TMAX) return false;
        } else {
            // eight tiles per item.  Filters of up to 512 taps are bound by memory: every wave its own tiles, nothing to add
            // up afterwards (bf16 B32 C256 L4096, TG = 4 / 2: K = 226 41 / 49 us, K = 300 46 / 51 us); longer ones by the
            // matrix pipe and LDS: more tiles per tap operand and shorter sums (fp32 K = L = 8192 633 us, 818 us with TG = 4).
            // Two tiles per wave in fp32 too, though one would leave room for a third workgroup (two / one: L4096 K200 104 / 108 us,
            // K300 125 / 128, K500 182 / 196; B100 C256 L700 K400 100 / 129; short rows B2048 C128 L256 K256 178 / 200)
            T = s.K <= 512 ? 2 : TMAX;
            g.TG = T == 2 && s.K <= 512 ? 4 : 2;
        }
        // fewer tiles per item where there would be less than two workgroups per compute unit (one for items of two tiles:
        // B1 C64 L13934 K226 fp32 7.0 us with two, 8.6 with one; B1 C130 L3148 K130 bf16 4.9 / 5.5)
        while (T * g.TG > 1 && (T * g.TG / 2 >= row_tiles || s.C * row_groups * ((row_tiles + T * g.TG - 1) / (T * g.TG)) <
                                                                 (T * g.TG > 2 ? 2 : 1) * kComputeUnits)) {
            if (T > 1) T /= 2;
            else g.TG /= 2;
        }
        // rows a little longer than one item: pieces of equal length instead of a second one of a tile or two (fp32 B16 C256
        // L2100 K400 53 -> 44 us), bf16 also of half the tiles (B8 C512 L2300: K = 200 20.1 -> 17.5, 1000 35 -> 29)
        const int rest = nb32 - T * g.TG * NBk;
        const bool two = nb32 > 32 && rest > 0 && rest <= 2 * NBk;
        if (two && NL == 1 && rest > 2 && T * g.TG == 8) T /= 2;
        const int pieces = (row_tiles + T * g.TG - 1) / (T * g.TG);
        g.PB = (two ? (row_tiles + pieces - 1) / pieces : std::min(T * g.TG, row_tiles)) * NBk;
        const int whole = nb32 + 2 * (NBk - 1);
        for (int F = s.K < 32768 ? (s.K + 1) & ~1 : 32768;; F = (F - 1) / 32 * 32) {
            if (F < s.K && (F <= 64 || whole_filter)) return false;       // (a chunk is 65 taps at least; a shorter filter is one chunk)
            g.F = F;
            int wb = g.PB + (F + 46) / 32 + 2;
            if (wb > whole) wb = whole;
            // rows of the window lie as if their blocks went on from one row to the next (16-byte units modulo 16): sixteen
            // neighbouring lanes then read sixteen different groups of banks
            int units = wb * (dwconv::band_block_bytes(NL) / 16);
            while (((units - NBk * (dwconv::band_block_bytes(NL) / 16)) & 15) != 0) ++units;
            g.pitch = 16 * units;
            if (g.RW * wb * 4 <= dwconv::band_prefetch(NL) * dwconv::kBandThreads &&
                (F >= s.K || dwconv::band_tap_dwords(F) <= dwconv::kBandTapPrefetch * dwconv::kBandThreads) &&
                dwconv::band_lds_bytes(NL, g.RW, g.pitch, F) <= kMaxLdsBytes / 2) {
                window_blocks = wb;
                return true;
            }
        }
    };
    // Columns of a tile: few blocks of many batch entries for short rows (every column is then at the same distance from the
    // ends of its row, and block pairs outside the row cost nothing), more blocks where the batch is small.
    int nb_min = nb32 <= 8 ? 0 : nb32 <= 16 ? 1 : nb32 <= 32 ? 2 : 3;
    while (nb_min < 5 && (32 >> nb_min) >= 2 * s.B) ++nb_min;
    bool ok = false;
    // (all taps at once where some form holds them: B8 C256 L8192 K8192 bf16 141 us with 16 blocks and all taps, 177 us with 8
    // blocks in chunks; otherwise chunks, the same shape in fp32 634 us with 16 blocks and 642 us with 8)
    for (int nb = nb_min; nb <= 5 && !ok; ++nb) ok = fit(nb, true);
    for (int nb = nb_min < 4 && nb32 > 32 ? 4 : nb_min; nb <= 5 && !ok; ++nb) ok = fit(nb, false);
    if (!ok) return false;
    g.NP = (nb32 + g.PB - 1) / g.PB;
    // Tiles q, 2 TG - 1 - q, ... for wave group q where the work of a tile falls along the row, the same from the end of the row where it
    // grows (spare tiles are where there is little to do); q, TG + q, ... where it is largest in the middle, or an item is not the
    // whole row and its tiles differ little (fp32 B19 C303 L1356 K1356 causal forward 85 us, 91 the other way).  Causal, forward and
    // input gradient, us: fp32 B2048 C128 L256 K256 169 -> 163, 164 -> 157, B186 C69 L736 K736 61 -> 57, 59 -> 54, B1 C583 L3040 K3040
    // 47 -> 42, 47 -> 42
    g.fold = g.NP == 1 && (4ll * pad_eff < s.K || 4ll * (s.K - 1 - pad_eff) < s.K) ? g.TG - 1 : 0;
    g.tile0 = g.fold && 2 * pad_eff > s.K ? (g.PB >> g.nb_log) - T * g.TG : 0;
    g.np_magic = g.NP > 1 ? (unsigned)((1ull << 32) / (unsigned)g.NP) + 1u : 0u;
    if (row_groups * g.NP * g.NP > 0xffffffffll || row_groups * g.NP > 0x3fffffff) return false;
    g.items = (int)(row_groups * g.NP);
    const size_t lds = dwconv::band_lds_bytes(NL, g.RW, g.pitch, g.F);
    // fp32, two tiles per wave: a third workgroup per compute unit where window and prefetch are small enough for it (two / three:
    // B2048 C128 L160 K160 117 / 104 us, B16 C256 L2100 K400 48.4 / 42.5, B1000 C128 L224 K100 70 / 65)
    const bool few = NL == 3 && T == 2 && g.F >= s.K && 3 * lds <= kMaxLdsBytes &&
                     g.RW * window_blocks * 4 <= dwconv::kBandPrefetchF32Few * dwconv::kBandThreads;
    // workgroups per channel: whole rounds of the resident ones, items spread evenly; a workgroup's start (its taps, a
    // first window that nothing hides) counts as half an item
    const int by_lds = (int)(kMaxLdsBytes / lds), by_regs = dwconv::band_waves(NL, T, few ? dwconv::kBandPrefetchF32Few : dwconv::band_prefetch(NL));
    const long long slots = (long long)kComputeUnits * (by_lds < by_regs ? by_lds : by_regs);
    int gy = 1;
    double best = 0.0;
    for (int y = 1; y <= g.items && y <= 4096; ++y) {
        const double rounds = (double)(((long long)s.C * y + slots - 1) / slots);
        const double cost = rounds * ((double)((g.items + y - 1) / y) + 0.5);
        if (y == 1 || cost < best * 0.999) { best = cost; gy = y; }
        if ((long long)s.C * y > 16 * slots) break;
    }
    p->T = T;
    p->few = few;
    p->gy = gy;
    p->lds = lds;
    return true;
}

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
    const long long wgs = (long long)s.C * g.nwin, slots = 2ll * kComputeUnits;
    long long S = (2 * slots + wgs - 1) / wgs;
    S = std::min(S, (16ll << 20) / ((long long)s.C * s.K * 4));
    S = std::max(1ll, std::min(S, (long long)std::min(g.stages, slices)));
    p->S = (int)S;
    // ... fp32, one window of offsets (its workgroups then take equally long): fewer, at least half, where that fills the last round of workgroups,
    // which was a nearly empty one.  Where a slice then has more stages, a workgroup sums them in two chains of additions (CHAINS), so that none is longer
    // than with S slices; what the second one costs (its start and its sums, 8 us a round) is only there from five stages on.  (Both in us: a start
    // with its diagonal sums, a stage.)  S slices -> fewer, us and error against 64 bits (normal data): B1310 C48 L192 K192, 528 workgroups of which 512
    // run at once -> 480, 56 -> 43, 1.28e-7 -> 1.12e-7; B2294 C96 L144 K176 155 -> 108, 1.7e-7 -> 1.5e-7; B3217 C36 L189 K189 99 -> 70, 1.6e-7 -> 1.4e-7;
    // in one chain, which is as long as before, B109 C96 L3056 K223 138 -> 118, 2.0e-7 -> 2.1e-7, B552 C69 L130 K130 35 -> 29, 1.10e-7 -> 1.13e-7.  Of
    // 412 calls 44 take two chains (mean gain 1.25, the worst 1.03, mean error 0.84 of that of S slices) and 29 fewer slices in one (1.19, 1.02, 1.01).
    // (One chain of more stages: error up to 1.46 times that of S slices.  bf16 waits for memory, and a workgroup more than fits takes up some
    // of the wait: B254 C508 L306 K243 53 / 61, B225 C288 L144 K228 24 / 32)
    g.chain = 0;
    if (NL == 3 && g.nwin == 1) {
        const long long most = (g.stages + S - 1) / S;
        double best = 0.0;
        for (long long t = S; t == S || (t > 1 && 2 * t >= S); --t) {          // (one slice would be the gradient, written once)
            const long long rounds = (wgs * t + slots - 1) / slots, stages = (g.stages + t - 1) / t;
            const bool one = stages <= most;                                   // (chain)
            const double cost = (double)rounds * ((one ? 5.9 : 13.9) + (0.4 + 0.056 * g.S32 * p->ND) * (double)stages);
            if (t == S || (cost < 0.95 * best && 20 * wgs * t >= 17 * rounds * slots && (one || stages >= 5))) {
                best = cost;
                p->S = (int)t;
                g.chain = one ? 0 : (int)(stages + 1) / 2;
            }
        }
    }
    p->lds = dwconv::dw_band_lds_bytes(NL, 1 << g.rg_log, g.S32, x_blocks(g.S32) - g.S32 + 1, p->ND);
    return true;
}

// ---- ... dw_toep_kernel

// Depends on the shape only.  False: no geometry (rows of fewer than eight positions).
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
    g.piece0 = 0;
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
    // root N of them, and as many totals, are the shortest of two levels: longer ones add up errors, shorter ones cost time (fp32, short sums:
    // chains of eight, B9 C49 L1147 15.1 us, of five 16.4).
    // fp32, where each run is a chain: error against 64 bits (normal data), dw_band_kernel -> here, and us: B9 L3000 1.07e-7 -> 1.03e-7 (1.26e-7
    // without a limit), B1 C348 L5664 0.96e-7 -> 0.97e-7 (1.5e-7), 209 -> 105; C256 L8192: B8 2.3e-7 -> 1.7e-7, 789 -> 632 (chains of
    // eight: 715), B7 2.2e-7 -> 1.7e-7, 764 -> 555 (chains of eight: 1.9e-7, 622), B5 2.0e-7 -> 1.4e-7, 732 -> 404 (446)
    // bf16: chains end with a stage, a break costs 5 % (B1 C544 L6988 46.4 -> 48.8 us): only few batch entries, whose error was small on
    // dw_band_kernel's virtual rows, have them inside one.  Error of the sums before they are rounded to bf16, dw_band_kernel -> here
    // without totals -> with: B8 L8192 2.3e-7, 6.7e-7, 1.9e-7, B32 L4097 3.3e-7, 9.5e-7, 1.9e-7, B1 L5952 0.91e-7, 1.9e-7, 0.85e-7,
    // B2 L1150 0.78e-7, 1.2e-7, 0.77e-7; what they cost: B8 C256 L8192 130 -> 131 us, B12 C355 L1832 43 -> 46, B2 C384 L1150 7.2 -> 8.4
    const int sets = dwconv::toep_sets(NL, p->T);
    int root = NL == 3 && s.B >= 5 ? 8 : 4;
    while ((long long)(root + 1) * (root + 1) <= (long long)g.rows * s.L / (64 * sets)) ++root;
    g.chain = 4 * sets * root;
    g.run = NL == 3 || s.B < 5 ? 4 * sets * root : 1 << 24;
    p->work *= s.B;
    return true;
}

}  // namespace dwhost
