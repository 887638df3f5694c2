// Launchers of the forward / input-gradient kernels (templates on the storage type; instantiated by
// dwconv_launch_corr_f32.hip and dwconv_launch_corr_bf16.hip).
//   out = correlate(in, f_eff, pad_eff): the forward is (x, w, pad); the input gradient is (dy, reversed w, K-1-pad).
#pragma once
#include "dwconv_host.hip.h"
#include "dwconv_valu.hip.h"

namespace dwhost {

template <typename T>
int launch_corr_valu(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    constexpr int R = 4, THREADS = 256, KCH = 512;
    constexpr int TILE = R * THREADS;
    static_assert(TILE == dwconv::kSegLen, "plan_valu_rows counts tiles of this size");
    const ValuRows vr = plan_valu_rows(s);
    if (vr.on) {
        // short rows: tiles of the virtual row of every channel
        const long long blocks = (long long)s.C * vr.tiles;
        if (blocks > 0x7fffffffLL) return DWCONV_ERR_SHAPE;
        hipLaunchKernelGGL((dwconv::corr_valu_kernel<T, R, THREADS, KCH, true>), dim3((unsigned)blocks), dim3(THREADS), 0, st,
                           static_cast<const T *>(in), static_cast<const T *>(f), static_cast<T *>(out), s.C, s.L, s.K,
                           pad_eff, reverse, (int)vr.tiles, vr.map);
        return launch_status();
    }
    const long long tiles_per_row = ((long long)s.L + TILE - 1) / TILE;
    const long long blocks = (long long)s.B * s.C * tiles_per_row;
    if (blocks > 0x7fffffffLL) return DWCONV_ERR_SHAPE;
    hipLaunchKernelGGL((dwconv::corr_valu_kernel<T, R, THREADS, KCH, false>), dim3((unsigned)blocks), dim3(THREADS), 0, st,
                       static_cast<const T *>(in), static_cast<const T *>(f), static_cast<T *>(out), s.C, s.L, s.K,
                       pad_eff, reverse, (int)tiles_per_row, dwconv::RowsMap{0, 0, 0, 0, 0u, 0u});
    return launch_status();
}

// Rows of at most 128 positions: sixteen rows of a channel (or of two neighbouring channels) per unit.  The block
// offsets are cropped to those that stay inside a row of m 16-blocks (rows_batch_offsets), so a filter as long as the
// row or longer costs the block pairs of the row and nothing else.  Returns -1 when no kernel is compiled for the case.
// (seven to fifteen offsets: translation units of their own, dwconv_launch_corr_rows_*.hip)
int launch_corr_rowbatch_wide_f32(dwconv::RowBatchGeom &rg, int nd, const void *in, const void *f, void *out, const Shape &s,
                                  hipStream_t st);
int launch_corr_rowbatch_wide_bf16(dwconv::RowBatchGeom &rg, int nd, const void *in, const void *f, void *out, const Shape &s,
                                   hipStream_t st);

// The kernels for seven and more block offsets of rows of MB blocks (MB = 4: seven offsets at most).
template <typename T>
int launch_corr_rowbatch_wide_t(dwconv::RowBatchGeom &rg, int nd, const void *in, const void *f, void *out, const Shape &s,
                                hipStream_t st);

template <typename T, typename Kernel>
int launch_corr_rowbatch_kernel(Kernel kernel, dwconv::RowBatchGeom &rg, int nc, const void *in, const void *f, void *out,
                                const Shape &s, hipStream_t st)
{
    // one resident round of waves: J per channel group, each walking units j, j + J, ...
    // (bf16: as many as its registers allow - a wave has half the bytes in flight)
    const long long groups = s.C / nc;
    const long long resident = sizeof(T) == 2 ? resident_waves(kernel, 64 * dwconv::kRbCorrWaves) : corr_wave_slots(kernel, 64 * dwconv::kRbCorrWaves);
    long long J = resident / groups;
    if (J < 1) J = 1;
    if (J > rg.n_units) J = rg.n_units;
    const long long upw = (rg.n_units + J - 1) / J;
    J = (rg.n_units + upw - 1) / upw;
    const long long blocks = (groups * J + dwconv::kRbCorrWaves - 1) / dwconv::kRbCorrWaves;
    if (blocks > 0x1fffffffLL) return -1;
    rg.J = (int)J;
    const size_t lds = (size_t)dwconv::kRbCorrWaves * dwconv::rb_corr_wave_bytes(s.L, nc, (int)sizeof(T));
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * dwconv::kRbCorrWaves), lds, st,
                       static_cast<const T *>(in), static_cast<const T *>(f), static_cast<T *>(out), rg);
    return launch_status();
}

template <typename T>
int launch_corr_rowbatch_wide_t(dwconv::RowBatchGeom &rg, int nd, const void *in, const void *f, void *out, const Shape &s,
                                hipStream_t st)
{
    auto go = [&](auto kernel) -> int { return launch_corr_rowbatch_kernel<T>(kernel, rg, 1, in, f, out, s, st); };
    if (rg.m <= 4) return nd == 7 ? go(dwconv::corr_rowbatch_kernel<T, 7, 1, 4, false>) : -1;
    if constexpr (!std::is_same<T, float>::value) return -1;           // (bf16 rows of more than 64 positions: corr_band_kernel)
    else
    switch (nd) {
    case 7: return go(dwconv::corr_rowbatch_kernel<T, 7, 1, 8, false>);
    case 8: return go(dwconv::corr_rowbatch_kernel<T, 8, 1, 8, false>);
    case 9: return go(dwconv::corr_rowbatch_kernel<T, 9, 1, 8, false>);
    case 10: return go(dwconv::corr_rowbatch_kernel<T, 10, 1, 8, false>);
    case 11: return go(dwconv::corr_rowbatch_kernel<T, 11, 1, 8, false>);
    case 12: return go(dwconv::corr_rowbatch_kernel<T, 12, 1, 8, false>);
    case 13: return go(dwconv::corr_rowbatch_kernel<T, 13, 1, 8, false>);
    case 14: return go(dwconv::corr_rowbatch_kernel<T, 14, 1, 8, false>);
    case 15: return go(dwconv::corr_rowbatch_kernel<T, 15, 1, 8, false>);
    default: return -1;
    }
}

template <typename T>
int launch_corr_rowbatch(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse,
                         const RowsPlan &rp, hipStream_t st)
{
    int dmin, nd;
    rows_batch_offsets(s.L, s.K, pad_eff, &dmin, &nd);
    dwconv::RowBatchGeom rg;
    rg.B = s.B; rg.C = s.C; rg.L = s.L; rg.K = s.K;
    rg.pad = pad_eff; rg.reverse = reverse; rg.dmin = dmin;
    rg.m = (s.L + 15) / 16;
    rg.n_units = rp.units;
    // two channels per wave where that makes whole cache lines of rows that are not, or at least longer pieces;
    // rows of at most 48 positions and at most five block offsets (register budget of the kernel)
    // (two channels are one piece of 2 L elements cut into granules: rows of whole granules)
    const int nc = (s.C % 2 == 0 && (s.L * (int)sizeof(T)) % 128 != 0 && s.L <= 48 && nd <= 5 && (s.L % 4) == 0) ? 2 : 1;
    const bool rag = (s.L % 4) != 0;                   // rows that end inside a granule
    auto launch_batch = [&](auto kernel) -> int { return launch_corr_rowbatch_kernel<T>(kernel, rg, nc, in, f, out, s, st); };
    if (nd > kMfmaMaxND) {
        if (rag) return -1;
        if constexpr (std::is_same<T, float>::value) return launch_corr_rowbatch_wide_f32(rg, nd, in, f, out, s, st);
        else return launch_corr_rowbatch_wide_bf16(rg, nd, in, f, out, s, st);
    }
    if (nc == 2) {
        switch (nd) {
        case 2: return launch_batch(dwconv::corr_rowbatch_kernel<T, 2, 2, 3, false>);
        case 3: return launch_batch(dwconv::corr_rowbatch_kernel<T, 3, 2, 3, false>);
        case 4: return launch_batch(dwconv::corr_rowbatch_kernel<T, 4, 2, 3, false>);
        case 5: return launch_batch(dwconv::corr_rowbatch_kernel<T, 5, 2, 3, false>);
        default: return -1;
        }
    }
    if (rg.m <= 4) {
        switch (nd) {
        case 2: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 2, 1, 4, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 2, 1, 4, false>);
        case 3: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 3, 1, 4, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 3, 1, 4, false>);
        case 4: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 4, 1, 4, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 4, 1, 4, false>);
        case 5: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 5, 1, 4, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 5, 1, 4, false>);
        case 6: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 6, 1, 4, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 6, 1, 4, false>);
        default: return -1;
        }
    }
    switch (nd) {                              // rows of five to eight blocks
    case 2: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 2, 1, 8, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 2, 1, 8, false>);
    case 3: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 3, 1, 8, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 3, 1, 8, false>);
    case 4: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 4, 1, 8, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 4, 1, 8, false>);
    case 5: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 5, 1, 8, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 5, 1, 8, false>);
    case 6: return rag ? launch_batch(dwconv::corr_rowbatch_kernel<T, 6, 1, 8, true>) : launch_batch(dwconv::corr_rowbatch_kernel<T, 6, 1, 8, false>);
    default: return -1;
    }
}

// One launch of a forward / input-gradient kernel on the virtual rows of the channels (short rows, see RowsMap): slots
// ordered (virtual segment, channel).
template <typename T, typename Kernel>
int launch_corr_vrows_kernel(Kernel kernel, dwconv::CorrGeom g, const RowsPlan &rp, const void *in, const void *f, void *out,
                             const Shape &s, hipStream_t st)
{
    constexpr int kThreads = 64 * dwconv::kCorrWavesPerBlock;
    const long long total = (long long)rp.nvs * s.C;
    if (total > 0x3fffffffLL) return -1;
    g.rows = rp.nvs;
    g.segs_per_row = s.C;
    const long long resident = corr_wave_slots(kernel, kThreads);
    long long spw = (total + resident - 1) / resident;
    if (spw < 1) spw = 1;
    long long waves = (total + spw - 1) / spw;
    if (s.C <= resident) {                                // whole virtual segments per round: channel fixed
        long long J = resident / s.C;
        if (J > rp.nvs) J = rp.nvs;
        const long long rounds = (rp.nvs + J - 1) / J;
        J = (rp.nvs + rounds - 1) / rounds;
        waves = J * s.C;
    }
    const long long blocks = (waves + dwconv::kCorrWavesPerBlock - 1) / dwconv::kCorrWavesPerBlock;
    g.n_waves = (int)waves;
    g.step_rows = g.n_waves / g.segs_per_row;
    g.step_seg = g.n_waves % g.segs_per_row;
    g.step_c = 0;
    g.walk_segs = g.segs_per_row; g.n_main = g.n_waves; g.n_light = 0; g.step_c_light = 0;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, static_cast<const T *>(in),
                       static_cast<const T *>(f), static_cast<T *>(out), g, rp.map);
    return launch_status();
}// (fp32, seven to twelve block offsets on virtual rows: a translation unit of its own, dwconv_launch_corr_rows_f32.hip)
int launch_corr_vrows_wide_f32(const dwconv::CorrGeom &g, const RowsPlan &rp, int nd, const void *in, const void *f, void *out,
                               const Shape &s, hipStream_t st);

// Returns -1 when the shape or the pointers do not fit the matrix-core kernel.
template <typename T>
int launch_corr_mfma(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    const int dmin = toeplitz_dmin(pad_eff), dmax = toeplitz_dmax(s.K, pad_eff);
    const int nd = dmax - dmin + 1;
    const RowsPlan rp = plan_rows(s);
    // (the sixteen-row kernels of short rows move granules with buffer loads and stores that need dword alignment only)
    if (rp.batch) return (aligned_to(in, 4) && aligned_to(out, 4)) ? launch_corr_rowbatch<T>(in, f, out, s, pad_eff, reverse, rp, st) : -1;
    if (rp.tall) return -1;
    if (s.K < kMfmaMinK || nd < 2 || nd > mfma_max_nd(s.dtype) || s.L > kMfmaMaxL) return -1;
    // whole granules of four elements; otherwise only the kernels that load rows straight into LDS apply (see ragged_rows_ok)
    const bool granular = (s.L % 4) == 0 && aligned_to(in, 4 * sizeof(T)) && aligned_to(out, 4 * sizeof(T));
    // bf16 virtual rows on the kernels that load raw rows straight into LDS: rows of even length (they start on a dword),
    // pitch a multiple of 8; fp32 virtual rows of any length on any fp32 tensor: the kernel that loads rows straight into
    // LDS (up to six offsets)
    const bool rows_direct_bf16 = sizeof(T) == 2 && rp.on && (s.L % 2) == 0 && (rp.map.P % 8) == 0 && aligned_to(in, 4) && aligned_to(out, 4);
    const bool rows_direct_f32 = sizeof(T) == 4 && rp.on && nd <= kMfmaMaxND;
    const bool odd = bf16_odd_rows(s, in, out);
    // (rows of a dozen positions are all gap as virtual rows: B50000 C128 L9 K9 fwd 249 us on the vector-ALU kernel, 323 us
    // here; L25 K7 320 against 309 us)
    if (odd && (nd > kMfmaMaxND || !bf16_odd_rows_ok(s, in, out, rp) || (rp.on && s.L < 24) || bf16_odd_small_call(s, rp))) return -1;
    if (!odd && !granular && !rows_direct_bf16 && !rows_direct_f32 && (!ragged_rows_ok(s, nd) || !aligned_to(in, 4) || !aligned_to(out, 4))) return -1;
    const long long rows = (long long)s.B * s.C;
    const int L_walk = odd ? s.L + 1 : s.L;             // (a shifted row may reach one position further)
    const long long segs_per_row = (L_walk + dwconv::kSegLen - 1) / dwconv::kSegLen;
    const long long total_segs = rows * segs_per_row;
    if (total_segs > 0x3fffffffLL) return -1;           // the kernel's segment walk is 32-bit
    dwconv::CorrGeom g;
    g.C = s.C; g.L = s.L; g.K = s.K; g.rows = (int)rows;
    g.pad = pad_eff; g.reverse = reverse; g.dmin = dmin;
    g.segs_per_row = (int)segs_per_row;
    g.walk_segs = (int)segs_per_row; g.n_main = 0; g.n_light = 0; g.step_c_light = 0;
    g.par0 = odd && !aligned_to(in, 4) ? 1 : 0;
    constexpr int kThreads = 64 * dwconv::kCorrWavesPerBlock;
    const dwconv::RowsMap no_rows{0, 0, 0, 0, 0u, 0u};
    // One resident round of waves, each walking segments wave, wave + n_waves, ...
    // slot_cap: the most wave slots to use.  balance_target > 0 (the kernels that load rows straight into LDS): the
    // number of waves is chosen among whole numbers J of batch entries per round (J * C * segments per row waves, which
    // keeps a wave on one channel) for even loading, the one nearest balance_target among the best: every SIMD gets
    // the same number of waves (a multiple of 1024 waves: with 2560 waves two SIMDs of a compute unit carry three
    // waves and two carry two, and the launch takes as long as the three) and the rounds divide the batch
    // (B32 C256 L4100 K64: 70.3 us with 2560 waves, 65.3 with 3840, 62.4 with 5120; L3000: 43.5 us with 3072).
    // own_light_waves (the kernels that have them): a ragged last segment of at most 512 positions (two live quarters)
    // is left out of this walk and gets waves of its own - about four per compute unit, more for short rows, a whole
    // number of times C where C allows (they then stay on one channel), and out of the resident round, so that all waves
    // of the launch start together.  The others then walk whole segments
    // only, in the order and number of a shape without the ragged end (fwd, B32 C256: L4160 K16 54.9 -> 50.5 us against
    // 48.8 us at L4096; L8196 K16 127 -> 104 us; L4100 K64 62.8 -> 58.4 us).  Where that would take more than a third of
    // the resident waves the light segments stay in the walk.
    auto launch = [&](auto kernel, auto *pi, auto *pf, auto *po, long long slot_cap = kTargetWaves,
                      long long balance_target = 0, bool own_light_waves = false) -> int {
        const long long capacity = balance_target > 0 ? resident_waves(kernel, kThreads) : corr_wave_slots(kernel, kThreads);
        const int last = L_walk % dwconv::kSegLen;
        long long n_light = 0;
        if (own_light_waves && balance_target > 0 && last != 0 && last <= dwconv::kSegLen / 2 && segs_per_row >= 2) {
            // a light segment costs its wave about a microsecond (a memory round trip), a row of the walk about
            // 2 L sizeof(T) / 5 TB/s spread over all waves: enough light waves to be done in 0.6 of the launch
            const long long need = (long long)(5.0e6 / (0.6 * 2.0 * (double)s.L * (double)sizeof(T))) + 1;
            const long long want = need > 1024 ? need : 1024;
            n_light = s.C >= want ? s.C : (long long)s.C * ((want + s.C - 1) / s.C);
            if (n_light > rows) n_light = rows;
            if (3 * n_light > capacity) n_light = 0;
        }
        const long long walk_segs = segs_per_row - (n_light > 0 ? 1 : 0);
        const long long walk_total = rows * walk_segs;
        long long resident = capacity - n_light < slot_cap ? capacity - n_light : slot_cap;
        long long spw = (walk_total + resident - 1) / resident;      // segments per wave, rounded up
        if (spw < 1) spw = 1;
        long long waves = (walk_total + spw - 1) / spw;
        // A whole number of batch entries per round where one fits: the stride of the walk is then a multiple of
        // C rows, a wave stays on one channel and loads its Toeplitz operands once.
        const long long per_b = (long long)s.C * walk_segs;
        if (per_b <= resident) {
            long long J = resident / per_b;
            if (J > s.B) J = s.B;
            if (balance_target > 0) {
                const long long simds = 4LL * kComputeUnits;
                long long best_j = 1;
                double best = -1.0;
                for (long long j = 1; j <= J; ++j) {
                    const long long w = j * per_b, rounds = (s.B + j - 1) / j;
                    const double even_simd = (double)w / (double)(simds * ((w + simds - 1) / simds));
                    const double even_rounds = (double)s.B / (double)(j * rounds);
                    const double near = 1.0 - 0.02 * (double)(w > balance_target ? w - balance_target : balance_target - w) /
                                                  (double)balance_target;
                    const double score = even_simd * even_rounds * near * (w < simds * 2 ? 0.8 : 1.0);
                    if (score > best) { best = score; best_j = j; }
                }
                J = best_j;
            } else {
                const long long rounds = (s.B + J - 1) / J;
                J = (s.B + rounds - 1) / rounds;                       // same number of rounds, evened out
            }
            waves = J * per_b;
        }
        g.walk_segs = (int)walk_segs;
        g.n_main = (int)waves;
        g.n_light = (int)n_light;
        g.step_c_light = (int)(n_light % s.C);
        g.n_waves = (int)(waves + n_light);
        g.step_rows = g.n_main / g.walk_segs;
        g.step_seg = g.n_main % g.walk_segs;
        g.step_c = g.step_rows % s.C;
        const long long blocks = (g.n_waves + dwconv::kCorrWavesPerBlock - 1) / dwconv::kCorrWavesPerBlock;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, pi, pf, po, g, no_rows);
        return launch_status();
    };
    if constexpr (sizeof(T) == 2) {
        if (odd) {
            // bf16 rows that do not all start on a dword, shifted to the dword in which they start (rows_odd_start).
            // Vector-ALU kernel -> here: B32 C256 L4097 K64 fwd 109 -> 30 us (L4096: 22.7), B128 C768 L1025 K32 442 -> 81 us,
            // virtual rows B4096 C128 L199 K48 314 -> 118 us, L47 K48 361 -> 150 us
            const bf16_t *pi = static_cast<const bf16_t *>(in), *pf = static_cast<const bf16_t *>(f);
            bf16_t *po = static_cast<bf16_t *>(out);
            const long long balance = (L_walk % dwconv::kSegLen) != 0 ? kTargetWaves : 0;
            auto go = [&](auto ndc) -> int {
                constexpr int N = decltype(ndc)::value;
                if (rp.on) return launch_corr_vrows_kernel<T>(dwconv::corr_direct_bf16_kernel<N, true, true>, g, rp, in, f, out, s, st);
                return launch(dwconv::corr_direct_bf16_kernel<N, false, true>, pi, pf, po, kTargetWaves, balance, true);
            };
            switch (nd) {
            case 2: return go(std::integral_constant<int, 2>{});
            case 3: return go(std::integral_constant<int, 3>{});
            case 4: return go(std::integral_constant<int, 4>{});
            case 5: return go(std::integral_constant<int, 5>{});
            case 6: return go(std::integral_constant<int, 6>{});
            default: return -1;
            }
        }
    }
    if (!granular && rp.on && !rows_direct_bf16 && !rows_direct_f32) return -1;
    {
        // longer short rows: segments of the virtual row of a channel, slots ordered (virtual segment, channel)
        if (rp.on) {
            auto launch_rows = [&](auto kernel) -> int { return launch_corr_vrows_kernel<T>(kernel, g, rp, in, f, out, s, st); };
            if constexpr (sizeof(T) == 2) {
                // bf16 rows of even length: raw rows straight into LDS, bf16 matrix instruction (B4096 C128 L200
                // K48: 186 -> 104 us against the widening kernel below, which needs whole granules of four)
                if (rows_direct_bf16) {
                    switch (nd) {
                    case 2: return launch_rows(dwconv::corr_direct_bf16_kernel<2, true>);
                    case 3: return launch_rows(dwconv::corr_direct_bf16_kernel<3, true>);
                    case 4: return launch_rows(dwconv::corr_direct_bf16_kernel<4, true>);
                    case 5: return launch_rows(dwconv::corr_direct_bf16_kernel<5, true>);
                    case 6: return launch_rows(dwconv::corr_direct_bf16_kernel<6, true>);
                    default: break;
                    }
                }
            }
            if constexpr (std::is_same<T, float>::value) {
                // fp32 rows that are not whole granules of four, or tensors that are only element-aligned (rows of whole
                // aligned granules: the register-staged kernel below, 1 to 4 % faster there)
                if (!granular) {
                    switch (nd) {
                    case 2: return launch_rows(dwconv::corr_direct_kernel<2, true>);
                    case 3: return launch_rows(dwconv::corr_direct_kernel<3, true>);
                    case 4: return launch_rows(dwconv::corr_direct_kernel<4, true>);
                    case 5: return launch_rows(dwconv::corr_direct_kernel<5, true>);
                    case 6: return launch_rows(dwconv::corr_direct_kernel<6, true>);
                    default: return -1;
                    }
                }
            }
            if (!granular) return -1;             // (the kernels below move whole granules of four)
            switch (nd) {
            case 2: return launch_rows(dwconv::corr_mfma_kernel<T, 2, true>);
            case 3: return launch_rows(dwconv::corr_mfma_kernel<T, 3, true>);
            case 4: return launch_rows(dwconv::corr_mfma_kernel<T, 4, true>);
            case 5: return launch_rows(dwconv::corr_mfma_kernel<T, 5, true>);
            case 6: return launch_rows(dwconv::corr_mfma_kernel<T, 6, true>);
            default: break;
            }
            if constexpr (std::is_same<T, float>::value) return launch_corr_vrows_wide_f32(g, rp, nd, in, f, out, s, st);
            return -1;
        }
    }
    if constexpr (sizeof(T) == 2) {
        // bf16 storage: the bf16 matrix instruction when 16-byte granules of 8 elements line up
        const bool whole8 = (s.L % 8) == 0 && aligned_to(in, 16) && aligned_to(out, 16);
        if (whole8 || (nd <= kMfmaMaxND && (s.L % 2) == 0 && aligned_to(in, 4) && aligned_to(out, 4))) {
            const bf16_t *pi = static_cast<const bf16_t *>(in), *pf = static_cast<const bf16_t *>(f);
            bf16_t *po = static_cast<bf16_t *>(out);
            {
                // two to six block offsets: rows straight into LDS, refilled in place (B128 C768 L1024 K32: 72 us
                // against 76 us through staging registers; a wave has half the bytes of an fp32 one in flight, and a
                // full round of sixteen waves per compute unit is the fastest here)
                const bool ragged_last = (s.L % dwconv::kSegLen) != 0;      // (then: balanced wave count, own waves for light segments)
                switch (nd) {
                case 2: return launch(dwconv::corr_direct_bf16_kernel<2>, pi, pf, po, kTargetWaves, ragged_last ? kTargetWaves : 0, true);
                case 3: return launch(dwconv::corr_direct_bf16_kernel<3>, pi, pf, po, kTargetWaves, ragged_last ? kTargetWaves : 0, true);
                case 4: return launch(dwconv::corr_direct_bf16_kernel<4>, pi, pf, po, kTargetWaves, ragged_last ? kTargetWaves : 0, true);
                case 5: return launch(dwconv::corr_direct_bf16_kernel<5>, pi, pf, po, kTargetWaves, ragged_last ? kTargetWaves : 0, true);
                case 6: return launch(dwconv::corr_direct_bf16_kernel<6>, pi, pf, po, kTargetWaves, ragged_last ? kTargetWaves : 0, true);
                // (seven to nine offsets would still fit the window's tail load; measured no faster than the register-staged
                // kernel below: B128 C768 L1024 K128 81.6 against 80.3 us)
                default: break;
                }
            }
            if (!whole8) return -1;
            switch (nd) {
            case 7: return launch(dwconv::corr_mfma_bf16_kernel<7>, pi, pf, po);
            case 8: return launch(dwconv::corr_mfma_bf16_kernel<8>, pi, pf, po);
            case 9: return launch(dwconv::corr_mfma_bf16_kernel<9>, pi, pf, po);
            case 10: return launch(dwconv::corr_mfma_bf16_kernel<10>, pi, pf, po);
            default: return -1;
            }
        }
    }
    const T *pi = static_cast<const T *>(in), *pf = static_cast<const T *>(f);
    T *po = static_cast<T *>(out);
    if constexpr (std::is_same<T, float>::value) {
        // fp32, two to six block offsets: rows straight into LDS, refilled in place.  Wave slots aimed at: fewer than a
        // full resident round, because a launch is the time its bytes take plus a fill and a drain that grow with the
        // bytes in flight (B32 C256 L4096: K = 7 93 us with 8 waves per compute unit, 96 us with 12 or 16; K = 64 51.4 /
        // 50.8 / 50.9 us with 8 / 12 / 16, the matrix pipe wanting more than two waves per SIMD there); up to 20 per
        // compute unit where that is what loads the SIMDs evenly (see `launch`)
        const long long target = (long long)kComputeUnits * (nd <= 3 ? 8 : 14), cap = (long long)kComputeUnits * (nd <= 3 ? 12 : 20);
        switch (nd) {
        case 2: return launch(dwconv::corr_direct_kernel<2>, pi, pf, po, cap, target, true);
        case 3: return launch(dwconv::corr_direct_kernel<3>, pi, pf, po, cap, target, true);
        case 4: return launch(dwconv::corr_direct_kernel<4>, pi, pf, po, cap, target, true);
        case 5: return launch(dwconv::corr_direct_kernel<5>, pi, pf, po, cap, target, true);
        case 6: return launch(dwconv::corr_direct_kernel<6>, pi, pf, po, cap, target, true);
        default: break;
        }
    }
    // (fp32 rows that are not whole granules: the register-staged kernel below takes them too, see ragged_rows_ok)
    if (!granular && !std::is_same<T, float>::value) return -1;
    if constexpr (!std::is_same<T, float>::value) {
        // (bf16 rows of odd length in whole granules of four: widened to fp32 on the way into LDS)
        switch (nd) {
        case 2: return launch(dwconv::corr_mfma_kernel<T, 2, false>, pi, pf, po);
        case 3: return launch(dwconv::corr_mfma_kernel<T, 3, false>, pi, pf, po);
        case 4: return launch(dwconv::corr_mfma_kernel<T, 4, false>, pi, pf, po);
        case 5: return launch(dwconv::corr_mfma_kernel<T, 5, false>, pi, pf, po);
        case 6: return launch(dwconv::corr_mfma_kernel<T, 6, false>, pi, pf, po);
        default: break;
        }
    }
    if constexpr (std::is_same<T, float>::value) {
        if ((s.L % 4) != 0) {
            switch (nd) {
            case 7: return launch(dwconv::corr_mfma_kernel<float, 7, false, true>, pi, pf, po);
            case 8: return launch(dwconv::corr_mfma_kernel<float, 8, false, true>, pi, pf, po);
            case 9: return launch(dwconv::corr_mfma_kernel<float, 9, false, true>, pi, pf, po);
            case 10: return launch(dwconv::corr_mfma_kernel<float, 10, false, true>, pi, pf, po);
            case 11: return launch(dwconv::corr_mfma_kernel<float, 11, false, true>, pi, pf, po);
            case 12: return launch(dwconv::corr_mfma_kernel<float, 12, false, true>, pi, pf, po);
            case 13: return launch(dwconv::corr_mfma_kernel<float, 13, false, true>, pi, pf, po);
            case 14: return launch(dwconv::corr_mfma_kernel<float, 14, false, true>, pi, pf, po);
            default: return -1;
            }
        }
        switch (nd) {
        case 7: return launch(dwconv::corr_mfma_kernel<float, 7, false>, pi, pf, po);
        case 8: return launch(dwconv::corr_mfma_kernel<float, 8, false>, pi, pf, po);
        case 9: return launch(dwconv::corr_mfma_kernel<float, 9, false>, pi, pf, po);
        case 10: return launch(dwconv::corr_mfma_kernel<float, 10, false>, pi, pf, po);
        case 11: return launch(dwconv::corr_mfma_kernel<float, 11, false>, pi, pf, po);
        case 12: return launch(dwconv::corr_mfma_kernel<float, 12, false>, pi, pf, po);
        default: break;
        }
    }
    return -1;
}

// Which filters of more than six block offsets go to corr_band_kernel (us, kernels it replaces there -> corr_band_kernel).  Small
// calls keep the register-resident kernels further up: a wave each for their segments, against workgroups that stage taps and
// window and add up four waves' parts.
//   fp32, ordinary rows of whole granules: from thirteen offsets (B32 C256 L4096: K = 160 87 / 107, 200 111 -> 89, 300 180 ->
//     133, 1024 496 -> 296, 4096 1050 -> 712), from eleven where rows fill less than three quarters of their 1024-position segments
//   fp32, other lengths: from nine (B32 C256 L4097: K = 128 156 -> 88, 200 223 -> 108, 4097 3537 -> 954; B64 C64 L1501, 8192 segments in
//     all: K = 160 38 -> 23), nine and ten from 10240 segments on (B2107 C1 L3979 K128, 8428: 26 / 30), eleven to fourteen from 4096 on
//     (B160 C5 L4809 K200, 4000: 18.9 / 21.9; B13 C257 L999 K160, 3341: 15.5 / 20.5) or where rows fill less than three quarters of
//     their segments (B1 C33 L1221 K192 7.6 -> 5.1)
//   bf16, rows of whole 16-byte granules: from eleven (B32 C256 L4096: K = 128 35 / 37, 226 50 -> 41, 4096 243 -> 148), from
//     seven where rows fill less than three quarters of their segments and there are more than 1024 (L512 K512 92 -> 48); other
//     lengths and alignments: all (L4097: K = 100 119 -> 65, 4097 3213 -> 200)
//   short rows with more than six offsets: fp32 virtual rows of up to 512 positions with more than 4096 segments up to eight offsets
//     (B1000 C128 L160 K84 50 -> 44; B20 C256 L400, 2304: 9.6 / 10.5), 1024 up to twelve (B64 C256 L512 K100 25 -> 22; B41 C47 L240
//     K130, 564: 6.4 / 9.3), all beyond; rows of up to 512 positions with filters of their own length (L256 K256 fp32 101 -> 76, bf16
//     105 -> 38), any alignment; rows of at most 128 positions: bf16 above 64 (L128 K128 61 -> 35; fp32 L96 K96 48 / 59).  Virtual rows of
//     more than 512 positions (fp32) keep the register-resident kernel up to twelve offsets: their blocks do not fill the tiles
//     of an item (B200 C32 L700 K80 15.4 / 18.6)
inline bool corr_takes_band(const Shape &s, int pad_eff, const void *in, const void *out)
{
    const int nd = toeplitz_dmax(s.K, pad_eff) - toeplitz_dmin(pad_eff) + 1;
    const RowsPlan rp = plan_rows(s);
    if (rp.tall) return true;
    if (nd <= kMfmaMaxND) return false;
    if (rp.batch) {
        int bd, bn;
        rows_batch_offsets(s.L, s.K, pad_eff, &bd, &bn);
        return s.dtype == DWCONV_BF16 && bn > kMfmaMaxND && s.L > 64;
    }
    const bool granules = aligned_to(in, 16) && aligned_to(out, 16);
    if (rp.on) return nd > 12 || !granules || (s.L <= 512 && (long long)rp.nvs * s.C > (nd <= 8 ? 4096 : 1024));
    if (s.L <= 512) return true;
    const long long segs_per_row = ((long long)s.L + dwconv::kSegLen - 1) / dwconv::kSegLen, segs = (long long)s.B * s.C * segs_per_row;
    const bool filled = 4ll * s.L >= 3 * segs_per_row * dwconv::kSegLen;
    if (s.dtype == DWCONV_F32 && (s.L % 4) != 0) return nd >= (segs > 10240 ? 9 : segs >= 4096 || !filled ? 11 : 15);
    if (s.dtype == DWCONV_F32) return nd >= (filled ? 13 : 11);
    return (s.L % 8) != 0 || !granules || nd >= (filled || segs <= 1024 ? 11 : 7);
}

// Which fp32 filters of seven and more block offsets that plan_corr_window takes go to corr_window_kernel (us per 2^20 positions unless said
// otherwise, inputs from memory, the kernel before / here; over 1000 calls, forward and input gradient).
//   in the place of corr_mfma_kernel: nine offsets and more always (mean gain 1.2; B11 C623 L3040 K138 58 / 71 us).  Seven and eight where an estimate of that
//     kernel - its products with the padding of rows to whole segments of 1024 positions, or of virtual rows to their pitch, 1.15 or 1.25 times as long as
//     at the clock under load; at least 2.2, its memory - is above one of this: 1.2 of the plan's, at least 2.6 for rows that are not whole cache lines,
//     whose pieces cost memory time, or 1.8.  Taken B61 C576 L1163 K94 4.3 / 2.7, B109 C256 L1082 K80 3.6 / 2.6, B974 C64 L1216 K80 2.2 / 1.9; left B244 C96
//     L2988 K88 2.1 / 2.6, B139 C544 L896 K75 2.3 / 2.7, B86 C128 L5680 K80 2.1 / 2.4, B500 C128 L516 K72 70 / 88 us.  (Eight offsets at 1.18: B9 C620
//     L4615 K107 4.4 / 3.2, B234 C64 L1184 K107 3.3 / 2.5, B42 C477 L1488 K98 2.9 / 2.4 stayed away)
//   in the place of corr_band_kernel: not rows of at most three steps of 64 positions off half cache lines where inputs and outputs are more than
//     the 256 MiB of the last-level cache and both wait for memory (B3967 C96 L186 K99 2.3 / 2.5, B702 C453 L186 K85 2.3 / 2.5; half lines B3244 C96 L144
//     K144 2.5 / 2.3; 16 calls of such a size 2.67 / 2.74 in the mean, 11 smaller ones 3.08 / 3.00, B374 C160 L180 K75 34 / 31 us), and not
//     calls that leave some SIMDs with two waves and most with one (405 workgroups of four waves): where, with the SIMD that has most waves in the place of
//     the mean one, less than 0.46 of the plan's estimate, or 0.57 in pieces of at most four steps, whose starts weigh more, is work that a full chip could not do
//     without.  Of 567 calls the 35 below that gain nothing (mean 0.995; us, B26 C538 L2665 K233 147 / 175, B549 C59 L561 K247 70 / 80, B277 C128
//     L498 K143 55 / 61, B94 C651 L208 K181 38 / 44), the others 1.14 in the mean, 15 of them less than 0.97 (B1184 C384 L176 K124 179 / 202).
//     (Rows in one piece with as many steps in front that only bring chunks as steps, the input gradient of causal filters as long as the row: in a training
//     step of B2048 C128 L256 K256 it takes 148 / 151 us, but forward and weight gradient 143 / 138 and 151 / 149 beside it, the step 443 / 439)
// (Up to six offsets memory bounds the fp32 instruction's kernels already: virtual rows of whole cache lines with five and six offsets are 1.1 to
// 1.25 times as fast here alone, but a step of separate calls is not: B1024 C64 L224 K56 87 / 93 us, B2048 C128 L384 K64 544 / 529.)
inline bool corr_takes_window(const Shape &s, int pad_eff, const WindowPlan &p, bool band)
{
    const int nd = toeplitz_dmax(s.K, pad_eff) - toeplitz_dmin(pad_eff) + 1;
    const RowsPlan rp = plan_rows(s);
    const double rows = (double)s.B * s.C, millions = rows * s.L / (1024.0 * 1024.0);
    // (tensors off a 16-byte granule send virtual rows to corr_band_kernel: seven offsets stay there where the estimates below would leave them)
    if (band)
        return (s.L > 192 || (s.L % 16) == 0 || millions < 32.0) && p.share >= (p.g.ns <= 4 ? 0.57 : 0.46) && !(nd == kMfmaMaxND + 1 && rp.on && s.L > 512 && (s.L % 32) != 0);
    if (nd > 8) return true;
    const double padded = rows * (rp.on ? rp.map.P : (s.L + dwconv::kSegLen - 1) / dwconv::kSegLen * dwconv::kSegLen);
    const double there = std::max((nd == 8 ? 1.25 : 1.15) * padded / 1024.0 * 16 * nd * 32 / (4 * kComputeUnits) / 2100.0, 2.2 * millions);
    const double here = std::max(1.2 * p.cycles / 2000.0, (s.L % 32) == 0 ? 1.8 * millions : 2.6 * millions);
    return here < there;
}

template <typename T>
int launch_corr(const void *in, const void *f, void *out, const Shape &s, int pad_eff, int reverse, hipStream_t st)
{
    int rc = -1;
    const bool band = corr_takes_band(s, pad_eff, in, out);
    if constexpr (std::is_same<T, float>::value) {
        WindowPlan p;
        if (toeplitz_dmax(s.K, pad_eff) - toeplitz_dmin(pad_eff) >= kMfmaMaxND && plan_corr_window(s, pad_eff, reverse, &p) &&
            corr_takes_window(s, pad_eff, p, band))
            return launch_corr_window_f32(in, f, out, s, p, st);
    }
    if (band) {
        if constexpr (std::is_same<T, float>::value) rc = launch_corr_band_f32(in, f, out, s, pad_eff, reverse, st);
        else rc = launch_corr_band_bf16(in, f, out, s, pad_eff, reverse, st);
        if (rc >= 0) return rc;
    }
    rc = launch_corr_mfma<T>(in, f, out, s, pad_eff, reverse, st);
    if (rc >= 0) return rc;
    return launch_corr_valu<T>(in, f, out, s, pad_eff, reverse, st);
}

}  // namespace dwhost
