// Stage 1 of the weight gradient (Sec. IV-A eq. (dk_def)) of fp32 filters of at most five 32-blocks (about 65 to 130 taps) on
// v_mfma_f32_32x32x16_bf16 with three exact bf16 limbs per operand (split_pair, limb_sum), the operands in registers:
//
//   G_d[q'][q] += X[m + d][q'] dY[m][q]      (32-blocks m, block offsets d),      dw[j] = sum over 32 d + q' - q + pad = j
//
// The sixteen entries of a contraction are sixteen columns of a channel; a column is a piece of P positions of one row.  An operand is eight
// values of a lane, a position's in eight columns, so nothing is transposed: rows go straight to a ring in LDS, four pairs of blocks deep, and
// a lane reads its eight dwords.  A wave walks the pieces of its columns block by block, holds the x blocks that its ND offsets reach as limbs,
// and splits every value once.  No wave waits for another until the sums at the end.
//
// One wave per SIMD: 48 ND accumulator registers for the scales of all offsets, 72 for x and 24 for dY.  What hides the splitting is then the wave
// itself: a step's 6 ND products are issued with the 136 vector instructions that split the next step's blocks between them (a product of
// 32 cycles leaves half of them to vector instructions), with one branch per step.  Tried: two waves per SIMD with three offsets each, both
// splitting everything (B32 C256 L4096 K128 100 us, here 77-85, inputs from memory), or eight offsets on two groups of waves (B2048 C128 L256 K256
// 224 us, dw_band_kernel 167: short rows are all starts of columns).
// What bounds it: B32 C256 L4096 K128 77 us with inputs from memory (dw_partial_direct_kernel, on the fp32 instruction, 96) and 74 in a training step, behind
// a kernel that leaves dY in the last-level cache (80 there); 52 without its loads and 57 without its products.  Relative error against 64 bits
// 2.0e-7, the fp32 instruction 4.2e-7 (of 140 calls half in the mean).
#pragma once
#include "dwconv_dw_band.hip.h"
#include "dwconv_dw_direct.hip.h"

namespace dwconv {

constexpr int kDwWinWaves = 4;
constexpr int kDwWinThreads = 64 * kDwWinWaves;
constexpr int kDwWinCols = 16;               // columns of a unit: the entries of a contraction
constexpr int kDwWinND = 5;                  // offsets at most
constexpr int kDwWinSlots = 6;               // x blocks in registers: those of a step and the next one
constexpr int kDwWinTensor = 4096 + 128;     // bytes of a pair of blocks of one tensor in the ring
constexpr int kDwWinPairs = 4;               // pairs of blocks of both tensors in the ring of a wave
constexpr int kDwWinRing = 2 * kDwWinPairs * kDwWinTensor;
inline int dw_win_lds_bytes()
{
    const int ring = kDwWinWaves * kDwWinRing, ep = (int)sizeof(float) * kDwWinWaves * (kDwBandDiag + 64 * kDwWinND);
    return ring > ep ? ring : ep;
}

struct DwWinGeom {
    int B, C, L, K, pad;
    int dmin, nd;       // block offsets (of 32) that hold a tap and have a block pair inside a row
    int NP, P;          // pieces of a row, positions of one (a multiple of 64)
    unsigned np_magic;  // floor(2^32 / NP) + 1 for NP > 1
    int units;          // groups of sixteen columns of a channel
    int rem;            // block of the last position of a row within its piece, modulo blocks of a piece
};

template <int ND>
__global__ __launch_bounds__(kDwWinThreads, 1) void dw_window_kernel(const float *__restrict__ x, const float *__restrict__ dy,
                                                                     float *__restrict__ part, float *__restrict__ dw_out, const DwWinGeom g,
                                                                     int slices)
{
    constexpr int NL = 3;
    extern __shared__ __align__(16) unsigned char dww_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x, sl = (int)blockIdx.y;
    const int CL = g.C * g.L;
    const int d0 = g.dmin;
    const int PB = g.P >> 5, NB = (g.L + 31) >> 5;
    // the last x block of a row, dY blocks of a piece; steps of a unit: pairs of them, those below 0 only bring x
    const int chi = g.NP > 1 ? 1 << 28 : NB - 1;
    const int nb = g.NP > 1 ? PB : NB;
    const int s_first = (g.NP > 1 ? -(ND - 1) : max(-(ND - 1), -d0 - (ND - 1))) & ~1, s_end = (min(nb, chi - d0 + 1) + 1) & ~1;

    floatx16 acc[ND], mid[ND], low[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[i][k] = mid[i][k] = low[i][k] = 0.f;

    const int stride = kDwWinWaves * (int)gridDim.y;
    int unit = wave + kDwWinWaves * sl;
    if (unit < g.units) {
        unsigned char *ring_p = dww_smem + wave * kDwWinRing;
        const unsigned ring = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) const void *)ring_p);
        // the load cursor.  Load q of a pair of blocks: lane i brings granule i % 16 of row 4 q + i / 16; ld_t its position in dY, ld_off its
        // byte offset from the unit's first row at step s_first, in x from dx positions further (rows past the batch: out of every range)
        const int dx = 32 * (d0 + ND - 1);                               // from a block of dY to the newest of x
        const int t_last = (g.NP - 1) * g.P + 64;                        // the end of a pair of step 0 in the last piece
        int ld_unit = unit, ld_s = s_first, ld_t[4], ld_off[4], slot = 0;
        uintx4 rx_desc, ry_desc;
        auto ld_place = [&]() {
            const int first = ld_unit * kDwWinCols;
            const int b0 = g.NP > 1 ? (int)__umulhi((unsigned)first, g.np_magic) : first;
            const size_t off = ((size_t)b0 * (size_t)g.C + (size_t)c) * (size_t)g.L;
            const size_t left = 4 * ((size_t)g.B * (size_t)CL - off);
            const unsigned bytes = (unsigned)(left < 0x3ff00000 ? left : 0x3ff00000);
            const unsigned long long ax = reinterpret_cast<unsigned long long>(x + off) + (unsigned long long)(4ll * (dx + 32 * s_first)),
                                     ay = reinterpret_cast<unsigned long long>(dy + off) + (unsigned long long)(128ll * s_first);
            rx_desc = uintx4{(unsigned)ax, (unsigned)(ax >> 32) & 0xffffu, bytes - (unsigned)(4 * (dx + 32 * s_first)), kBufferFlags};
            ry_desc = uintx4{(unsigned)ay, (unsigned)(ay >> 32) & 0xffffu, bytes - (unsigned)(128 * s_first), kBufferFlags};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int mine = first + 4 * q + (lane >> 4);
                const int b = g.NP > 1 ? (int)__umulhi((unsigned)mine, g.np_magic) : mine;
                const int t0 = (mine - b * g.NP) * g.P + 4 * (lane & 15);
                ld_t[q] = t0 + 32 * s_first;
                ld_off[q] = b < g.B ? 4 * ((b - b0) * CL + t0) : kOutOfRow;
            }
        };
        auto load = [&]() {
            const bool has_y = ld_s >= 0 && ld_s < nb;
            const int tx = 32 * ld_s + dx;
            if (has_y && tx >= 0 && t_last + max(tx, 32 * ld_s) <= g.L) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned to = ring + (unsigned)slot + 1024u * q + (q >= 2 ? 128u : 0u);
                    buffer_load_x4_to_lds_keep(rx_desc, ld_off[q], to);
                    buffer_load_x4_to_lds_keep(ry_desc, ld_off[q], to + kDwWinTensor);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned to = ring + (unsigned)slot + 1024u * q + (q >= 2 ? 128u : 0u);
                    buffer_load_x4_to_lds_keep(rx_desc, ld_unit < g.units && (unsigned)(ld_t[q] + dx) < (unsigned)g.L ? ld_off[q] : kOutOfRow, to);
                    buffer_load_x4_to_lds_keep(ry_desc, ld_unit < g.units && has_y && (unsigned)ld_t[q] < (unsigned)g.L ? ld_off[q] : kOutOfRow, to + kDwWinTensor);
                }
            }
            slot = slot + 2 * kDwWinTensor == kDwWinRing ? 0 : slot + 2 * kDwWinTensor;
        };
        auto ld_next = [&]() {
            ld_s += 2;
            if (ld_s >= s_end) {
                ld_unit += stride;
                ld_s = s_first;
                if (ld_unit < g.units) {
                    ld_place();
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) ld_off[q] = kOutOfRow;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ld_t[q] += 64;
                    ld_off[q] += 256;
                }
            }
        };
        const int pos = lane & 31, kg = lane >> 5;
        const unsigned char *raw_p = ring_p + kg * (2048 + 128) + 4 * pos;
        const bool ragged = (g.L & 3) != 0;
        // the read cursor: raw values of a block of either tensor, lane (position, half kg) those of rows 8 kg .. 8 kg + 7
        int rd_slot = 0, rd_s = s_first, rd_unit = unit;
        float rx[8], ry[8];
        auto read_pair = [&](float (&r)[8], int at, int i) {
#pragma unroll
            for (int v = 2 * i; v < 2 * i + 2; ++v) r[v] = *reinterpret_cast<const float *>(raw_p + at + (v >> 2) * 1024 + (v & 3) * 256);
        };
        // (positions behind the end of a row in the granule in which it ends: those of the next row)
        auto trim = [&](float (&r)[8], int u, int blk) {
            if (ragged && (blk == g.rem || blk == g.rem - PB || blk == g.rem + PB)) {
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const int mine = u * kDwWinCols + 8 * kg + v;
                    const int b = g.NP > 1 ? (int)__umulhi((unsigned)mine, g.np_magic) : mine;
                    r[v] = (mine - b * g.NP) * g.P + 32 * blk + pos < g.L ? r[v] : 0.f;
                }
            }
        };
        uintx4 X[kDwWinSlots][NL], Y[2][NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
#pragma unroll
            for (int i = 0; i < kDwWinSlots; ++i) X[i][l] = uintx4{0u, 0u, 0u, 0u};
            Y[0][l] = Y[1][l] = uintx4{0u, 0u, 0u, 0u};
        }
        auto split_into = [&](uintx4 (&to)[NL], const float (&r)[8], int i) {
            unsigned p[3];
            split_pair(r[2 * i], r[2 * i + 1], p);
            to[0][i] = p[0]; to[1][i] = p[1]; to[2][i] = p[2];
        };
        ld_place();
#pragma unroll
        for (int i = 0; i < kDwWinPairs; ++i) {
            if (i > 0) ld_next();
            load();
        }
        // what step s multiplies is split before it, and read before that
        wait_vmcnt_at_most<8 * (kDwWinPairs - 1)>();
        auto rd_at = [&](int half) { return rd_slot + 128 * half; };
#pragma unroll
        for (int i = 0; i < 4; ++i) { read_pair(rx, rd_at(0), i); read_pair(ry, rd_at(0) + kDwWinTensor, i); }
        trim(rx, rd_unit, rd_s + d0 + ND - 1);
        trim(ry, rd_unit, rd_s);
#pragma unroll
        for (int i = 0; i < 4; ++i) { split_into(X[0], rx, i); split_into(Y[0], ry, i); }
#pragma unroll
        for (int i = 0; i < 4; ++i) { read_pair(rx, rd_at(1), i); read_pair(ry, rd_at(1) + kDwWinTensor, i); }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        int s = s_first;
        bool done = false;
        auto rd_next = [&]() {
            if (++rd_s == s_end) {
                rd_unit += stride;
                rd_s = s_first;
            }
        };
        rd_next();
        // Step s (slot PH of x): multiplies its blocks, splits the raw values of the next step and reads those of the one after
        auto step = [&](auto phc) {
            constexpr int PH = decltype(phc)::value, HALF = PH & 1, NXT = (PH + 1) % kDwWinSlots;
            // (raw values: of step rd_s; read in this step: the first block of the next pair in even steps, the second in odd ones)
            if constexpr (HALF == 0) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (the pair whose place is taken has been read)
                ld_next();
                load();
                rd_slot = rd_slot + 2 * kDwWinTensor == kDwWinRing ? 0 : rd_slot + 2 * kDwWinTensor;
                wait_vmcnt_at_most<8 * (kDwWinPairs - 1)>();             // (the pairs after it are the last that were asked for)
            }
            trim(rx, rd_unit, rd_s + d0 + ND - 1);
            trim(ry, rd_unit, rd_s);
            const int at = rd_at(HALF);
            const bool has_y = s >= 0 && s < nb;
            auto chunk = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if constexpr (k < 4) {
                    split_into(X[NXT], rx, k);
                    read_pair(rx, at, k);
                } else {
                    split_into(Y[1 - HALF], ry, k - 4);
                    read_pair(ry, at + kDwWinTensor, k - 4);
                }
            };
            if (has_y) {
                const uintx4 (&y)[NL] = Y[HALF];
                static_for<0, ND>([&](auto ic) {
                    constexpr int I = decltype(ic)::value;
                    const uintx4 (&a)[NL] = X[(PH + kDwWinSlots + I - (ND - 1)) % kDwWinSlots];
                    low[I] = mfma32x32x16(a[2], y[0], low[I]);
                    acc[I] = mfma32x32x16(a[0], y[0], acc[I]);
                    mid[I] = mfma32x32x16(a[1], y[0], mid[I]);
                    low[I] = mfma32x32x16(a[0], y[2], low[I]);
                    mid[I] = mfma32x32x16(a[0], y[1], mid[I]);
                    low[I] = mfma32x32x16(a[1], y[1], low[I]);
                });
                static_for<0, 8>(chunk);
                // a vector instruction or six behind each product
#pragma unroll
                for (int k = 0; k < 6 * ND; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, (8 * 17 + 6 * ND - 1) / (6 * ND), 0);
                    if (k % 3 == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            } else {
                static_for<0, 8>(chunk);
            }
            rd_next();
            if (++s == s_end) {
                unit += stride;
                s = s_first;
                done = unit >= g.units;
                if (g.NP == 1) {
                    // (blocks in front of the row, of which the next step brings the first that is not)
#pragma unroll
                    for (int i = 0; i < kDwWinSlots; ++i)
                        if (i != NXT)
#pragma unroll
                            for (int l = 0; l < NL; ++l) X[i][l] = uintx4{0u, 0u, 0u, 0u};
                }
            }
        };
        auto walk = [&](auto self, auto phc) -> void {
            constexpr int PH = decltype(phc)::value;
            if constexpr (PH < kDwWinSlots) {
                step(phc);
                if (!done) self(self, std::integral_constant<int, PH + 1>{});
            }
        };
        while (!done) walk(walk, std::integral_constant<int, 0>{});
        wait_vmcnt_at_most<0>();                                         // (no load may write LDS that the sums below take)
    }

    // ---- diagonal sums: every wave those of its offsets (e = q' - q + 31 of each), then the two offsets a tap belongs to and the
    // waves' parts of each added in order
    __syncthreads();
    float *img = reinterpret_cast<float *>(dww_smem) + wave * kDwBandDiag;
    float *taps = reinterpret_cast<float *>(dww_smem) + kDwWinWaves * kDwBandDiag;
    constexpr int TW = 64 * ND;
    float *tap = taps + wave * TW;
    for (int i = lane; i < kDwBandDiag / 4; i += 64) *reinterpret_cast<floatx4 *>(img + 4 * i) = floatx4{0.f, 0.f, 0.f, 0.f};
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < ND; ++i) {
        // lane (column q, half kg) holds rows q' = 8 (k / 4) + 4 kg + k % 4 in element k
        const int q = lane & 31, kg = lane >> 5;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            img[(8 * (k >> 2) + 4 * kg + (k & 3) - q + 31) * kDwBandDiagPitch + q] = limb_sum(acc[i][k], mid[i][k], low[i][k]);
        wave_lds_fence();
        if (lane < 63) {
            floatx4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const floatx4 *>(img + lane * kDwBandDiagPitch + 4 * j);
            floatx4 sum = v[0];
#pragma unroll
            for (int j = 1; j < 8; ++j) sum += v[j];
            tap[64 * i + lane] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        }
        wave_lds_fence();
    }
    __syncthreads();
    // tap T = 0 .. 32 nd + 30 is j = 32 dmin - 31 + pad + T (taps no offset reaches are zero)
    const int j0 = 32 * g.dmin - 31 + g.pad;
    float *dst = part + ((size_t)sl * (size_t)g.C + (size_t)c) * (size_t)g.K;
    for (int j = tid; j < g.K; j += kDwWinThreads) {
        const int t = j - j0;
        float sum = 0.f;
        if (t >= 0 && t < 32 * g.nd + 31) {
            // diagonal t % 32 of offset t / 32 and t % 32 + 32 of the one before it
#pragma unroll
            for (int h = 1; h >= 0; --h) {
                const int o = (t >> 5) - h, e = (t & 31) + 32 * h;
                if (o >= 0 && o < g.nd && e < 63) {
#pragma unroll
                    for (int k = 0; k < kDwWinWaves; ++k) sum += taps[k * TW + 64 * o + e];
                }
            }
        }
        if (dw_out) {
            dw_out[(size_t)c * (size_t)g.K + (size_t)j] = sum;
        } else {
            dst[j] = sum;
            // (slices beyond those of this launch are part of the workspace's layout: zeros)
            for (int o = sl + (int)gridDim.y; o < slices; o += (int)gridDim.y)
                part[((size_t)o * (size_t)g.C + (size_t)c) * (size_t)g.K + (size_t)j] = 0.f;
        }
    }
}

}  // namespace dwconv
