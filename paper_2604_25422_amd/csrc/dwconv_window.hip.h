// Forward / input gradient of fp32 filters of about 65 to 260 taps on rows from 129 positions: the blocked-Toeplitz contraction on
// v_mfma_f32_16x16x32_bf16 with three exact bf16 limbs per operand (split_pair), the inputs in registers.
//
//   Y[16 m + r][col] = sum_ci sum_k A_q[r][k] X[32 ci - phi + k][col],   q = 2 ci - m,   A_q[r][k] = w[16 q + k - r - phi + pad]
//
// A column is a piece of P positions of one row, a unit sixteen columns of a channel (neighbouring pieces, then batch entries).  A wave walks
// the pieces of its unit from front to back, 64 positions (four tiles of 16) a step, and keeps the limbs of the chunks of 32 positions
// that a step reaches in registers: every input is loaded, split and read once, and no wave waits for another.  The taps of the channel lie in
// LDS, shared by the waves of a workgroup, in eight copies (one for each alignment of a lane's eight taps), so that an operand is
// three aligned reads; it serves two products of six, (m, ci) and (m + 2, ci + 1).  Chunk ci has slot ci modulo WR, so the steps are unrolled PER deep.
//
// Chunk pairs come through a ring in LDS, two steps ahead (loads that write LDS directly: whole lines of the sixteen rows, granules permuted so
// that the reads of a column are free of bank conflicts); the tiles of a step leave through the ring's free slot, 256 bytes of a row at a time
// (straight from the tiles they were pieces of 64 bytes: B114 C192 L3776 K110 201 -> 162 us, B32 C256 L4097 K128 80 -> 76).
//
// What bounds it: vector instructions (limbs, sums) and these products of 16 cycles take turns on a SIMD (a product of 32 x 32 x 16 hides vector
// instructions for half of its 32 cycles, this one for none), together 40 us of the 69 us of B32 C256 L4096 K128 (inputs from memory, mean of four
// cards), whose memory takes 52 (pieces of rows cost some: a walk of whole segments takes 50); corr_mfma_kernel on the fp32 instruction takes 81. B2048
// C128 L256 K256 causal: forward 140 us, input gradient, which brings four steps of chunks in front of every row, 148 (corr_band_kernel 152 and
// 150; in a training step 138 and 151, corr_band_kernel 150 and 148, the step 439 and 449), memory 103.  Three waves per SIMD in place of two (168
// registers): no faster, and 90 us where they spill.  Relative error against 64 bits (2-norm, normal data): 5-9e-8, as corr_band_kernel; the fp32 instruction 1.5-2.1e-7.
#pragma once
#include "dwconv_band.hip.h"

namespace dwconv {

__device__ __forceinline__ floatx4 mfma16x16x32(uintx4 a, uintx4 b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kWinWaves = 4;                 // of a workgroup, at most
constexpr int kWinThreads = 64 * kWinWaves;
constexpr int kWinCols = 16;                 // columns of a unit

// bytes of one copy of the staged taps: 64 more than a multiple of 256 (sixteen lanes of a read then take sixteen banks of 16 bytes)
__host__ __device__ constexpr int win_tap_pitch(int NW) { return ((16 * (4 * NW + 6) - 64 + 255) / 256) * 256 + 64; }
constexpr int kWinRing = 2;                  // chunk pairs of a wave on their way, 4096 bytes each
__host__ __device__ constexpr int win_lds_bytes(int NL, int NW, int waves) { return NL * 8 * win_tap_pitch(NW) + waves * kWinRing * 4096; }

struct WindowGeom {
    int B, C, L, K;
    int pad;            // effective pad of this correlation
    int reverse;        // filter index reversed (input gradient)
    int phi;            // chunk ci holds the positions 32 ci - phi .. + 31 of a piece
    int q0;             // first q, odd
    int qn;             // q0 .. q0 + qn - 1 hold taps
    int NP, P;          // pieces of a row, positions of one (a multiple of 64)
    unsigned np_magic;  // floor(2^32 / NP) + 1 for NP > 1
    int units;          // groups of sixteen columns of a channel
    int s_first, ns;    // steps of a unit: those below 0 only bring chunks
    int clo, chi;       // chunks that meet a row
    int waves;          // of a workgroup
    int lines;          // outputs are whole cache lines
};

constexpr int kWinPerSimd = 2;               // waves

// NW: chunks that a tile reads.  WR: chunks in registers, the NW + 1 of a step or, on rows that have no more, all of a row.
template <int NW, int WR>
__global__ __launch_bounds__(kWinThreads, kWinPerSimd) void corr_window_kernel(const float *__restrict__ in, const float *__restrict__ f,
                                                                                 float *__restrict__ out, const WindowGeom g)
{
    constexpr int NL = 3, G = 2, PER = WR / G;
    static_assert(WR % G == 0, "steps start at the same slots every PER of them");
    constexpr int TP = win_tap_pitch(NW);
    extern __shared__ __align__(16) unsigned char win_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x;
    const int col = lane & 15, kg = lane >> 4;
    const int CL = g.C * g.L;

    // taps: copy k, granule n: taps T0 + 8 n + k .. + 7
    {
        const float *f_c = f + (size_t)c * (size_t)g.K;
        const int T0 = 16 * g.q0 - g.phi + g.pad - 15;
        constexpr int NG = 4 * NW + 6;
        for (int i = tid; i < 8 * NG; i += 64 * g.waves) {
            const int k = i & 7, n = i >> 3, j = T0 + 8 * n + k;
            Raw8F raw;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int jj = min(max(j + v, 0), g.K - 1);
                raw.v[v] = __float_as_uint(f_c[g.reverse ? g.K - 1 - jj : jj]);
            }
#pragma unroll
            for (int v = 0; v < 8; ++v) raw.v[v] = (unsigned)(j + v) < (unsigned)g.K ? raw.v[v] : 0u;
            uintx4 limbs[NL];
            raw8_limbs(raw, limbs);
#pragma unroll
            for (int l = 0; l < NL; ++l) *reinterpret_cast<uintx4 *>(win_smem + (8 * l + k) * TP + 16 * n) = limbs[l];
        }
    }
    __syncthreads();
    const int stride = (int)gridDim.y * g.waves;
    int unit = (int)blockIdx.y * g.waves + wave;
    if (unit >= g.units) return;
    const unsigned char *a_base = win_smem + ((15 - col) & 7) * TP + 16 * (kg + ((15 - col) >> 3));

    // the load cursor.  Load q of a pair of chunks: lane i brings granule (i % 16) ^ row of row 4 q + i / 16
    int ld_unit = unit, ld_s = g.s_first, ld_u[4], ld_off[4], ld_b0 = 0;
    const int w0 = (g.q0 + 1) >> 1;
    auto ld_place = [&]() {
        const int first = ld_unit * kWinCols;
        ld_b0 = g.NP > 1 ? (int)__umulhi((unsigned)first, g.np_magic) : first;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 4 * q + (lane >> 4), mine = first + row;
            const int b = g.NP > 1 ? (int)__umulhi((unsigned)mine, g.np_magic) : mine;
            const int u = (mine - b * g.NP) * g.P - g.phi + 4 * ((lane & 15) ^ row) + 32 * (G * g.s_first + w0 + NW - 1);
            ld_u[q] = b < g.B ? u : -(1 << 30);
            ld_off[q] = 4 * ((b - ld_b0) * CL + u);
        }
    };
    const unsigned ring = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) const void *)(win_smem + NL * 8 * TP + wave * kWinRing * 4096));
    int ld_slot = 0;
    auto load = [&]() {
        const size_t off = ((size_t)ld_b0 * (size_t)g.C + (size_t)c) * (size_t)g.L;
        const size_t left = 4 * ((size_t)g.B * (size_t)CL - off);
        const unsigned long long ad = reinterpret_cast<unsigned long long>(in + off);
        const uintx4 rsrc = {(unsigned)ad, (unsigned)(ad >> 32) & 0xffffu, (unsigned)(left < 0x3fffffff ? left : 0x3fffffff), kBufferFlags};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            buffer_load_x4_to_lds_keep(rsrc, (unsigned)ld_u[q] < (unsigned)g.L ? ld_off[q] : kOutOfRow, ring + (unsigned)ld_slot + 1024u * q);
        ld_slot ^= 4096;
    };
    auto ld_next = [&]() {
        if (++ld_s == g.ns) {
            ld_unit += stride;
            ld_s = g.s_first;
            if (ld_unit < g.units) {
                ld_place();
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) ld_u[q] = -(1 << 30);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ld_u[q] += 32 * G;
                ld_off[q] += 128 * G;
            }
        }
    };
    // the compute cursor.  cu: the lane's first position in chunk 0 of its column; store q of a step: granule (i % 16) ^ row of row
    // 4 q + i / 16, st_left of its positions from there to the end of the piece
    int s = g.s_first, cu = 0, st_off[4], st_left[4], st_b0 = 0;
    auto cu_place = [&]() {
        const int mine = unit * kWinCols + col, b = g.NP > 1 ? (int)__umulhi((unsigned)mine, g.np_magic) : mine;
        cu = (mine - b * g.NP) * g.P - g.phi + 8 * kg;
    };
    auto st_place = [&]() {
        const int first = unit * kWinCols;
        st_b0 = g.NP > 1 ? (int)__umulhi((unsigned)first, g.np_magic) : first;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 4 * q + (lane >> 4), mine = first + row;
            const int b = g.NP > 1 ? (int)__umulhi((unsigned)mine, g.np_magic) : mine;
            const int t0 = (mine - b * g.NP) * g.P, at = 4 * ((lane & 15) ^ row);
            st_left[q] = b < g.B ? min(t0 + g.P, g.L) - t0 - at : 0;
            st_off[q] = 4 * ((b - st_b0) * CL + t0 + at);
        }
    };
    ld_place();
    load();
    ld_next();
    load();
    cu_place();
    st_place();

    uintx4 X[WR][NL];
#pragma unroll
    for (int i = 0; i < WR; ++i)
#pragma unroll
        for (int l = 0; l < NL; ++l) X[i][l] = uintx4{0u, 0u, 0u, 0u};
    const bool ragged = (g.L & 3) != 0;
    const int tiles_len = g.NP > 1 ? g.P : g.L;

    // the chunk pair of step s to its slots (chunks behind the rows' last are never read, and on short rows their slots hold others)
    auto convert = [&](auto phc) {
        constexpr int PH = decltype(phc)::value;
        const int u0 = cu + 32 * (G * s + w0 + NW - 1);
        wait_vmcnt_at_most<4>();                                         // (the pair after it is the last that was asked for)
        const unsigned char *from = win_smem + NL * 8 * TP + wave * kWinRing * 4096 + ld_slot + 256 * col;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (G * s + w0 + NW - 1 + i > g.chi) continue;
            Raw8F r;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uintx4 v4 = *reinterpret_cast<const uintx4 *>(from + 16 * ((8 * i + 2 * kg + h) ^ col));
#pragma unroll
                for (int v = 0; v < 4; ++v) r.v[4 * h + v] = v4[v];
            }
            // (positions behind the end of a row in the granule in which it ends: those of the next row)
            if (ragged && __any(u0 + 32 * i + 7 >= g.L)) {
#pragma unroll
                for (int v = 0; v < 8; ++v) r.v[v] = u0 + 32 * i + v < g.L ? r.v[v] : 0u;
            }
            raw8_limbs(r, X[(G * PH + i) % WR]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // the four tiles of step s.  Chunks outside the rows, tiles behind their end and q without taps are skipped
    floatx4 res[2 * G];
    auto compute = [&](auto phc) {
        constexpr int PH = decltype(phc)::value;
        // window index i of this step: slot
        constexpr int BASE = ((G * (PH + 1) - (NW + G - 1)) % WR + WR) % WR;
        const int first = w0 + G * s;
        const int lo = max(g.clo - first, 0), hi = min(g.chi - first, 30);
        const unsigned live = hi < lo ? 0u : ((2u << hi) - 1u) & ~((1u << lo) - 1u);
        const int tiles = (tiles_len - 64 * s + 15) >> 4;
        uintx4 a[2][NL];
        auto read_limb = [&](uintx4 (&to)[NL], int l, int n) { to[l] = *reinterpret_cast<const uintx4 *>(a_base + 8 * l * TP + 32 * n); };
        // n-th q of the step, odd ones first: granule 2 k of the odd, 2 k + 1 of the even
        auto granule = [](int i) { return i < NW ? 2 * i : 2 * (i - NW) + 1; };
#pragma unroll
        for (int l = NL - 1; l >= 0; --l) read_limb(a[0], l, 0);
        const unsigned ks[2] = {(1u << (g.qn >> 1)) - 1u, (1u << ((g.qn + 1) >> 1)) - 1u};
        auto finish = [&](int par, const floatx4 (&big)[G], const floatx4 (&mid)[G], floatx4 (&low)[G]) {
            float check = 0.f;
#pragma unroll
            for (int j = 0; j < G; ++j) {
#pragma unroll
                for (int v = 0; v < 4; ++v) low[j][v] = __builtin_fmaf(__builtin_fmaf(low[j][v], 0x1p-8f, mid[j][v]), 0x1p-8f, big[j][v]);
                check = __builtin_fmaf(low[j][0], low[j][1], __builtin_fmaf(low[j][2], low[j][3], check));
            }
            // (a sum that is not finite, or finite ones above 10^19: as limb_sum)
            if (__any(!__builtin_isfinite(check))) {
#pragma unroll
                for (int j = 0; j < G; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) low[j][v] = __builtin_isfinite(low[j][v]) ? low[j][v] : big[j][v];
            }
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) res[par + 2 * j][v] = 4.f * low[j][v];
        };
        // Behind products that a branch may have passed by: the compiler counts the wait states from a product to the read of its sum along
        // the way through the branch only, and along the other one the sum was read two states behind it instead of eight, without that
        // product in it
        auto settle = [](floatx4 (&big)[G], floatx4 (&mid)[G], floatx4 (&low)[G]) {
            asm volatile("s_nop 7" : "+v"(big[0]), "+v"(big[1]), "+v"(mid[0]), "+v"(mid[1]), "+v"(low[0]), "+v"(low[1]));
        };
        constexpr unsigned ALL = (1u << (NW + 1)) - 1u;
        if (tiles >= 4 && (live & ALL) == ALL && ks[0] == ALL >> 1) {
#pragma unroll
            for (int par = 1; par >= 0; --par) {
                floatx4 big[G], mid[G], low[G];
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    const int i = (par ? 0 : NW) + k;
                    const bool next = i + 1 < 2 * NW;
                    const uintx4 (&x0)[NL] = X[(BASE + k) % WR];
                    const uintx4 (&x1)[NL] = X[(BASE + k + 1) % WR];
                    uintx4 (&av)[NL] = a[0];
                    // (a limb of the next taps is read behind the last product of this one)
                    low[0] = mfma16x16x32(av[2], x0[0], k ? low[0] : zero);
                    low[1] = mfma16x16x32(av[2], x1[0], k ? low[1] : zero);
                    if (next) read_limb(av, 2, granule(i + 1));
                    mid[0] = mfma16x16x32(av[1], x0[0], k ? mid[0] : zero);
                    mid[1] = mfma16x16x32(av[1], x1[0], k ? mid[1] : zero);
                    low[0] = mfma16x16x32(av[1], x0[1], low[0]);
                    low[1] = mfma16x16x32(av[1], x1[1], low[1]);
                    if (next) read_limb(av, 1, granule(i + 1));
                    big[0] = mfma16x16x32(av[0], x0[0], k ? big[0] : zero);
                    big[1] = mfma16x16x32(av[0], x1[0], k ? big[1] : zero);
                    mid[0] = mfma16x16x32(av[0], x0[1], mid[0]);
                    mid[1] = mfma16x16x32(av[0], x1[1], mid[1]);
                    low[0] = mfma16x16x32(av[0], x0[2], low[0]);
                    low[1] = mfma16x16x32(av[0], x1[2], low[1]);
                    if (next) read_limb(av, 0, granule(i + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
                finish(par, big, mid, low);
            }
        } else {
#pragma unroll
            for (int par = 1; par >= 0; --par) {
                floatx4 big[G], mid[G], low[G];
                unsigned m[G];
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    big[j] = mid[j] = low[j] = floatx4{0.f, 0.f, 0.f, 0.f};
                    m[j] = par + 2 * j < tiles ? (live >> j) & ks[par] : 0u;
                }
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    const int i = (par ? 0 : NW) + k;
                    constexpr int SETS = WR == 6 ? 2 : 1;
                    uintx4 (&av)[NL] = a[i % SETS], (&an)[NL] = a[(i + 1) % SETS];
                    if (SETS == 2 && i + 1 < 2 * NW) {
#pragma unroll
                        for (int l = NL - 1; l >= 0; --l) read_limb(an, l, granule(i + 1));
                    }
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        if (m[j] >> k & 1u) {
                            const uintx4 (&x)[NL] = X[(BASE + k + j) % WR];
                            low[j] = mfma16x16x32(av[2], x[0], low[j]);
                            mid[j] = mfma16x16x32(av[1], x[0], mid[j]);
                            big[j] = mfma16x16x32(av[0], x[0], big[j]);
                            low[j] = mfma16x16x32(av[1], x[1], low[j]);
                            mid[j] = mfma16x16x32(av[0], x[1], mid[j]);
                            low[j] = mfma16x16x32(av[0], x[2], low[j]);
                        }
                    }
                    if (SETS == 1 && i + 1 < 2 * NW) {
#pragma unroll
                        for (int l = NL - 1; l >= 0; --l) read_limb(an, l, granule(i + 1));
                    }
                }
                settle(big, mid, low);
                finish(par, big, mid, low);
            }
        }
    };
    // The tiles of a step through the ring's free slot, so that a store is whole rows of 256 bytes: straight from the tiles it is
    // pieces of 64
    auto store = [&](int s_done) {
        const size_t at = ((size_t)st_b0 * (size_t)g.C + (size_t)c) * (size_t)g.L;
        const size_t rest = 4 * ((size_t)g.B * (size_t)CL - at);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(out + at, 0, (int)(rest < 0x3fffffff ? rest : 0x3fffffff), kBufferFlags);
        unsigned char *free_slot = win_smem + NL * 8 * TP + wave * kWinRing * 4096 + ld_slot;
#pragma unroll
        for (int i = 0; i < 2 * G; ++i) *reinterpret_cast<floatx4 *>(free_slot + 256 * col + 16 * ((4 * i + kg) ^ col)) = res[i];
        wave_lds_fence();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uintx4 v = *reinterpret_cast<const uintx4 *>(free_slot + 1024 * q + 16 * lane);
            const int n = st_left[q] - 64 * s_done, o = st_off[q] + 256 * s_done;
            if (n >= 4) {
                if (g.lines) __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, o, 0, 2);
                else __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, o, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < n) __builtin_amdgcn_raw_buffer_store_b32(v[e], rsrc, o + 4 * e, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    convert(std::integral_constant<int, 0>{});
    ld_next();
    load();
    bool done = false;
    auto step = [&](auto phc) {
        constexpr int PH = decltype(phc)::value;
        const bool has = s >= 0;
        if (has) compute(phc);
        const int s_done = s;
        bool last = false, next = false;
        if (++s == g.ns) {
            unit += stride;
            s = g.s_first;
            next = true;
            if (unit < g.units) cu_place();
            else last = true;
        }
        if (!last) convert(std::integral_constant<int, (PH + 1) % PER>{});
        else wait_vmcnt_at_most<4>();                                    // (of loads past the end, into the slot that the tiles take)
        if (has) store(s_done);
        if (next && !last) st_place();
        if (!last) {
            ld_next();
            load();
        }
        done = last;
    };
    auto walk = [&](auto self, auto phc) -> void {
        constexpr int PH = decltype(phc)::value;
        if constexpr (PH < PER) {
            step(phc);
            if (!done) self(self, std::integral_constant<int, PH + 1>{});
        }
    };
    while (!done) walk(walk, std::integral_constant<int, 0>{});
    wait_vmcnt_at_most<0>();                                             // (no load may write LDS that is no longer this workgroup's)
}

}  // namespace dwconv
