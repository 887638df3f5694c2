// Stage 1 of the weight gradient (Sec. IV-A eq. (dk_def)) for filters of hundreds of taps and more: the forward kernel's form
// (dwconv_band.hip.h) with a row of dY as the filter.  With the lag o = j - pad,
//
//   dw[o] = sum_b sum_t dY[b][t] X[b][t + o],      G[r][col] = sum_e sum_k Toep_e[r][k] X[16 e + k + 32 col],
//   Toep_e[r][k] = dY[16 e + k - r]
//
// a tile is 32 x 32 lags (lag 32 col + r), on v_mfma_f32_32x32x16_bf16 in either storage type (fp32: three bf16 limbs per
// operand, six of the nine limb products, dwconv_band.hip.h).  What bounds dw_band_kernel on such filters is its staging: it
// brings, splits and transposes every row once per window of twelve or sixteen offsets (eight rows of 51 blocks for 240 block
// pairs).  Here a stage of F positions of dY and 1024 T + F of X serves 1024 T x F products, nothing is transposed, lags are
// summed where they are (no diagonals), and a single batch entry fills the operands as well as eight.  A tile is 1024 lags
// whatever the filter, so shorter filters leave columns idle: dw_band_kernel has them (dw_takes_toep).
//
// What bounds it (counters, B8 C256 K = L = 8192): fp32 the matrix pipe, 78 % of the launch's cycles under a lowered clock (dw_band_kernel
// 54 %): 775-793 -> 619-654 us; bf16 LDS reads (78 %) and the matrix pipe (65 %; dw_band_kernel 59 % and 30 %): 201 -> 131-135 us.  Relative
// error of the fp32 gradient against 64 bits there (2-norm, normal data) 2.3e-7 -> 1.7e-7.  A few batch entries on few channels: the chain of
// a stage, some 1.2 us of loads, splitting, barriers, and its products (fp32 B1 C365 L5675 K5675 causal 215 -> 73 us, bf16 B2 C384
// L1150 K1150 17 -> 8.3).
//
// Workgroup (c, slice, piece): T tiles of lags, the rows of its slice in chunks of F positions; the four waves split the e of a
// chunk.  The next chunk's granules are loaded into registers while one is multiplied.  Pieces go out in falling order of
// their work (lag 0 meets a whole row, lag L - 1 one position), so that the short ones fill in behind the long ones.
#pragma once
#include "dwconv_band.hip.h"

namespace dwconv {

struct DwToepGeom {
    int B, C, L, K, pad;
    int blk0, nblk;     // 32-blocks of lags, block m being lags 32 m + shift ..: the first (may be negative), how many there are (all
    int shift;          // lags inside (-L, L) that have a tap are in them, and possibly more in front)
    int npiece;         // pieces of T tiles
    int piece0;         // the launch's first (in its order)
    int F;              // positions of dY per chunk (a multiple of 32)
    int rows;           // batch entries per slice
    int run;            // the e (of all four waves) between two additions to the totals (fp32: up to half as many more), a multiple of 4
    int chain;          // bf16: the least e between two, at the ends of stages (fp32: after each run)
    int tap_off;        // byte offset of the taps in LDS
};
constexpr int kToepThreads = 256;
constexpr int kToepX = 4, kToepY = 2;       // granules of eight positions a thread brings per stage: of X, of dY
constexpr int toep_blocks(int T, int F) { return 32 * T + F / 32 + 1; }    // blocks of X a stage reads at most
inline size_t dw_toep_tap_offset(int NL, int blocks)
{
    const size_t stage = (size_t)blocks * (size_t)band_block_bytes(NL), red = (size_t)kBandWaves * 32 * kBandRedPitch * 4;
    return stage > red ? stage : red;
}
inline size_t dw_toep_lds_bytes(int NL, int blocks, int F) { return dw_toep_tap_offset(NL, blocks) + (size_t)NL * 8 * (size_t)band_tap_dwords(F); }
// The granule moved up by sh elements (0 .. 7), zeros in front: what a granule that starts before its row becomes when the first
// eight elements of the row were loaded in its place.
__device__ __forceinline__ void shift_up_raw8(Raw8F &r, int sh)
{
#pragma unroll
    for (int step = 4; step > 0; step >>= 1) {
        const bool on = (sh & step) != 0;
#pragma unroll
        for (int i = 7; i >= 0; --i) r.v[i] = on ? (i >= step ? r.v[i - step] : 0u) : r.v[i];
    }
}
__device__ __forceinline__ void shift_up_raw8(Raw8H &r, int sh)
{
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        const bool on = (sh & (2 * step)) != 0;
#pragma unroll
        for (int i = 3; i >= 0; --i) r.v[i] = on ? (i >= step ? r.v[i - step] : 0u) : r.v[i];
    }
#pragma unroll
    for (int i = 3; i >= 0; --i) r.v[i] = (sh & 1) ? __builtin_amdgcn_alignbit(r.v[i], i > 0 ? r.v[i - 1] : 0u, 16) : r.v[i];
}
// A stage: positions t0 .. t0 + F - 1 of dY of one batch entry and the blocks of X that the piece's lags reach from them.
struct DwToepStage {
    int b, t0;
    int e_lo, e_hi;                 // the e that hold a position of the chunk and meet the row from some lag of the piece
    int wb0, n8;                    // first window block, granules of eight positions
    int inside;                     // all of the window inside the row
};
// Block m + e / 2, half e % 2, of the window is positions 32 m + 16 e + shift .. + 15: inside the row from some k for 2 m + e in
// [-before, nch).
__host__ __device__ __forceinline__ int dw_toep_before(const DwToepGeom &g) { return (15 + g.shift) >> 4; }
__host__ __device__ __forceinline__ int dw_toep_chunks(const DwToepGeom &g) { return ((g.L - 1 - g.shift) >> 4) + 1; }
// Its window, from t0, for the PB blocks of lags from p0 on; false: no position of the chunk meets the row.
__host__ __device__ __forceinline__ bool dw_toep_set_window(const DwToepGeom &g, int p0, int PB, DwToepStage &s)
{
    const int before = dw_toep_before(g), nch = dw_toep_chunks(g);
    const int first = s.t0 >> 4, e0 = -2 * (p0 + PB - 1) - before, t1 = s.t0 + g.F < g.L ? s.t0 + g.F : g.L, last = (t1 + 30) >> 4, e1 = nch - 1 - 2 * p0;
    s.e_lo = first > e0 ? first : e0;
    s.e_hi = last < e1 ? last : e1;
    if (s.e_lo > s.e_hi) return false;
    const int wb_min = -31 - ((before + 1) >> 1), wb_max = ((nch - 1) >> 1) + 31;        // blocks that any tile reads
    const int w0 = p0 + (s.e_lo >> 1), w1 = p0 + PB - 1 + (s.e_hi >> 1);
    s.wb0 = w0 > wb_min ? w0 : wb_min;
    s.n8 = 4 * ((w1 < wb_max ? w1 : wb_max) - s.wb0 + 1);
    s.inside = s.wb0 >= 0 && 32 * s.wb0 + g.shift + 8 * s.n8 <= g.L;
    return true;
}
// The e of a stage that meet the row from the tile that starts with block m0 of lags (behind the last block: a spare one).
__host__ __device__ __forceinline__ void dw_toep_tile_range(const DwToepGeom &g, const DwToepStage &s, int m0, int &lo, int &hi)
{
    const int e0 = -2 * (m0 + 31) - dw_toep_before(g), e1 = dw_toep_chunks(g) - 1 - 2 * m0;
    lo = s.e_lo > e0 ? s.e_lo : e0;
    hi = s.e_hi < e1 ? s.e_hi : e1;
    if (m0 >= g.blk0 + g.nblk) {
        lo = kNoWorkLo;
        hi = kNoWorkHi;
    }
}
// Sets of accumulators: bf16, one tile, two, for even and odd e, which halves the chains (of two tiles: B8 C256 K = L = 8192 133 -> 143 us)
constexpr int toep_sets(int NL, int T) { return NL == 1 && T == 1 ? 2 : 1; }
constexpr int toep_waves(int NL, int T) { return NL == 3 && T == 2 ? 2 : 3; }

template <typename E, int T>
__global__ __launch_bounds__(kToepThreads, toep_waves(Limbs<E>::N, T)) void dw_toep_kernel(
    const E *__restrict__ x, const E *__restrict__ dy, float *__restrict__ part, E *__restrict__ dw_out, const DwToepGeom g, int slices)
{
    constexpr int NL = Limbs<E>::N, BS = band_block_bytes(NL), THREADS = kToepThreads, KS = kBandWaves, PB = 32 * T;
    static_assert(T == 1 || T == 2, "register budget");
    extern __shared__ __align__(16) unsigned char toep_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x, sl = (int)blockIdx.y;
    int piece;
    {
        // rank z counts from the piece that holds lag 0 outwards, on both sides while there are two
        const int zero = min(max(-g.blk0 / PB, 0), g.npiece - 1), k = g.piece0 + (int)blockIdx.z;
        const int both = min(zero, g.npiece - 1 - zero);
        if (k <= 2 * both) piece = (k & 1) ? zero - (k + 1) / 2 : zero + k / 2;
        else piece = zero > both ? g.npiece - 1 - k : k;
    }
    const int p0 = g.blk0 + piece * PB;
    const int TP = band_tap_dwords(g.F);
    unsigned char *xs = toep_smem;
    unsigned *fs = reinterpret_cast<unsigned *>(toep_smem + g.tap_off);          // limb l, copy p at (2 l + p) TP
    const size_t CL = (size_t)g.C * (size_t)g.L;
    const int b_end = min(g.B, (sl + 1) * g.rows);

    typedef DwToepStage Stage;
    auto settle = [&](Stage &s) {       // the first stage from s on that has work; b >= b_end: none
        for (;; s.t0 += g.F) {
            if (s.t0 >= g.L) { s.t0 = 0; ++s.b; }
            if (s.b >= b_end) return;
            if (dw_toep_set_window(g, p0, PB, s)) return;
        }
    };
    decltype(load_raw8(x)) px[kToepX], py[kToepY];
    E prev[kToepY];                                                      // the element in front of each granule of dY
    auto prefetch = [&](const Stage &s) {
        const int tl = band_hide(tid);
        const E *xr = x + ((size_t)s.b * CL + (size_t)c * (size_t)g.L), *yr = dy + ((size_t)s.b * CL + (size_t)c * (size_t)g.L);
#pragma unroll
        for (int i = 0; i < kToepX; ++i)
            if (i * THREADS < s.n8) px[i] = load_raw8(xr + max(0, min(32 * s.wb0 + g.shift + 8 * (tl + i * THREADS), g.L - 8)));
#pragma unroll
        for (int i = 0; i < kToepY; ++i)
            if (8 * i * THREADS < g.F) {
                const int t = s.t0 + 8 * (tl + i * THREADS);
                py[i] = load_raw8(yr + min(t, g.L - 8));
                prev[i] = yr[max(0, min(t - 1, g.L - 1))];
            }
    };
    auto put = [&](const Stage &s) {
        const int tl = band_hide(tid);
#pragma unroll
        for (int i = 0; i < kToepX; ++i) {
            const int gi = tl + i * THREADS;
            if (gi < s.n8) {
                if (!s.inside) {
                    const int u = 32 * s.wb0 + g.shift + 8 * gi;
                    if (u + 8 > g.L) shift_raw8(px[i], (u + 8 - g.L) & 7);
                    if (u < 0) shift_up_raw8(px[i], -u & 7);
                    zero_raw8(px[i], u <= -8 || u >= g.L);
                }
                uintx4 limbs[NL];
                raw8_limbs(px[i], limbs);
#pragma unroll
                for (int l = 0; l < NL; ++l) *reinterpret_cast<uintx4 *>(xs + (gi >> 2) * BS + (gi & 3) * 16 + 64 * l) = limbs[l];
            }
        }
        // Dword 24 + m: taps 2 m, 2 m + 1 of the chunk in the one copy, 2 m - 1, 2 m in the other.  (The even and the odd lanes of a
        // read then take the same dwords of the two copies, 16 of 32 banks apart; with 2 m + 1, 2 m + 2 in the other they met in a bank,
        // and a third of the LDS cycles were conflicts)
#pragma unroll
        for (int i = 0; i < kToepY; ++i) {
            const int gi = tl + i * THREADS;
            if (8 * gi < g.F) {
                const int t = s.t0 + 8 * gi;
                if (t + 8 > g.L) shift_raw8(py[i], (t + 8 - g.L) & 7);
                zero_raw8(py[i], t >= g.L);
                const float pv = gi > 0 && t <= g.L ? ld_elem(&prev[i]) : 0.f;
                uintx4 limbs[NL];
                unsigned before8[NL];
                raw8_limbs(py[i], limbs);
                pair_limbs(0.f, pv, before8);
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    unsigned *to = fs + 2 * l * TP + kBandTapMargin / 2 + 4 * gi;
                    *reinterpret_cast<uintx4 *>(to) = limbs[l];
                    uintx4 odd;
#pragma unroll
                    for (int k = 0; k < 4; ++k) odd[k] = __builtin_amdgcn_alignbit(limbs[l][k], k > 0 ? limbs[l][k - 1] : before8[l], 16);
                    *reinterpret_cast<uintx4 *>(to + TP) = odd;
                    if (8 * gi + 8 == g.F) to[TP + 4] = limbs[l][3] >> 16;
                }
            }
        }
    };

    constexpr int SETS = toep_sets(NL, T);
    floatx16 acc[SETS][T], mid[NL == 3 ? T : 1], low[NL == 3 ? T : 1], total[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            acc[0][t][i] = acc[SETS - 1][t][i] = total[t][i] = 0.f;
            if constexpr (NL == 3) mid[t][i] = low[t][i] = 0.f;
        }
    Stage cur;
    cur.b = sl * g.rows; cur.t0 = 0;
    settle(cur);
    if (cur.b < b_end) prefetch(cur);
    // (the margins of the taps stay zero)
    for (int m = tid; m < TP; m += THREADS)
        if (m < kBandTapMargin / 2 || m >= kBandTapMargin / 2 + g.F / 2)
#pragma unroll
            for (int l = 0; l < 2 * NL; ++l) fs[l * TP + m] = 0u;
    // The sums of the tiles t0 .. t0 + n - 1 added to totals of their own, so that no chain of additions gets long.
    auto fold = [&](auto t0c, auto nc) {
        constexpr int T0 = decltype(t0c)::value, N = decltype(nc)::value;
#pragma unroll
        for (int t = T0; t < T0 + N; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if constexpr (NL == 3) {
                    total[t][i] += limb_sum(acc[0][t][i], mid[t][i], low[t][i]);
                    mid[t][i] = low[t][i] = 0.f;
                } else {
                    total[t][i] += SETS == 2 ? acc[0][t][i] + acc[SETS - 1][t][i] : acc[0][t][i];
                    acc[SETS - 1][t][i] = 0.f;
                }
                acc[0][t][i] = 0.f;
            }
    };
    int since = 0;                                                       // bf16: the e since the totals were added to
    while (cur.b < b_end) {
        __syncthreads();                                                 // everyone is done with what LDS holds
        put(cur);
        __syncthreads();
        Stage nxt = cur;
        nxt.t0 += g.F;
        settle(nxt);
        if (nxt.b < b_end) prefetch(nxt);

        const int ln = band_hide(lane), col = ln & 31, kg = ln >> 5;
        // A: dY[16 e + 8 kg + v - r], r = col.  B: the lane's column of tile t, block p0 + 32 t + col + e / 2, half e % 2.
        const int a0 = 8 * kg - col - cur.t0 + kBandTapMargin;
        const unsigned *a_base = fs + (a0 & 1) * TP + ((a0 + 1) >> 1);
        const unsigned char *b_base = xs + 16 * kg + (col + p0 - cur.wb0) * BS;
        int lo[T], hi[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            dw_toep_tile_range(g, cur, p0 + 32 * t, lo[t], hi[t]);
            asm volatile("" : "+s"(lo[t]), "+s"(hi[t]));                // (hidden, as in corr_band_kernel)
        }
        // e = ea .. eb (those of this wave: ks modulo 4) for the tiles T0 .. T0 + N - 1
        auto run = [&](auto t0c, auto nc, int ea, int eb) {
            constexpr int T0 = decltype(t0c)::value, N = decltype(nc)::value;
            ea += (cur.e_lo + ks - ea) & (KS - 1);
            if (ea > eb) return;
            const unsigned *ap = a_base + 8 * ea;
            const unsigned char *bp = b_base + (32 * T0 + (ea >> 1)) * BS + (ea & 1) * 32;
            auto read_limb = [&](uintx4 (&to)[NL], int l) {
#pragma unroll
                for (int i = 0; i < 4; ++i) to[l][i] = ap[2 * l * TP + i];
            };
            auto read_b = [&](uintx4 (&to)[NL], int t) {
#pragma unroll
                for (int l = 0; l < NL; ++l) to[l] = *reinterpret_cast<const uintx4 *>(bp + 32 * t * BS + 64 * l);
            };
            auto step = [&](int e) {                                     // (past the last e: the same addresses again)
                const bool more = e + KS <= eb;
                ap += more ? 8 * KS : 0;
                bp += more ? (KS / 2) * BS : 0;
            };
            if constexpr (NL == 3) {
                // the operands of the next tile are read while this one's are multiplied, each limb of A behind its last product
                uintx4 a[NL], b[2][NL];
#pragma unroll
                for (int l = 0; l < NL; ++l) read_limb(a, l);
                read_b(b[0], 0);
#pragma unroll 1
                for (int e = ea; e <= eb;) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {                        // (two e per trip: two register sets)
                        if (u == 0 || e <= eb) {
#pragma unroll
                            for (int t = 0; t < N; ++t) {
                                const int k = u * N + t, tt = T0 + t;
                                const bool last = t + 1 == N;
                                const uintx4 (&bb)[NL] = b[k & 1];
                                if (last) step(e);
                                read_b(b[(k + 1) & 1], last ? 0 : t + 1);
                                low[tt] = mfma32x32x16(a[2], bb[0], low[tt]);
                                if (last) read_limb(a, 2);
                                low[tt] = mfma32x32x16(a[1], bb[1], low[tt]);
                                mid[tt] = mfma32x32x16(a[1], bb[0], mid[tt]);
                                if (last) read_limb(a, 1);
                                acc[0][tt] = mfma32x32x16(a[0], bb[0], acc[0][tt]);
                                mid[tt] = mfma32x32x16(a[0], bb[1], mid[tt]);
                                low[tt] = mfma32x32x16(a[0], bb[2], low[tt]);
                                if (last) read_limb(a, 0);
                            }
                            e += KS;
                        }
                    }
                }
            } else {
                // all operands of the next e are read while this one's are multiplied
                uintx4 a[2][NL], b[2][N][NL];
                auto read_e = [&](int u) {
                    read_limb(a[u], 0);
#pragma unroll
                    for (int t = 0; t < N; ++t) read_b(b[u][t], t);
                };
                read_e(0);
#pragma unroll 1
                for (int e = ea; e <= eb;) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (u == 0 || e <= eb) {
                            step(e);
                            read_e(1 - u);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int t = 0; t < N; ++t) acc[u % SETS][T0 + t] = mfma32x32x16(a[u][0], b[u][t][0], acc[u % SETS][T0 + t]);
                            __builtin_amdgcn_sched_barrier(0);
                            e += KS;
                        }
                    }
                }
            }
        };
        // (the tiles lie in increasing order of their lags, so lo and hi fall with t)
        active_runs(lo, hi, [&](auto ac, auto nc, int ea, int eb) {
            if constexpr (NL == 3) {
#pragma unroll 1
                while (ea <= eb) {
                    const int to = ea + g.run + (g.run >> 1) > eb ? eb : ea + g.run - 1;      // (no short rest)
                    run(ac, nc, ea, to);
                    fold(ac, nc);
                    ea = to + 1;
                }
            } else {
#pragma unroll 1
                for (; ea <= eb; ea += g.run) {
                    run(ac, nc, ea, min(eb, ea + g.run - 1));
                    if (ea + g.run <= eb) fold(ac, nc);
                }
            }
        });
        if constexpr (NL == 1) {
            since += cur.e_hi - cur.e_lo + 1;
            if (since >= g.chain || nxt.b >= b_end) {
                since = 0;
                fold(std::integral_constant<int, 0>{}, std::integral_constant<int, T>{});
            }
        }
        cur = nxt;
    }

    // ---- the waves' parts of a tile are added in wave order on their way through LDS; wave w stores columns 8 w .. 8 w + 7
    float *red = reinterpret_cast<float *>(toep_smem);
    {
        const int col = lane & 31, kg = lane >> 5;
        // lane (column, half kg) holds lags 8 q + 4 kg + 0..3 in elements 4 q .. 4 q + 3
        float *wr = red + ks * 32 * kBandRedPitch + col * kBandRedPitch + 4 * kg;
        const int o_col = 8 * ks + (lane >> 3), o_pos = 4 * (lane & 7);
        const float *rd = red + o_col * kBandRedPitch + o_pos;
        const size_t row = (size_t)c * (size_t)g.K;
        float *dst = part + ((size_t)sl * (size_t)g.C * (size_t)g.K + row);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = total[t][4 * q + i];
                *reinterpret_cast<floatx4 *>(wr + 8 * q) = v;
            }
            __syncthreads();
            floatx4 v = *reinterpret_cast<const floatx4 *>(rd);
#pragma unroll
            for (int k = 1; k < KS; ++k) v += *reinterpret_cast<const floatx4 *>(rd + k * 32 * kBandRedPitch);
            const int blk = p0 + 32 * t + o_col, j = 32 * blk + g.shift + o_pos + g.pad;
            if (blk < g.blk0 + g.nblk) {
                if (j >= 0 && j + 3 < g.K) {
                    const float4 v4 = make_float4(v[0], v[1], v[2], v[3]);
                    if (dw_out) st4_any(dw_out + row + j, v4);
                    else st4_any(dst + j, v4);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (j + i >= 0 && j + i < g.K) {
                            if (dw_out) st_elem(dw_out + row + j + i, v[i]);
                            else dst[j + i] = v[i];
                        }
                }
            }
        }
        // taps whose lag lies outside (-L, L), and the slices of the workspace beyond those of this launch: zeros
        const int j_lo = 32 * g.blk0 + g.shift + g.pad, j_hi = j_lo + 32 * g.nblk;
        if (g.piece0 + (int)blockIdx.z == 0) {
            for (int j = tid; j < g.K; j += THREADS)
                if (j < j_lo || j >= j_hi) {
                    if (dw_out) st_elem(dw_out + row + j, 0.f);
                    else dst[j] = 0.f;
                }
            if (!dw_out)
                for (int o = sl + (int)gridDim.y; o < slices; o += (int)gridDim.y)
                    for (int j = tid; j < g.K; j += THREADS) part[(size_t)o * (size_t)g.C * (size_t)g.K + row + j] = 0.f;
        }
    }
}

}  // namespace dwconv
