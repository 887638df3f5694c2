// Weight gradient (eq. (dk_def)) for filters whose length is of the order of the sequence (K up to 8192, L up to 8192):
// the blocked form of dwconv_mfma.hip.h with hundreds of block offsets, split over the waves of a workgroup that keeps whole
// rows in LDS.  (Forward and input gradient of such filters: dwconv_band.hip.h.)
#pragma once
#include "dwconv_common.hip.h"
#include "dwconv_mfma.hip.h"

namespace dwconv {

constexpr int kLkWaves = 16;            // waves per workgroup (1024 threads)
constexpr int kLkRows = 2;              // rows staged together
constexpr int kLkMaxBlocks = 512;       // 16-blocks per row: L <= 8192
constexpr int kLkMaxK = 8192;

// ------------------------------------------------------------------------------------------------
// Stage 1 of the weight gradient for long filters (eq. (dk_def)):
//     G_d[q'][q] = sum_b sum_n X[n + d][q'] dY[n][q],      dw[j] = sum over 16 d + q' - q + pad = j.
// There are hundreds of offsets d, each with a 16x16 accumulator, so the offsets are what is split
// over waves: they are cut into contiguous groups of at most GD offsets and every one of the
// W = 16 * gridDim.y wave slots of a channel owns at most two groups.  An offset far from lag 0 reaches
// the row in few chunks, one near lag 0 in all of them, so the host sizes the groups and pairs heavy with
// light ones until the slots carry about equal work (LongKDwTable).  A workgroup stages two rows of x (256 zero floats on both
// sides) and of dY at a time; a wave walks the 64-position chunks that its groups can touch: one LDS
// dword of dY and, per offset, one of x feed one matrix instruction.  At the end each wave sums the
// diagonals of its accumulators into the taps of its groups and stores them into slice (group & 1)
// of the partial tensor: groups of equal parity own disjoint taps, so nothing is added in memory;
// the slices are zero-filled beforehand by fill_zero_kernel and summed by the ordinary stage 2.
constexpr int kLkDwMargin = 256;        // zero floats on both sides of a staged x row
constexpr int kLkDwMaxGD = 9;           // offsets per group (4 accumulator registers each, two groups per wave)

struct LongKDwGeom {
    int B, C, L, K, pad;
    int dmin, dmax;
    int NCH;        // 64-position chunks per row
    int bper;       // batch entries per batch slice (a multiple of the rows staged together): workgroup (c, y, z) walks
                    // entries z * bper .. and writes the slices 2 z and 2 z + 1, so that few channels or few offsets
                    // still fill the chip
};

// Which offsets a wave slot owns.  The block offsets dmin..dmax are cut into contiguous groups of 1..9 offsets
// (group i: offsets da[i] .. da[i] + n[i] - 1, in increasing order of i); every wave slot owns at most two groups.
// The host balances the work (offsets near the edge of the filter reach the row in few chunks, offsets near lag 0
// in all of them) and passes the table by value with the launch.
constexpr int kLkDwMaxGroups = 128;
constexpr int kLkDwMaxSlots = 64;
constexpr unsigned char kLkDwNoGroup = 255;
struct LongKDwTable {
    short da[kLkDwMaxGroups];
    unsigned char n[kLkDwMaxGroups];
    unsigned char g0[kLkDwMaxSlots], g1[kLkDwMaxSlots];
};

inline size_t longk_dw_lds_bytes(int L, int NCH)
{
    const size_t stage = sizeof(float) * (size_t)kLkRows * ((size_t)((L + 2 * kLkDwMargin + 3) & ~3) + (size_t)NCH * 64);
    const size_t reduce = sizeof(float) * (size_t)kLkWaves * (256 + 16 * kLkDwMaxGD + 32);   // epilogue scratch of every wave
    return stage > reduce ? stage : reduce;
}

__device__ __forceinline__ int floor_div(int a, int b) { return (a >= 0) ? a / b : -((-a + b - 1) / b); }
__device__ __forceinline__ int ceil_div(int a, int b) { return -floor_div(-a, b); }

template <int UNUSED = 0>   // (a template only so that the header can be included by several translation units)
__global__ __launch_bounds__(256) void fill_zero_kernel(float *__restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0.f;
}

// The chunks [ch_lo, ch_hi] of one staged row for a group of N offsets.
template <int N, int GD>
__device__ __forceinline__ void lk_dw_chunks(floatx4 (&G)[GD], const float *xp, const float *gp, int ch_lo, int ch_hi)
{
#pragma unroll 2
    for (int ch = ch_lo; ch <= ch_hi; ++ch) {
        const float gq = gp[64 * ch];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float xa = xp[64 * ch + 16 * i];
            G[i] = mfma16x16x4(xa, gq, G[i]);
        }
    }
}
// ... for a group size known at run time (wave-uniform)
template <int GD, int N = GD>
__device__ __forceinline__ void lk_dw_chunks_n(int n, floatx4 (&G)[GD], const float *xp, const float *gp, int ch_lo, int ch_hi)
{
    if (n == N) lk_dw_chunks<N, GD>(G, xp, gp, ch_lo, ch_hi);
    else if constexpr (N > 1) lk_dw_chunks_n<GD, N - 1>(n, G, xp, gp, ch_lo, ch_hi);
}

template <typename T, int GD>
__global__ __launch_bounds__(64 * kLkWaves, 4) void dw_longk_kernel(const T *__restrict__ x, const T *__restrict__ dy,
                                                                     float *__restrict__ part, const LongKDwGeom g,
                                                                     const LongKDwTable tb)
{
    extern __shared__ __align__(16) float lk_smem[];
    const int XW = (g.L + 2 * kLkDwMargin + 3) & ~3;        // floats of one staged x row
    const int GW = g.NCH * 64;                              // floats of one staged dY row
    float *sx = lk_smem;                                    // sx[rb * XW + kLkDwMargin + u] = x[u]
    float *sg = lk_smem + kLkRows * XW;                     // sg[rb * GW + t] = dy[t]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x;
    const int slot = (int)blockIdx.y * kLkWaves + wave;

    // the two groups of this wave: offsets [da, db] inclusive, empty if da > db
    int grp[2], da[2], db[2], nn[2], ch_lo[2], ch_hi[2];
    grp[0] = tb.g0[slot];
    grp[1] = tb.g1[slot];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool valid = grp[k] != kLkDwNoGroup;
        const int gi = valid ? grp[k] : 0;
        nn[k] = valid ? min((int)tb.n[gi], GD) : 0;
        da[k] = tb.da[gi];
        db[k] = da[k] + nn[k] - 1;
        // chunks in which some offset of the group reaches the row
        ch_lo[k] = max(0, ceil_div(-63 - 16 * db[k], 64));
        ch_hi[k] = valid ? min(g.NCH - 1, floor_div(g.L - 1 - 16 * da[k], 64)) : -1;
    }

    floatx4 G0[GD], G1[GD];
#pragma unroll
    for (int i = 0; i < GD; ++i) {
        G0[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        G1[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    const int b_begin = (int)blockIdx.z * g.bper, b_end = min(g.B, b_begin + g.bper);
    for (int b0 = b_begin; b0 < b_end; b0 += kLkRows) {
        __syncthreads();
        for (int rb = 0; rb < kLkRows; ++rb) {
            const int b = b0 + rb;
            float *xrow = sx + rb * XW;
            float *grow = sg + rb * GW;
            const size_t row = ((size_t)(b < b_end ? b : 0) * (size_t)g.C + (size_t)c) * (size_t)g.L;
            for (int i = tid; i < 2 * kLkDwMargin; i += 64 * kLkWaves)
                xrow[i < kLkDwMargin ? i : g.L + i] = 0.f;
            for (int gi0 = tid; gi0 < g.NCH * 16; gi0 += 64 * kLkWaves) {
                // (addresses recomputed from gi every trip rather than kept as induction variables across the whole
                // kernel, next to the accumulators)
                int gi = gi0;
                asm volatile("" : "+v"(gi));
                const int u = 4 * gi;
                float4 vx = make_float4(0.f, 0.f, 0.f, 0.f), vg = vx;
                if (b < b_end && u + 3 < g.L) {
                    vx = ld_elem4(x + row + u);
                    vg = ld_elem4(dy + row + u);
                }
                if (u + 3 < g.L) *reinterpret_cast<float4 *>(xrow + kLkDwMargin + u) = vx;
                *reinterpret_cast<float4 *>(grow + u) = vg;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            for (int rb = 0; rb < kLkRows; ++rb) {
                // A operand: X[n0 + kk + d][q'] = sx[64 ch + 16 d + lane];  B operand: dY[n0 + kk][q] = sg[64 ch + lane]
                const float *xp = sx + rb * XW + kLkDwMargin + 16 * da[k] + lane;
                const float *gp = sg + rb * GW + lane;
                if (k == 0) lk_dw_chunks_n<GD>(nn[0], G0, xp, gp, ch_lo[0], ch_hi[0]);
                else lk_dw_chunks_n<GD>(nn[1], G1, xp, gp, ch_lo[1], ch_hi[1]);
            }
        }
    }

    // ---- diagonal sums.  Wave-private scratch in the (now free) x region: 256 floats of one
    // accumulator plus the taps of one group, tap T = 16 i + e + 15 for offset da + i, e = q' - q.
    __syncthreads();
    constexpr int NTAP = 16 * GD + 32;
    float *scr = lk_smem + wave * (256 + NTAP);
    float *tap = scr + 256;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (da[k] > db[k]) continue;
        for (int i = lane; i < NTAP; i += 64) tap[i] = 0.f;
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < GD; ++i) {
            const floatx4 Gi = (k == 0) ? G0[i] : G1[i];
#pragma unroll
            for (int v = 0; v < 4; ++v) scr[(4 * (lane >> 4) + v) * 16 + (lane & 15)] = Gi[v];
            wave_lds_fence();
            if (lane < 31) {
                const int e = lane - 15;
                const int q_lo = e > 0 ? e : 0, q_hi = e > 0 ? 15 : 15 + e;
                float sum = 0.f;
                for (int qp = q_lo; qp <= q_hi; ++qp) sum += scr[qp * 16 + (qp - e)];
                if (da[k] + i <= db[k]) tap[16 * i + lane] += sum;     // a short last group owns fewer offsets
            }
            wave_lds_fence();
        }
        const int ntap = 16 * (db[k] - da[k]) + 31;
        float *dst = part + ((size_t)(2 * (int)blockIdx.z + (grp[k] & 1)) * (size_t)g.C + (size_t)c) * (size_t)g.K;
        for (int i = lane; i < ntap; i += 64) {
            const int j = 16 * da[k] + (i - 15) + g.pad;
            if (j >= 0 && j < g.K) dst[j] = tap[i];
        }
        wave_lds_fence();
    }
}

// ------------------------------------------------------------------------------------------------
// The same stage 1 for bf16 storage on the bf16 matrix instruction (v_mfma_f32_16x16x16_bf16): the contraction of
// one instruction runs over 16 consecutive blocks n, so a chunk is 256 positions and a wave issues a quarter of the
// instructions.  Same groups, same table, same epilogue as dw_longk_kernel (the accumulators have the same lane
// layout).  Lane (i = lane % 16, kg = lane / 16) holds the contraction entries k = 4 kg + v: element i of blocks
// n0 + 4 kg + v (+ d), v = 0..3.  So that these four values are ONE LDS read, the rows are staged transposed:
//     xt[i][m] = x[16 (m - 32) + i]   (16 lines of bf16, one entry per block, 32 zero blocks on both sides),
//     gt[i][n] = dy[16 n + i],
// and the operand of offset d is xt[i][32 + n0 + 4 kg + d .. + 3].  Its alignment is that of d: x is kept twice, the
// second copy shifted by one entry, which makes every operand two aligned dwords (ds_read2_b32); dY needs one copy
// (8-byte aligned).  Lines are 16 bytes modulo 256 apart: the 32 lanes of a half wave then read 64 different banks.
constexpr int kLkDwBf16MarginBlocks = 32;
__host__ __device__ inline int lk_bf16_line_bytes(int entries) { return (2 * entries + 255 - 16) / 256 * 256 + 16; }
inline size_t longk_dw_bf16_lds_bytes(int L)
{
    const int nb = (L + 255) / 256 * 16;                            // blocks per row, whole chunks
    const size_t xcopy = (size_t)16 * lk_bf16_line_bytes(nb + 2 * kLkDwBf16MarginBlocks);
    const size_t stage = (size_t)kLkRows * (2 * xcopy + (size_t)16 * lk_bf16_line_bytes(nb));
    const size_t reduce = sizeof(float) * (size_t)kLkWaves * (256 + 16 * kLkDwMaxGD + 32);
    return stage > reduce ? stage : reduce;
}

typedef __attribute__((address_space(3))) const uint32_t *lds_u32_ptr;
typedef unsigned int lk_uintx2 __attribute__((ext_vector_type(2)));

// The 256-position chunks [ch_lo, ch_hi] of one staged row for a group of N offsets.  The operand of offset da + i is
// the four entries m0 + i .. m0 + i + 3 of this lane's line.  Even i read them from the copy in which m0 is
// dword-aligned (xe: address of entry m0 there), odd i from the other copy (xo: entry m0 + 1): the windows of a copy
// overlap, so a chunk needs (N + 1) / 2 + 1 dwords of one copy and N / 2 + 1 of the other instead of two per
// offset.  ga: the dY operand.  A chunk further is 16 entries = 32 bytes.
template <int N, int GD>
__device__ __forceinline__ void lk_dw_chunks_bf16(floatx4 (&G)[GD], lds_u32_ptr xe, lds_u32_ptr xo, lds_u32_ptr ga,
                                                  int ch_lo, int ch_hi)
{
    constexpr int NE = (N + 1) / 2, NO = N / 2;
#pragma unroll 2
    for (int ch = ch_lo; ch <= ch_hi; ++ch) {
        const lk_uintx2 bw = {ga[8 * ch], ga[8 * ch + 1]};
        const shortx4 bq = __builtin_bit_cast(shortx4, bw);
        unsigned e[NE + 1], o[NO + 1];
#pragma unroll
        for (int t = 0; t <= NE; ++t) e[t] = xe[8 * ch + t];
#pragma unroll
        for (int t = 0; t <= NO; ++t) o[t] = NO > 0 ? xo[8 * ch + t] : 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const lk_uintx2 aw = (i & 1) ? lk_uintx2{o[i / 2], o[i / 2 + 1]} : lk_uintx2{e[i / 2], e[i / 2 + 1]};
            G[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(shortx4, aw), bq, G[i], 0, 0, 0);
        }
    }
}
template <int GD, int N = GD>
__device__ __forceinline__ void lk_dw_chunks_bf16_n(int n, floatx4 (&G)[GD], lds_u32_ptr xe, lds_u32_ptr xo, lds_u32_ptr ga,
                                                    int ch_lo, int ch_hi)
{
    if (n == N) lk_dw_chunks_bf16<N, GD>(G, xe, xo, ga, ch_lo, ch_hi);
    else if constexpr (N > 1) lk_dw_chunks_bf16_n<GD, N - 1>(n, G, xe, xo, ga, ch_lo, ch_hi);
}

template <int GD>
__global__ __launch_bounds__(64 * kLkWaves, 4) void dw_longk_bf16_kernel(const bf16_t *__restrict__ x,
                                                                          const bf16_t *__restrict__ dy,
                                                                          float *__restrict__ part, const LongKDwGeom g,
                                                                          const LongKDwTable tb)
{
    extern __shared__ __align__(16) unsigned char lkb_dw_smem[];
    constexpr int MB = kLkDwBf16MarginBlocks;
    const int NB = (g.L + 255) / 256 * 16;                  // blocks per row, whole chunks
    const int NC256 = NB / 16;
    const int XL = lk_bf16_line_bytes(NB + 2 * MB);         // bytes of one line of a transposed x copy
    const int GL = lk_bf16_line_bytes(NB);                  // ... of transposed dY
    const int XC = 16 * XL;                                 // bytes of one x copy
    const int ROWB = 2 * XC + 16 * GL;                      // bytes of one staged row: x copy 0, x copy 1, dY
    // row rb: x copy s at rb * ROWB + s * XC, entry (i, m) at + i * XL + 2 (m - s);  dY at rb * ROWB + 2 XC + i * GL + 2 n

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, kg = lane >> 4;
    const int c = blockIdx.x;
    const int slot = (int)blockIdx.y * kLkWaves + wave;

    // the two groups of this wave: offsets [da, db] inclusive, empty if da > db
    int grp[2], da[2], db[2], nn[2], ch_lo[2], ch_hi[2];
    grp[0] = tb.g0[slot];
    grp[1] = tb.g1[slot];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool valid = grp[k] != kLkDwNoGroup;
        const int gi = valid ? grp[k] : 0;
        nn[k] = valid ? min((int)tb.n[gi], GD) : 0;
        da[k] = tb.da[gi];
        db[k] = da[k] + nn[k] - 1;
        // chunks in which some offset of the group reaches the row: x positions 256 ch + 16 da .. 256 ch + 255 + 16 db
        ch_lo[k] = max(0, ceil_div(-255 - 16 * db[k], 256));
        ch_hi[k] = valid ? min(NC256 - 1, floor_div(g.L - 1 - 16 * da[k], 256)) : -1;
    }

    floatx4 G0[GD], G1[GD];
#pragma unroll
    for (int i = 0; i < GD; ++i) {
        G0[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        G1[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    // the margins of the x copies stay zero for the whole kernel: clear the staging region once
    for (int i = tid; i < kLkRows * ROWB / 16; i += 64 * kLkWaves)
        *reinterpret_cast<uint4 *>(lkb_dw_smem + 16 * i) = make_uint4(0u, 0u, 0u, 0u);

    const int b_begin = (int)blockIdx.z * g.bper, b_end = min(g.B, b_begin + g.bper);
    for (int b0 = b_begin; b0 < b_end; b0 += kLkRows) {
        __syncthreads();
        for (int rb = 0; rb < kLkRows; ++rb) {
            const int b = b0 + rb;
            unsigned char *x0 = lkb_dw_smem + rb * ROWB, *gt = x0 + 2 * XC;
            const size_t row = ((size_t)(b < b_end ? b : 0) * (size_t)g.C + (size_t)c) * (size_t)g.L;
#pragma unroll 1
            for (int gi0 = tid; gi0 < NB * 4; gi0 += 64 * kLkWaves) {
                // (the addresses below are recomputed from gi every time: kept as induction variables they would
                // occupy two dozen registers for the whole kernel, next to the accumulators)
                int gi = gi0;
                asm volatile("" : "+v"(gi));
                const int u = 4 * gi;
                uint2 vx = make_uint2(0u, 0u), vg = vx;
                if (b < b_end && u + 3 < g.L) {
                    vx = *reinterpret_cast<const uint2 *>(x + row + u);
                    vg = *reinterpret_cast<const uint2 *>(dy + row + u);
                }
                const int blk = u >> 4, i0 = u & 15;
                const uint16_t ex[4] = {(uint16_t)vx.x, (uint16_t)(vx.x >> 16), (uint16_t)vx.y, (uint16_t)(vx.y >> 16)};
                const uint16_t eg[4] = {(uint16_t)vg.x, (uint16_t)(vg.x >> 16), (uint16_t)vg.y, (uint16_t)(vg.y >> 16)};
                unsigned char *px = x0 + i0 * XL + 2 * (MB + blk), *pg = gt + i0 * GL + 2 * blk;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    *reinterpret_cast<uint16_t *>(px) = ex[e];
                    *reinterpret_cast<uint16_t *>(px + XC - 2) = ex[e];          // the copy shifted by one entry
                    *reinterpret_cast<uint16_t *>(pg) = eg[e];
                    px += XL;
                    pg += GL;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (nn[k] == 0) continue;
            for (int rb = 0; rb < kLkRows; ++rb) {
                const unsigned char *x0 = lkb_dw_smem + rb * ROWB;
                // operand of offset da + i: entries m0 + i .. m0 + i + 3, m0 = MB + 4 kg + da; copy s holds entry m at m - s
                const int m0 = MB + 4 * kg + da[k];
                const int sh = m0 & 1;                                   // (wave-uniform: the parity of da)
                const lds_u32_ptr xe = (lds_u32_ptr)(x0 + sh * XC + i16 * XL + 2 * (m0 - sh));
                const lds_u32_ptr xo = (lds_u32_ptr)(x0 + (1 - sh) * XC + i16 * XL + 2 * (m0 + sh));
                const lds_u32_ptr ga = (lds_u32_ptr)(x0 + 2 * XC + i16 * GL + 8 * kg);
                if (k == 0) lk_dw_chunks_bf16_n<GD>(nn[0], G0, xe, xo, ga, ch_lo[0], ch_hi[0]);
                else lk_dw_chunks_bf16_n<GD>(nn[1], G1, xe, xo, ga, ch_lo[1], ch_hi[1]);
            }
        }
    }

    // ---- diagonal sums.  Wave-private scratch in the (now free) staging region: 256 floats of one
    // accumulator plus the taps of one group, tap T = 16 i + e + 15 for offset da + i, e = q' - q.
    __syncthreads();
    constexpr int NTAP = 16 * GD + 32;
    float *scr = reinterpret_cast<float *>(lkb_dw_smem) + wave * (256 + NTAP);
    float *tap = scr + 256;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (da[k] > db[k]) continue;
        for (int i = lane; i < NTAP; i += 64) tap[i] = 0.f;
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < GD; ++i) {
            const floatx4 Gi = (k == 0) ? G0[i] : G1[i];
#pragma unroll
            for (int v = 0; v < 4; ++v) scr[(4 * (lane >> 4) + v) * 16 + (lane & 15)] = Gi[v];
            wave_lds_fence();
            if (lane < 31) {
                const int e = lane - 15;
                const int q_lo = e > 0 ? e : 0, q_hi = e > 0 ? 15 : 15 + e;
                float sum = 0.f;
                for (int qp = q_lo; qp <= q_hi; ++qp) sum += scr[qp * 16 + (qp - e)];
                if (da[k] + i <= db[k]) tap[16 * i + lane] += sum;     // a short last group owns fewer offsets
            }
            wave_lds_fence();
        }
        const int ntap = 16 * (db[k] - da[k]) + 31;
        float *dst = part + ((size_t)(2 * (int)blockIdx.z + (grp[k] & 1)) * (size_t)g.C + (size_t)c) * (size_t)g.K;
        for (int i = lane; i < ntap; i += 64) {
            const int j = 16 * da[k] + (i - 15) + g.pad;
            if (j >= 0 && j < g.K) dst[j] = tap[i];
        }
        wave_lds_fence();
    }
}

}  // namespace dwconv
