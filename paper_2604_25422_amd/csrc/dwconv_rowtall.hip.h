// Weight gradient of rows of 129 to 512 positions with filters of the order of the row length, four rows at a time (fp32, or
// bf16 storage widened to fp32 on the way into LDS).  Rows need to start on a dword only (bf16: even L): a last granule of
// four that holds elements of the next row gets zeros in their place on the way into LDS (see dwconv_rowbatch.hip.h).
// (Forward and input gradient of such rows: dwconv_band.hip.h.)
//
// The contraction runs over the rows (b, c) of one channel at the same block positions, and only block pairs inside the row
// are contracted, for rows of m = 9 .. 32 blocks: the accumulators are indexed by the relative block offset, fifteen per
// launch window (grid z); every window walks the batch on its own and owns the taps its offsets reach, its slices hold
// zeros elsewhere, and stage 2 adds the slices of all windows.
// Units are loaded without prefetch across the contraction (a few granules per lane at a time, waited for at once); two
// or three workgroups per compute unit, where LDS allows, hide the load of one behind the matrix work of another.
#pragma once
#include "dwconv_rowbatch.hip.h"

namespace dwconv {

constexpr int kRtMinBlocks = 9;        // rows of fewer blocks take the kernels of dwconv_rowbatch.hip.h
constexpr int kRtMaxBlocks = 32;       // rows of at most 512 positions
constexpr int kRtWaves = 4;            // waves per workgroup, each with a unit of its own
constexpr int kRtWindow = 15;          // relative block offsets per weight-gradient window

struct RowTallGeom {
    int B, C, L, K;
    int pad;
    int dmin, dmax;     // block offsets inside a row (cropped to -(m-1) .. m-1)
    int m;              // 16-blocks per row
    int n_units;        // ceil(B / 4)
    int win;            // relative block offsets per window (at most kRtWindow; the windows are of equal size)
    unsigned lg_recip;  // floor(2^32 / ceil(L / 4)) + 1: granule index -> (row of the unit, granule of the row)
};

// Stage 1 of the weight gradient for such rows.  grid = (C, S, windows), W = 4 waves per block; wave w of slice s takes
// the units W s + w, W s + w + W S, ... of four rows of its channel (walked from the last batch to the first, like the
// other weight-gradient kernels).  Window z owns the relative block offsets wlo = dmin + 15 z .. wlo + 14: accumulator e
// is offset wlo + e,  G_e[q'][q] += x[b][16 (mo + wlo + e) + q'] * dY[b][16 mo + q]  over the four rows b of a unit (the
// contraction index of one matrix instruction) and all output blocks mo whose partner lies inside the row.  The block
// writes slice z * S + s of part: the taps its window reaches, zeros elsewhere.
__host__ __device__ constexpr int rt_dw_pitch(int m)
{
    int p = 16 * m;
    while (p % 64 != 16 && p % 64 != 48) p += 16;
    return p;
}
__host__ __device__ constexpr int rt_dw_wave_floats(int m)
{
    const int stage = 2 * 4 * rt_dw_pitch(m);
    const int diag = ((16 * kRtWindow + 15) * 17 + 3) / 4 * 4;
    return stage > diag ? stage : diag;
}
__host__ __device__ constexpr size_t rt_dw_lds_bytes(int m)
{
    return (size_t)kRtWaves * (size_t)(rt_dw_wave_floats(m) + rb_tap_floats(kRtWindow)) * sizeof(float);
}

template <typename T>
__global__ __launch_bounds__(64 * kRtWaves, 2) void dw_rowtall_kernel(const T *__restrict__ x, const T *__restrict__ dy,
                                                                       float *__restrict__ part, const RowTallGeom g)
{
    constexpr int ES = (int)sizeof(T);
    constexpr int NE = kRtWindow;
    constexpr int RU = 4;                       // rows per unit: the contraction of one matrix instruction
    constexpr int NLD = RU * (16 * kRtMaxBlocks / 4) / 64;      // granule loads per lane, unit and tensor, at most (8)
    extern __shared__ __align__(16) float dyn_lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, k4 = lane >> 4;
    const int c = (int)blockIdx.x;
    const int wreg = rt_dw_wave_floats(g.m);
    float *s_wave = dyn_lds + wave * wreg;
    float *s_dw = dyn_lds + kRtWaves * wreg;          // [wave][rb_tap_floats(NE)]
    const int Lp = rt_dw_pitch(g.m);
    float *sx = s_wave, *sg = s_wave + RU * Lp;
    const int wlo = g.dmin + g.win * (int)blockIdx.z;  // first relative offset of this window
    const int whi = min(g.dmax, wlo + g.win - 1);      // ... and its last

    floatx4 G[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) G[e] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int i = lane; i < 2 * RU * Lp / 4; i += 64)
        *reinterpret_cast<float4 *>(s_wave + 4 * i) = make_float4(0.f, 0.f, 0.f, 0.f);
    wave_lds_fence();

    const int CL = g.C * g.L;
    const int Lg = (g.L + 3) >> 2;              // (the last granule of a row partial when L % 4 != 0)
    const int NG = RU * Lg;                     // granules of a unit, per tensor
    const int nld = (NG + 63) >> 6;             // loads per lane (wave-uniform)
    int gl_off[NLD], idx[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int gi = lane + 64 * i;
        const int row = (int)__umulhi((unsigned)gi, g.lg_recip);
        const int cg = gi - row * Lg;
        gl_off[i] = gi < NG ? ES * (row * CL + 4 * cg) : kOutOfRow;
        idx[i] = gi < NG ? ((row * Lp + 4 * cg) | (cg == Lg - 1 ? (g.L & 3) : 0)) : -1;      // (low bits: see corr_rowtall_kernel)
    }
    const int stride = (int)gridDim.y * kRtWaves;
    int unit = (int)blockIdx.y * kRtWaves + wave;
    // A unit is loaded and waited for before it is contracted (no registers that untracked loads are still writing stay
    // live across the contraction: see corr_rowtall_kernel); two workgroups per compute unit overlap instead.
    auto load_unit = [&](int u) {
        const int b0 = RU * (g.n_units - 1 - u);
        const int nr = g.B - b0 < RU ? g.B - b0 : RU;
        const size_t first = ((size_t)b0 * (size_t)g.C + (size_t)c) * (size_t)g.L;
        const uintx4 rx = rb_unit_resource(x + first, nr, CL, g.L);
        const uintx4 rg = rb_unit_resource(dy + first, nr, CL, g.L);
        typename Raw4<T>::type px[NLD], pg[NLD];
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            if (i < nld) {
                px[i] = Raw4<T>::load(rx, gl_off[i]);
                pg[i] = Raw4<T>::load(rg, gl_off[i]);
            }
        wait_untracked_loads();
        release_after_wait(px);
        release_after_wait(pg);
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            if (i < nld && idx[i] >= 0) {
                *reinterpret_cast<float4 *>(sx + (idx[i] & ~3)) = rb_granule<T>(px[i], idx[i] & 3);
                *reinterpret_cast<float4 *>(sg + (idx[i] & ~3)) = rb_granule<T>(pg[i], idx[i] & 3);
            }
    };
    const float *xrow = sx + k4 * Lp + i16;     // lane (q' = i16, row k4): x[row][16 mi + q']
    const float *grow = sg + k4 * Lp + i16;     // lane (q = i16, row k4): dY[row][16 mo + q]
    for (; unit < g.n_units; unit += stride) {
        load_unit(unit);
        wave_lds_fence();
        // one relative offset at a time over the output blocks whose partner lies inside the row: no branch inside the
        // loops (a test per matrix instruction left the matrix pipe waiting on its LDS reads: 26 against 42 TFLOP/s at L = K = 256)
        static_for<0, NE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            const int rel = wlo + e;
            if (rel <= whi) {
                const int mo_lo = rel < 0 ? -rel : 0;
                const int mo_hi = rel > 0 ? g.m - 1 - rel : g.m - 1;
                // (two chains of dependent matrix instructions, even and odd output blocks, added at the end)
                floatx4 acc = G[e], acc2 = floatx4{0.f, 0.f, 0.f, 0.f};
                const float *xp = xrow + 16 * rel;
                int mo = mo_lo;
#pragma unroll 2
                for (; mo + 1 <= mo_hi; mo += 2) {
                    acc = mfma16x16x4(xp[16 * mo], grow[16 * mo], acc);
                    acc2 = mfma16x16x4(xp[16 * mo + 16], grow[16 * mo + 16], acc2);
                }
                if (mo <= mo_hi) acc = mfma16x16x4(xp[16 * mo], grow[16 * mo], acc);
                G[e] = acc + acc2;
            }
        });
        wave_lds_fence();       // (the images are rewritten by the next unit's loads)
    }

    // ---- per-wave diagonal sums over this window's offsets, then the waves of the block in wave order
    // (rb_diagonal_sums with accumulator e = relative offset wlo + e: its M chosen so that e - (M - 1) is that offset)
    const int TF = rb_tap_floats(NE);
    rb_diagonal_sums<NE>(G, 1 - wlo, s_wave, s_dw + wave * TF, lane, g.K, g.pad, wlo, NE);
    wave_lds_fence();
    __syncthreads();
    const int j0 = rb_tap_j0(g.pad, wlo), j1 = rb_tap_j1(g.K, g.pad, wlo, NE);
    const size_t slice = (size_t)blockIdx.z * (size_t)gridDim.y + (size_t)blockIdx.y;
    for (int j = tid; j < g.K; j += 64 * kRtWaves) {
        float sum = 0.f;
        if (j >= j0 && j < j1) {
#pragma unroll
            for (int w = 0; w < kRtWaves; ++w) sum += s_dw[w * TF + (j - j0)];
        }
        part[(slice * (size_t)g.C + (size_t)c) * (size_t)g.K + (size_t)j] = sum;
    }
}

}  // namespace dwconv
