// Forward / input gradient (Sec. IV-A eq. (dwconv) and its adjoint) for filters of more than six 16-blocks, up to any
// length, on rows of any length and alignment: the blocked-Toeplitz contraction on v_mfma_f32_32x32x16_bf16, the bf16
// instruction in either storage type.
//
//   Y[t + r][col] = sum_e sum_k Toep_e[r][k] X[t + 16 e + k][col],    Toep_e[r][k] = w[16 e + k - r + pad]
//
// A tile is 32 output positions (r) x 32 columns; a column is one 32-position block of one row, and the columns of a
// tile are NB consecutive blocks of 32 / NB batch entries of a channel.  Its operands: A (lane r, half kg) eight
// consecutive taps, B (lane col, half kg) eight consecutive positions.
//
// fp32 storage on the bf16 instruction: every operand is the exact sum of three bf16 limbs (24 = 8 + 8 + 8 significant bits,
// rounded to nearest, so a limb is at most 2^-8 of the one before it); products of limbs are exact in fp32, sums fp32.
// Six of the nine limb products are kept; the three left out are together at most 2^-24 of the product, the unit roundoff
// of fp32.  The limbs are kept scaled to the size of the operand, with an accumulator for each scale of their products
// (split_pair, limb_sum).
// The instruction does sixteen times the fp32 one's products a cycle, so six of them are 2.7 times cheaper (an fp32
// matrix kernel is bound by the matrix pipe from about seven block offsets on).
//
// A workgroup (four waves) works on items of RW rows x PB blocks of a channel and walks the filter in chunks of F taps.  Per
// chunk the taps and the input window the chunk reaches (zeros outside the row) are staged as limbs, the window through
// registers that are loaded while the stage before it is multiplied; blocks of 32 positions are 80 bytes apart, so the
// 16-byte operand reads of eight neighbouring lanes fall on different banks (measured 220 bytes a cycle and compute
// unit; 63 at the natural 64 bytes).  The waves split the tiles TG ways and the e of a chunk KS = 4 / TG ways, so
// a wave has up to T tiles per A operand: 3 + 3 T reads for 6 T instructions.  Rounds through LDS add the KS parts in a fixed
// order and turn the tiles into whole rows for the stores.
#pragma once
#include "dwconv_common.hip.h"
#include "dwconv_mfma.hip.h"
#include "dwconv_dw_direct.hip.h"

namespace dwconv {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ floatx16 mfma32x32x16(uintx4 a, uintx4 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The three limbs of HALF of x and of y, the second times 2^8 and the third times 2^16: they are then all of the size of the
// operand, so every fp32 value from 2^-125 on keeps its bits, and the smaller ones theirs but the last, 2^-149 (unscaled, the third
// limb of a value below 2^-110 would lie below the smallest bf16: values around 2^-125 had an error of one per cent; the scaled
// ones and their third accumulator cost 1 % of a step of B2048 C128 L256 K256, 512 -> 520 us).  Halves, because
// rounding may take a first limb (and a product of two) up to 2^-8 past its value: no finite operand, and no product inside the
// range of a float, turns into infinity.
__device__ __forceinline__ void split_pair(float x, float y, unsigned (&p)[3])
{
    p[0] = pack_bf16(0.5f * x, 0.5f * y);
    x = 128.f * __builtin_fmaf(-2.f, __uint_as_float(p[0] << 16), x);
    y = 128.f * __builtin_fmaf(-2.f, __uint_as_float(p[0] & 0xffff0000u), y);
    p[1] = pack_bf16(x, y);
    x = 256.f * (x - __uint_as_float(p[1] << 16));
    y = 256.f * (y - __uint_as_float(p[1] & 0xffff0000u));
    p[2] = pack_bf16(x, y);
}
// The sum of products whose operands were halves: big holds the products of first limbs, mid those of a first and a second limb
// (times 2^8), low the others (times 2^16).  Where big is not finite it is what the definition gives (the first limb of an
// infinity is that infinity), and the small products - infinities of either sign, or the NaN that is left of an infinity behind its
// first limb - say nothing; nor do they where the sum of their absolute values exceeds the range of a float.
__device__ __forceinline__ float limb_sum(float big, float mid, float low)
{
    const float sum = __builtin_fmaf(__builtin_fmaf(low, 0x1p-8f, mid), 0x1p-8f, big);
    return 4.f * (__builtin_isfinite(sum) ? sum : big);
}

// Limbs per element: fp32 three, bf16 itself.
template <typename T> struct Limbs;
template <> struct Limbs<float> { static constexpr int N = 3; };
template <> struct Limbs<bf16_t> { static constexpr int N = 1; };

// Eight consecutive elements at any element-aligned address, as loaded (uintx4 pairs or one).
struct __attribute__((packed, aligned(4))) Raw8F { unsigned v[8]; };
struct __attribute__((packed, aligned(2))) Raw8H { unsigned v[4]; };
__device__ __forceinline__ Raw8F load_raw8(const float *p) { return *reinterpret_cast<const Raw8F *>(p); }
__device__ __forceinline__ Raw8H load_raw8(const bf16_t *p) { return *reinterpret_cast<const Raw8H *>(p); }
__device__ __forceinline__ void zero_raw8(Raw8F &r, bool zero)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) r.v[i] = zero ? 0u : r.v[i];
}
__device__ __forceinline__ void zero_raw8(Raw8H &r, bool zero)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = zero ? 0u : r.v[i];
}
// The granule moved down by sh elements (0 .. 7), zeros behind it: what a granule that ends behind its row becomes when the
// last eight elements of the row were loaded in its place.
__device__ __forceinline__ void shift_raw8(Raw8F &r, int sh)
{
#pragma unroll
    for (int step = 4; step > 0; step >>= 1) {
        const bool on = (sh & step) != 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) r.v[i] = on ? (i + step < 8 ? r.v[i + step] : 0u) : r.v[i];
    }
}
__device__ __forceinline__ void shift_raw8(Raw8H &r, int sh)
{
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        const bool on = (sh & (2 * step)) != 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.v[i] = on ? (i + step < 4 ? r.v[i + step] : 0u) : r.v[i];
    }
    const int bits = 16 * (sh & 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = __builtin_amdgcn_alignbit(i < 3 ? r.v[i + 1] : 0u, r.v[i], bits);
}
__device__ __forceinline__ void raw8_limbs(const Raw8F &r, uintx4 (&out)[3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned p[3];
        split_pair(__uint_as_float(r.v[2 * i]), __uint_as_float(r.v[2 * i + 1]), p);
        out[0][i] = p[0]; out[1][i] = p[1]; out[2][i] = p[2];
    }
}
__device__ __forceinline__ void raw8_limbs(const Raw8H &r, uintx4 (&out)[1])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) out[0][i] = r.v[i];
}
// The granule back to front.
__device__ __forceinline__ void reverse_raw8(Raw8F &r)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) { const unsigned t = r.v[i]; r.v[i] = r.v[7 - i]; r.v[7 - i] = t; }
}
__device__ __forceinline__ void reverse_raw8(Raw8H &r)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned t = r.v[i];
        r.v[i] = __builtin_amdgcn_alignbit(r.v[3 - i], r.v[3 - i], 16);
        r.v[3 - i] = __builtin_amdgcn_alignbit(t, t, 16);
    }
}
// Two neighbouring taps as limbs (zeros outside the chunk are passed in).
__device__ __forceinline__ void pair_limbs(float a, float b, unsigned (&p)[3]) { split_pair(a, b, p); }
__device__ __forceinline__ void pair_limbs(float a, float b, unsigned (&p)[1])
{
    p[0] = (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u);      // (widened bf16: exact)
}

// Four consecutive outputs at any element-aligned address.
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned uintx2_u __attribute__((ext_vector_type(2), aligned(2)));
__device__ __forceinline__ void st4_any(float *p, float4 v)
{
    floatx4_u t = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<floatx4_u *>(p) = t;
}
__device__ __forceinline__ void st4_any(bf16_t *p, float4 v)
{
    uintx2_u t = {pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
    *reinterpret_cast<uintx2_u *>(p) = t;
}

// a staged 32-position block: 64 bytes per limb + 16 (an odd number of 16-byte units)
__host__ __device__ constexpr int band_block_bytes(int NL) { return 64 * NL + 16; }
constexpr int kBandWaves = 4;
constexpr int kBandThreads = 64 * kBandWaves;
constexpr int kBandTapMargin = 48;           // zero taps in front of a staged chunk (and as many behind it)
constexpr int kBandRedPitch = 36;            // floats per column of the output image
// what a thread prefetches: granules of eight positions (fp32 8 registers each, bf16 4), pairs of taps
// (fp32, two tiles per wave: with at most four granules 167 registers, three waves per SIMD instead of two)
constexpr int band_prefetch(int NL) { return NL == 3 ? 5 : 10; }
constexpr int kBandPrefetchF32Few = 4;
constexpr int kBandTapPrefetch = 4;

// Places 0 .. N - 1 of a wave, place i with work from lo[i] to hi[i], both falling with i: call f(a, n, from, to) for the runs in
// which exactly the places a .. a + n - 1 have work, [lo[a], lo[a - 1]) and (hi[a + n], hi[a + n - 1]].  A place without any,
// wherever it stands, has its lo beyond every hi and its hi before every lo (either alone would put it into the runs of the places
// on one side of it).  (On the host too: a test follows the operand addresses of the kernels.)
template <int A, int B, int N, typename F>
__host__ __device__ __forceinline__ void active_runs_from(const int (&lo)[N], const int (&hi)[N], F &f)
{
    if constexpr (A < N) {
        int from = lo[A], to = hi[B];
        if constexpr (A > 0) to = to < lo[A - 1] - 1 ? to : lo[A - 1] - 1;
        if constexpr (B + 1 < N) from = from > hi[B + 1] + 1 ? from : hi[B + 1] + 1;
        f(std::integral_constant<int, A>{}, std::integral_constant<int, B - A + 1>{}, from, to);
        if constexpr (B + 1 < N) active_runs_from<A, B + 1>(lo, hi, f);
        else active_runs_from<A + 1, A + 1>(lo, hi, f);
    }
}
template <int N, typename F>
__host__ __device__ __forceinline__ void active_runs(const int (&lo)[N], const int (&hi)[N], F &&f)
{
    active_runs_from<0, 0>(lo, hi, f);
}
constexpr int kNoWorkLo = 1 << 28, kNoWorkHi = -(1 << 28);

struct BandGeom {
    int B, C, L, K;
    int pad;            // effective pad of this correlation
    int reverse;        // filter index reversed (input gradient)
    int nb_log;         // log2 of the blocks of a row that are columns of a tile
    int RW;             // rows per item = 32 >> nb_log
    int PB;             // 32-position blocks of a row per item (a whole number of tiles)
    int NP;             // pieces per row
    unsigned np_magic;  // floor(2^32 / NP) + 1: item / NP == umulhi(item, np_magic) for NP > 1
    int items;          // row groups x pieces of a channel
    int F;              // taps per chunk
    int pitch;          // bytes of one staged row
    int TG;             // tile groups; the e of a chunk are split W / TG ways
    int fold;           // TG - 1 (TG is a power of two): every other round of tiles over the groups goes back to front (causal filters: the
                        // work grows or falls along the row); otherwise 0
    int tile0;          // the first tile of the first round: negative where there are spare tiles and the work grows
};
// One stage of the walk: an item (RW rows x PB blocks) and a chunk of taps.
struct BandStage {
    int round, item, j0;            // item < 0: the walk has ended
    int b0, p0;                     // first row, first block of the item
    int e_lo, e_hi;                 // the e that hold a tap of the chunk and meet the row from some block of the piece
    int wb0, n8;                    // first window block any tile of the piece reads, granules of eight positions per row
    int inside;                     // every row of the item is in the batch and all of the window inside the rows
};
// Its window, from item and chunk; false: no tap of the chunk meets the row.
__host__ __device__ __forceinline__ bool band_set_window(const BandGeom &g, BandStage &s)
{
    const int NBk = 1 << g.nb_log, NCH = (g.L + 15) >> 4, NB32 = (g.L + 31) >> 5;
    // (arithmetic shifts: floor division)
    const int first = (s.j0 - g.pad) >> 4, e0 = -2 * (s.p0 + g.PB - 1);
    s.e_lo = first > e0 ? first : e0;
    const int j1 = s.j0 + g.F < g.K ? s.j0 + g.F : g.K, last = (j1 + 30 - g.pad) >> 4, e1 = NCH - 1 - 2 * s.p0;
    s.e_hi = last < e1 ? last : e1;
    if (s.e_lo > s.e_hi) return false;
    const int w0 = s.p0 + (s.e_lo >> 1), w1 = s.p0 + g.PB - 1 + (s.e_hi >> 1);
    s.wb0 = w0 > -(NBk - 1) ? w0 : -(NBk - 1);
    s.n8 = 4 * ((w1 < NB32 + NBk - 2 ? w1 : NB32 + NBk - 2) - s.wb0 + 1);
    s.inside = s.wb0 >= 0 && 32 * s.wb0 + 8 * s.n8 <= g.L && s.b0 + g.RW <= g.B;
    return true;
}
// The t-th tile of a wave of a tile group; whether an item has such a tile (the first block of the row behind the last: a spare one).
__host__ __device__ __forceinline__ int band_tile(const BandGeom &g, int group, int t) { return g.tile0 + g.TG * t + ((t & 1) ? group ^ g.fold : group); }
__host__ __device__ __forceinline__ bool band_has_tile(const BandGeom &g, int p0, int tile)
{
    const int rel = tile << g.nb_log;
    return p0 + rel < ((g.L + 31) >> 5) && (unsigned)rel < (unsigned)g.PB;
}
// The e of a stage that meet the row from a tile.
__host__ __device__ __forceinline__ void band_tile_range(const BandGeom &g, const BandStage &s, int tile, int &lo, int &hi)
{
    const int m0 = s.p0 + (tile << g.nb_log), NBk = 1 << g.nb_log;
    const int e0 = -2 * (m0 + NBk - 1), e1 = ((g.L + 15) >> 4) - 1 - 2 * m0;
    lo = s.e_lo > e0 ? s.e_lo : e0;
    hi = s.e_hi < e1 ? s.e_hi : e1;
    if (!band_has_tile(g, s.p0, tile)) {                                 // (in front or behind: active_runs)
        lo = kNoWorkLo;
        hi = kNoWorkHi;
    }
}

// dwords of one of the two copies of a chunk's taps (copies 16 banks apart: the even and the odd lanes of a read)
__host__ __device__ inline int band_tap_dwords(int F) { return ((F + 2 * kBandTapMargin) / 2 + 1 + 31) / 32 * 32 + 16; }
// the taps lie behind the window and behind the output image, which shares the window's place
__host__ __device__ inline unsigned band_tap_offset(int RW, int pitch)
{
    const unsigned stage = (unsigned)(RW * pitch), red = (unsigned)(kBandWaves * 32 * kBandRedPitch * 4);
    return stage > red ? stage : red;
}
inline size_t band_lds_bytes(int NL, int RW, int pitch, int F)
{
    return band_tap_offset(RW, pitch) + (size_t)NL * 8 * band_tap_dwords(F);
}

// A lane's number, hidden from the compiler at each use: it would keep every address that follows from it in a register
// for the whole kernel.
__device__ __forceinline__ int band_hide(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}
// waves per SIMD the kernel is compiled for
constexpr int band_waves(int NL, int T, int NPF) { return NL == 3 && T == 2 ? (NPF <= kBandPrefetchF32Few ? 3 : 2) : NL == 1 && T == 1 ? 4 : 3; }

//
// FOLD (fp32, filters in several chunks): the sums of a chunk are added to totals of their own behind it, so that no chain of
// additions is longer than the e of one chunk (B8 C256 K = L = 8192: error against 64 bits 1.7e-7 and 645 us, without 3.2e-7
// and 634 us; the fp32 instruction it replaced 5.6e-7 and 1007 us).
template <typename E, int T, bool FOLD = false, int NPF = band_prefetch(Limbs<E>::N)>
__global__ __launch_bounds__(kBandThreads, FOLD ? 2 : band_waves(Limbs<E>::N, T, NPF)) void corr_band_kernel(
    const E *__restrict__ in, const E *__restrict__ f, E *__restrict__ out, const BandGeom g)
{
    constexpr int NL = Limbs<E>::N;
    constexpr int W = kBandWaves, THREADS = kBandThreads;
    static_assert(T == 1 || T == 2 || (T == 4 && NL == 1), "register budget");
    extern __shared__ __align__(16) unsigned char band_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NBk = 1 << g.nb_log;
    const int c = blockIdx.x;
    const int tg = wave % g.TG, ks = wave / g.TG, KS = W / g.TG;
    constexpr int BS = band_block_bytes(NL);
    const int TP = band_tap_dwords(g.F);
    unsigned char *xs = band_smem;
    unsigned *fs = reinterpret_cast<unsigned *>(band_smem + band_tap_offset(g.RW, g.pitch));   // limb l, copy p at (2 l + p) TP
    const E *f_c = f + (size_t)c * (size_t)g.K;
    const E *in_c = in + (size_t)c * (size_t)g.L;
    const size_t CL = (size_t)g.C * (size_t)g.L;

    // (items y, 2 gy - 1 - y, 2 gy + y, ...: pieces of a causal filter cost what they lie from the start of the row, and this order
    // evens them out)
    typedef BandStage Stage;
    auto set_item = [&](Stage &s) {
        const int gy = (int)gridDim.y, y = (int)blockIdx.y;
        s.item = s.round * gy + ((s.round & 1) ? gy - 1 - y : y);
        if (s.item >= g.items) { s.item = -1; return; }      // (only the last round is short)
        const int rg = g.NP > 1 ? (int)__umulhi((unsigned)s.item, g.np_magic) : s.item;
        s.b0 = rg * g.RW;
        s.p0 = (s.item - rg * g.NP) * g.PB;
    };
    auto advance = [&](Stage &s, bool first) {
        for (;;) {
            if (first) {
                first = false;
            } else {
                s.j0 += g.F;
                if (s.j0 >= g.K) { s.j0 = 0; ++s.round; set_item(s); }
            }
            if (s.item < 0) return;
            if (band_set_window(g, s)) return;
        }
    };
    // The window of a stage travels through registers: its loads are issued before the stage in front of it is multiplied.
    // THREADS / RW neighbouring threads bring one row.
    const int tpr_log = 3 + g.nb_log;                     // log2(THREADS / RW)
    const int TPR = 1 << tpr_log;
    decltype(load_raw8(in)) pre[NPF];
    auto prefetch = [&](const Stage &s) {
        const int tl = band_hide(tid), ld_row = tl >> tpr_log, ld_g = tl & (TPR - 1);
        // (granules past the window: its last one again; rows past the batch, positions outside the row: loaded from inside, zeroed later)
        if constexpr (NL == 3) {
            // (one place for the loads: from two the compiler copies what one of them loads, and waits for it ahead of the products.  fp32 B285
            // C114 L2718 K140 forward 292 -> 275 us, B2048 C128 L256 K256 161 -> 152; bf16, whose registers fall the other way: L2718 121, 155 us)
            const E *row = in_c + (size_t)min(s.b0 + ld_row, g.B - 1) * CL;
            const int u0 = 32 * s.wb0 + 8 * ld_g, last = s.inside ? 32 * s.wb0 + 8 * (s.n8 - 1) : g.L - 8;
#pragma unroll
            for (int i = 0; i < NPF; ++i)
                if (i * TPR < s.n8) pre[i] = load_raw8(row + max(0, min(u0 + 8 * i * TPR, last)));
        } else if (s.inside) {
            const E *p = in_c + (size_t)(s.b0 + ld_row) * CL + (32 * s.wb0 + 8 * ld_g);
            const E *last = p + 8 * (s.n8 - 1 - ld_g);
#pragma unroll
            for (int i = 0; i < NPF; ++i)
                if (i * TPR < s.n8) pre[i] = load_raw8(ld_g + i * TPR < s.n8 ? p + 8 * i * TPR : last);
        } else {
            const E *row = in_c + (size_t)min(s.b0 + ld_row, g.B - 1) * CL;
            const int u0 = 32 * s.wb0 + 8 * ld_g;
#pragma unroll
            for (int i = 0; i < NPF; ++i)
                if (i * TPR < s.n8) pre[i] = load_raw8(row + max(0, min(u0 + 8 * i * TPR, g.L - 8)));
        }
    };
    // The taps of a chunk, likewise where there is more than one chunk.  Dword m of copy 0: taps 2 m, 2 m + 1 behind the margin; of copy 1:
    // 2 m + 1, 2 m + 2 for an odd pad, 2 m - 1, 2 m for an even one.  (The even lanes of a tap read take one copy, the odd ones the
    // other, and either way both the same dwords, 16 of 32 banks apart; with the first form for all pads they met in a bank on the even
    // ones: a third of the LDS cycles were conflicts, dx of bf16 B8 C256 K = L = 8192 129 -> 124 us.  Kernels of fewer tiles than there
    // can be have the small calls: a few more instructions ahead of the first product are 0.2 us of 7 there, and LDS is not what they
    // wait for)
    constexpr bool LONG = FOLD || T == (NL == 3 ? 2 : 4);
    const int odd_pad = LONG ? g.pad & 1 : 1;
    // ... dword by dword: the shortest way to the first product.  NTF of them per thread and chunk travel through registers (bf16)
    constexpr int NTF = kBandTapPrefetch;
    auto tap_triple = [&](int j0, int Fc, int m, E (&t3)[3]) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int jj = min(max(2 * m + i + odd_pad - 1 - kBandTapMargin, 0), Fc - 1);
            t3[i] = f_c[g.reverse ? g.K - 1 - (j0 + jj) : j0 + jj];
        }
    };
    auto store_triple = [&](int Fc, int m, const E (&t3)[3]) {
        const int jj = 2 * m + odd_pad - 1 - kBandTapMargin;
        float v[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = (jj + i >= 0 && jj + i < Fc) ? ld_elem(&t3[i]) : 0.f;
        unsigned p[NL], q[NL];
        pair_limbs(v[0], v[1], p);
        pair_limbs(v[1], v[2], q);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            fs[(2 * l + 1 - odd_pad) * TP + m] = p[l];
            fs[(2 * l + odd_pad) * TP + m] = q[l];
        }
    };
    // ... and by granules of eight, a tenth of the loads: filters of a thousand taps and more in one chunk, and every chunk of several
    // in fp32 (a granule of a thread in registers).  On shorter filters a thread's chain of instructions is what counts: 0.5 us of 6.
    typedef decltype(load_raw8(in)) Raw;
    const int n_taps8 = g.F / 8 + 1;                                     // (the last takes over what is left)
    auto load_taps = [&](int j0, int gi, Raw &raw, E &next) {
        // (from inside the filter: what lies outside the chunk is put right below)
        const int j = min(j0 + 8 * gi, g.K - 8), n = min(max(j0 + 8 * gi + (odd_pad ? 8 : -1), 0), g.K - 1);
        raw = load_raw8(f_c + (g.reverse ? g.K - 8 - j : j));
        next = f_c[g.reverse ? g.K - 1 - n : n];
    };
    auto store_taps = [&](int j0, int gi, Raw &raw, const E &next) {
        const int Fc = min(g.F, g.K - j0), over = j0 + 8 * gi - (g.K - 8);
        if (g.reverse) reverse_raw8(raw);
        if (over > 0) shift_raw8(raw, over & 7);
        zero_raw8(raw, 8 * gi >= Fc);
        const float v = (odd_pad ? 8 * gi + 8 < Fc : gi > 0 && 8 * gi <= Fc) ? ld_elem(&next) : 0.f;
        uintx4 limbs[NL];
        unsigned side[NL];
        raw8_limbs(raw, limbs);
        pair_limbs(v, v, side);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            unsigned *to = fs + 2 * l * TP + kBandTapMargin / 2 + 4 * gi;
            uintx4 odd;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                odd[k] = odd_pad ? __builtin_amdgcn_alignbit(k < 3 ? limbs[l][k + 1] : side[l], limbs[l][k], 16)
                                 : __builtin_amdgcn_alignbit(limbs[l][k], k > 0 ? limbs[l][k - 1] : side[l], 16);
            *reinterpret_cast<uintx4 *>(to) = limbs[l];
            *reinterpret_cast<uintx4 *>(to + TP) = odd;
            if (gi == 0) {
                to[-1] = 0u;
                to[TP - 1] = odd_pad ? limbs[l][0] << 16 : 0u;
            }
        }
    };
    const bool one_chunk = (NL == 3 && !FOLD) || g.K <= g.F;             // (fp32 in several chunks: FOLD)
    Raw tap8;
    E beside8, tap[FOLD ? 1 : NTF][3];
    auto prefetch_taps = [&](const Stage &s) {
        const int tl = band_hide(tid);
        if constexpr (FOLD) {
            load_taps(s.j0, min(tl, n_taps8 - 1), tap8, beside8);
        } else {
            const int Fc = min(g.F, g.K - s.j0);
#pragma unroll
            for (int i = 0; i < NTF; ++i)
                if (THREADS * i < TP) tap_triple(s.j0, Fc, tl + THREADS * i, tap[i]);
        }
    };

    floatx16 acc[T], mid[NL == 3 ? T : 1], low[NL == 3 ? T : 1], total[FOLD ? T : 1];
    Stage cur;
    cur.round = 0; cur.j0 = 0;
    set_item(cur);
    if (cur.item < 0) return;
    advance(cur, true);
    prefetch(cur);
    // (K >= 1024: bf16 B8 C256 L8192 K8192 125.9 -> 122.8 us, B1 C544 L6988 K6988 40.3 -> 39.4; in the kernels of fewer tiles the code alone, not run, took the registers of
    // their stages: bf16 B1579 C472 L112 K108 111 -> 125 us)
    const bool granules = FOLD || (LONG && one_chunk && g.K >= 1024);
    if (granules) {
        // (what lies in front of the taps and behind them stays zero)
        for (int m = tid; m < TP; m += THREADS)
            if (m < kBandTapMargin / 2 - 1 || m >= kBandTapMargin / 2 + 4 * n_taps8)
#pragma unroll
                for (int l = 0; l < 2 * NL; ++l) fs[l * TP + m] = 0u;
    }
    if (!one_chunk) {
        prefetch_taps(cur);
    } else if (granules) {
        // (not unrolled: what a launch runs through it first fetches from memory)
        Raw ahead;
        E ahead_beside;
        if (tid < n_taps8) load_taps(0, tid, ahead, ahead_beside);
#pragma unroll 1
        for (int gi = tid; gi < n_taps8; gi += THREADS) {
            Raw raw = ahead;
            const E beside = ahead_beside;
            if (gi + THREADS < n_taps8) load_taps(0, gi + THREADS, ahead, ahead_beside);
            store_taps(0, gi, raw, beside);
        }
        // (vmcnt 0: every load ahead has been used, but the compiler cannot tell, and would wait for its registers in every stage, also in
        // launches without granules: for the window that was just asked for)
        __builtin_amdgcn_s_waitcnt(0x0f70);
    } else {
        for (int m = tid; m < TP; m += THREADS) {
            E t3[3];
            tap_triple(0, g.K, m, t3);
            store_triple(g.K, m, t3);
        }
    }
    bool fresh = true;                                                   // first chunk of its item
    while (cur.item >= 0) {
        if (fresh) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    acc[t][i] = 0.f;
                    if constexpr (NL == 3) mid[t][i] = low[t][i] = 0.f;
                    if constexpr (FOLD) total[t][i] = 0.f;
                }
        }
        __syncthreads();                                                 // everyone is done with what LDS holds
        if (!one_chunk) {
            const int tl = band_hide(tid);
            if constexpr (FOLD) {
                if (tl < n_taps8) store_taps(cur.j0, tl, tap8, beside8);
            } else {
                const int Fc = min(g.F, g.K - cur.j0);
#pragma unroll
                for (int i = 0; i < NTF; ++i)
                    if (tl + THREADS * i < TP) store_triple(Fc, tl + THREADS * i, tap[i]);
            }
        }
        {
            const int tl = band_hide(tid), ld_row = tl >> tpr_log, ld_g = tl & (TPR - 1);
            unsigned char *dst = xs + ld_row * g.pitch + (ld_g >> 2) * BS + (ld_g & 3) * 16;
            const int dstep = (TPR >> 2) * BS;
            if (!cur.inside) {
                const int u0 = 32 * cur.wb0 + 8 * ld_g;
                const bool no_row = cur.b0 + ld_row >= g.B;
#pragma unroll
                for (int i = 0; i < NPF; ++i) {
                    const int u = u0 + 8 * i * TPR;
                    if (i * TPR < cur.n8) {
                        if (u + 8 > g.L) shift_raw8(pre[i], (u + 8 - g.L) & 7);
                        zero_raw8(pre[i], no_row || u < 0 || u >= g.L);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < NPF; ++i) {
                if (ld_g + i * TPR < cur.n8) {
                    uintx4 limbs[NL];
                    raw8_limbs(pre[i], limbs);
#pragma unroll
                    for (int l = 0; l < NL; ++l) *reinterpret_cast<uintx4 *>(dst + i * dstep + 64 * l) = limbs[l];
                }
            }
        }
        __syncthreads();
        Stage nxt = cur;
        advance(nxt, false);
        if (nxt.item >= 0) {
            prefetch(nxt);
            if (!one_chunk) prefetch_taps(nxt);
        }

        const int ln_m = band_hide(lane), col = ln_m & 31, kg = ln_m >> 5;
        // A: taps 16 e + 8 kg + v - r + pad, r = col: four dwords of the copy in which the first starts one.  B: the lane's column of tile t, block (m0 + blk + e / 2), half e % 2.
        const int a0 = 8 * kg - col + g.pad - cur.j0 + kBandTapMargin;
        const unsigned *a_base = fs + (a0 & 1) * TP + ((a0 + 1 - odd_pad) >> 1);
        const unsigned char *b_base = xs + (col >> g.nb_log) * g.pitch + 16 * kg + ((col & (NBk - 1)) + cur.p0 - cur.wb0) * BS;
        int rel[T], lo[T], hi[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            rel[t] = band_tile(g, tg, t) << g.nb_log;
            band_tile_range(g, cur, band_tile(g, tg, t), lo[t], hi[t]);
            // (hidden: the compiler would make a second set of loops for waves with a spare tile)
            asm volatile("" : "+s"(lo[t]), "+s"(hi[t]));
        }
        // e = ea .. eb (those of this wave: cur.e_lo + ks modulo KS) for the tiles T0 .. T0 + N - 1.  The operands of the next
        // tile are read while this one's are multiplied.
        auto run = [&](auto t0c, auto nc, int ea, int eb) {
            constexpr int T0 = decltype(t0c)::value, N = decltype(nc)::value;
            ea += (cur.e_lo + ks - ea) & (KS - 1);
            if (ea > eb) return;
            const unsigned *ap = a_base + 8 * ea;
            const unsigned char *bp[N];
#pragma unroll
            for (int t = 0; t < N; ++t) bp[t] = b_base + ((rel[T0 + t] + (ea >> 1)) * BS + (ea & 1) * 32);
            // (two register sets for A and B; fp32 one for A, whose limbs are each read again behind their last product: a dozen
            // registers less, and 1 % of B8 C256 K = L = 8192)
            constexpr int SETS = NL == 3 ? 1 : 2;
            uintx4 a[SETS][NL], b[2][NL];
            auto read_limb = [&](uintx4 (&to)[NL], int l) {
#pragma unroll
                for (int i = 0; i < 4; ++i) to[l][i] = ap[2 * l * TP + i];
            };
            auto read_b = [&](uintx4 (&to)[NL], int t) {
#pragma unroll
                for (int l = 0; l < NL; ++l) to[l] = *reinterpret_cast<const uintx4 *>(bp[t] + 64 * l);
            };
            auto step = [&](int e, bool more) {                          // (past the last e: the same addresses again)
                ap += more ? 8 * KS : 0;
                const int by = (KS & 1) ? ((e & 1) ? BS - 32 : 32) : (KS >> 1) * BS;
#pragma unroll
                for (int t = 0; t < N; ++t) bp[t] += more ? by : 0;
            };
#pragma unroll
            for (int l = 0; l < NL; ++l) read_limb(a[0], l);
            read_b(b[0], 0);
#pragma unroll 1
            for (int e = ea; e <= eb;) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {                            // (two e per trip: two register sets)
                    if (u == 0 || e <= eb) {
                        const bool more = e + KS <= eb;
#pragma unroll
                        for (int t = 0; t < N; ++t) {
                            const int k = u * N + t, tt = T0 + t;
                            const bool last = t + 1 == N;
                            const uintx4 (&bb)[NL] = b[k & 1];
                            if constexpr (NL == 3) {
                                uintx4 (&av)[NL] = a[0];
                                if (last) step(e, more);
                                read_b(b[(k + 1) & 1], last ? 0 : t + 1);
                                // (an accumulator for each scale: what rounds at the size of the sum is one addition per e, not six)
                                low[tt] = mfma32x32x16(av[2], bb[0], low[tt]);
                                if (last) read_limb(av, 2);
                                low[tt] = mfma32x32x16(av[1], bb[1], low[tt]);
                                mid[tt] = mfma32x32x16(av[1], bb[0], mid[tt]);
                                if (last) read_limb(av, 1);
                                acc[tt] = mfma32x32x16(av[0], bb[0], acc[tt]);
                                mid[tt] = mfma32x32x16(av[0], bb[1], mid[tt]);
                                low[tt] = mfma32x32x16(av[0], bb[2], low[tt]);
                                if (last) read_limb(av, 0);
                            } else {
                                if (t + 1 < N) {
                                    read_b(b[(k + 1) & 1], t + 1);
                                } else {
                                    step(e, more);
                                    read_limb(a[1 - u], 0);
                                    read_b(b[(k + 1) & 1], 0);
                                }
                                acc[tt] = mfma32x32x16(a[u][0], bb[0], acc[tt]);
                            }
                        }
                        e += KS;
                    }
                }
            }
        };
        // (the tiles lie in increasing order along the row, so lo and hi fall with t)
        active_runs(lo, hi, run);
        if constexpr (FOLD) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    total[t][i] += limb_sum(acc[t][i], mid[t][i], low[t][i]);
                    acc[t][i] = mid[t][i] = low[t][i] = 0.f;
                }
            }
        }
        fresh = nxt.item != cur.item;
        if (fresh) {
            // ---- tile t of every wave goes through LDS so that whole runs of a row are stored; where the e were split, the
            // parts are added there in order.  A thread owns four positions of one column; a tile is 256 of them.
            float *red = reinterpret_cast<float *>(band_smem);
            const int ln = band_hide(lane);
            const int col = ln & 31, kg = ln >> 5;
            // lane (column, half kg) holds outputs 8 q + 4 kg + 0..3 in elements 4 q .. 4 q + 3
            float *wr = red + wave * 32 * kBandRedPitch + col * kBandRedPitch + 4 * kg;
            // A thread stores four positions of one column; the columns of eight neighbouring threads' groups, eight apart,
            // lie a uniform distance apart (col8 of them: (8 col8 / NB) rows and (8 col8 % NB) blocks).
            const int o_col = ln >> 3, o_pos = 4 * (ln & 7);
            const int o_b = cur.b0 + (o_col >> g.nb_log), o_t = 32 * (cur.p0 + (o_col & (NBk - 1))) + o_pos;
            E *o_base = out + (size_t)o_b * CL + (size_t)c * (size_t)g.L + o_t;
            const bool whole = cur.b0 + g.RW <= g.B && 32 * (cur.p0 + g.PB) <= g.L;
            auto store4 = [&](int tile, int col8, floatx4 v) {
                const int db = (8 * col8) >> g.nb_log, dt = 32 * ((tile << g.nb_log) + ((8 * col8) & (NBk - 1)));
                E *o = o_base + ((size_t)db * CL + (size_t)dt);
                if (whole) {
                    st4_any(o, make_float4(v[0], v[1], v[2], v[3]));
                } else {
                    const int pos = o_t + dt;
                    if (o_b + db < g.B && pos < g.L) {                                 // (not a spare tile, column or position)
                        if (pos + 3 < g.L) {
                            st4_any(o, make_float4(v[0], v[1], v[2], v[3]));
                        } else {
                            st_elem(o, v[0]);
                            if (pos + 1 < g.L) st_elem(o + 1, v[1]);
                            if (pos + 2 < g.L) st_elem(o + 2, v[2]);
                        }
                    }
                }
            };
            const float *r_base = red + o_col * kBandRedPitch + o_pos;
            __syncthreads();                                             // everyone is done with the window
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (t > 0 && KS > 1) __syncthreads();
                if constexpr (FOLD) {
                    acc[t] = total[t];
                } else if constexpr (NL == 3) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[t][i] = limb_sum(acc[t][i], mid[t][i], low[t][i]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<floatx4 *>(wr + 8 * q) = floatx4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
                if (KS == 1) {
                    // the wave's own tile
                    wave_lds_fence();
                    const int tile = band_tile(g, tg, t);
                    if (band_has_tile(g, cur.p0, tile)) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            store4(tile, q, *reinterpret_cast<const floatx4 *>(r_base + (32 * wave + 8 * q) * kBandRedPitch));
                    }
                    wave_lds_fence();
                } else {
                    __syncthreads();
                    // wave w stores columns 8 w .. 8 w + 7 of every tile
                    for (int gq = 0; gq < g.TG; ++gq) {
                        const float *r = r_base + (32 * gq + 8 * wave) * kBandRedPitch;
                        floatx4 v = *reinterpret_cast<const floatx4 *>(r);
                        for (int k = 1; k < KS; ++k) v += *reinterpret_cast<const floatx4 *>(r + k * g.TG * 32 * kBandRedPitch);
                        const int tile = band_tile(g, gq, t);
                        if (band_has_tile(g, cur.p0, tile)) store4(tile, wave, v);
                    }
                }
            }
        }
        cur = nxt;
    }
}

}  // namespace dwconv
