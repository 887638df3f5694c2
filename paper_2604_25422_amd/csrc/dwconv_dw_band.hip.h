// Stage 1 of the weight gradient (Sec. IV-A eq. (dk_def)) for filters of more than six 16-blocks, up to any length, on rows of
// any length and alignment, on v_mfma_f32_32x32x16_bf16 in either storage type (fp32: three exact bf16 limbs per operand,
// six of the nine limb products, see dwconv_band.hip.h).
//
//   G_d[q'][q] += X[m + d][q'] dY[m][q]      (32-blocks m, block offsets d),      dw[j] = sum over 32 d + q' - q + pad = j
//
// The sixteen entries of a contraction are eight rows of a channel at two neighbouring blocks: lane (q', half kg) holds element
// q' of block m + d + kg of the eight rows, so LDS holds, per position, the eight rows side by side (16 bytes per limb), every
// operand is one aligned 16-byte read whatever the offset, and staging transposes in registers: a thread brings four
// positions of eight rows and writes four times eight rows.  Positions are permuted inside every 32 (pos ^ ((pos >> 3) & 3))
// so that those writes fall on different banks.
//
// Workgroup (c, slice, window): 4 ND / KS offsets of one channel over every S-th stage; a stage is 8 RGN (virtual) rows x S32
// blocks of dY and the blocks of x its offsets reach.  The waves split the offsets DG ways and the block pairs KS = 4 / DG
// ways.  Few batch entries (fewer than five): rows are cut into nseg virtual rows of Lv positions, each with its own piece of
// dY.
// Several windows (more than twelve offsets in fp32, sixteen in bf16): a tap takes its products from two neighbouring
// offsets, so a window shares its last offset with the next one and owns the taps that need no other window's offsets.
//
// Filters of a thousand taps and more mostly go to dw_toep_kernel (dwconv_dw_toep.hip.h).
//
// What bounds it (counters: share of a launch's cycles in which the unit is busy).  Short rows, B2048 C128 K = L = 256 fp32: matrix pipe
// 44 %, vector ALU 39 % (splitting and transposing), 150-166 us of which two reads of memory are 104 (204-210 before the waves of a
// group shared its items and the offsets were dealt, 27 % and 42 %; 366 on the fp32 instruction): one stage in LDS at a time, so that
// these only overlap across the two workgroups of a compute unit.  The reads of the next operand go out ahead of each group of
// products, the loads of the next stage ahead of a stage's.  Relative error against 64 bits (2-norm, normal data): fp32 B8 C256
// K = L = 8192 2.3e-7, the fp32 instruction 9.4e-7.
#pragma once
#include "dwconv_band.hip.h"

namespace dwconv {

struct DwBandGeom {
    int B, C, L, K, pad;
    int dmin, nd;       // block offsets (of 32) that hold a tap and have a block pair inside a row
    int ndw;            // offsets per window: ND (per wave) x DG
    int dg_log;         // log2 of the offset groups among the waves (DG; KS = 4 / DG).  (Powers of two as their logarithms, other
                        // divisors with the reciprocals they need: a division by a number of run time is some 200 cycles, and
                        // a small call is a few thousand)
    int nwin;           // window w: offsets from dmin + w (ndw - 1)
    int nseg, Lv;       // virtual rows per row and their length (a multiple of 64; nseg == 1: the row)
    unsigned seg_magic; // floor(2^16 / nseg) + 1: v / nseg == v * seg_magic >> 16 for the at most eight virtual rows there are
    int rg_log;         // log2 of the groups of eight virtual rows per stage (RGN)
    int S32;            // dY blocks per stage (even)
    int nstep;          // stages along a virtual row
    unsigned step_magic;// floor(2^32 / nstep) + 1: st / nstep == umulhi(st, step_magic); 0: too many stages for that
    int stages;         // all stages
    int chain;          // stages whose products a workgroup sums in one chain of additions (0: all of them)
    int rev;            // windows in falling order (the dear ones first)
    int fold;           // DG - 1: a wave's second offset (and fourth) counts from the other end of the groups; otherwise 0
};
constexpr int kDwBandThreads = 256;
__host__ __device__ constexpr int dw_band_block_bytes(int NL) { return 32 * 16 * NL; }     // one 32-block of eight rows
inline size_t dw_band_stage_bytes(int NL, int RGN, int S32, int ndw) { return (size_t)RGN * (size_t)(2 * S32 + ndw - 1) * dw_band_block_bytes(NL); }
// One wave's diagonal image: 63 diagonals x 32 columns, pitch 36 (lane q writes diagonal c - q, so a pitch P puts the lanes
// P - 1 floats apart: an even P spreads them over the banks; a lane's diagonal is eight 16-byte reads, sixteen lanes' on
// different banks).
constexpr int kDwBandDiagPitch = 36;
constexpr int kDwBandDiag = 63 * kDwBandDiagPitch;
inline size_t dw_band_lds_bytes(int NL, int RGN, int S32, int ndw, int ND)
{
    const size_t stage = dw_band_stage_bytes(NL, RGN, S32, ndw), ep = sizeof(float) * 4 * (size_t)(kDwBandDiag + 64 * ND);
    return stage > ep ? stage : ep;
}

// What a workgroup walks, as functions of the geometry: the kernel's, and those of a test on the host that follows its operand addresses.
struct DwBandWindow {
    int dlo, nd;        // first offset, offsets
    int spare;          // places in front that have no offset
};
__host__ __device__ __forceinline__ DwBandWindow dw_band_window(const DwBandGeom &g, int win, bool dealt)
{
    const int left = g.nd - win * (g.ndw - 1), nd = left < g.ndw ? left : g.ndw;
    return DwBandWindow{g.dmin + win * (g.ndw - 1), nd, dealt && g.fold && g.rev ? g.ndw - nd : 0};
}
// Blocks of a virtual row; blocks from the start of the first virtual row of a row to that of the last.
__host__ __device__ __forceinline__ int dw_band_row_blocks(const DwBandGeom &g) { return g.nseg == 1 ? (g.L + 31) >> 5 : g.Lv >> 5; }
__host__ __device__ __forceinline__ int dw_band_seg_blocks(const DwBandGeom &g) { return (g.nseg - 1) * dw_band_row_blocks(g); }
// The offsets of the ND places of a wave of group dg, relative to the window's first (outside 0 .. nd - 1: none).  Dealt: one of every DG,
// otherwise a range.
template <int ND, int DG, bool DEALT>
struct DwBandPlaces {
    static constexpr int STEP = DEALT ? DG : 1;
    int off0, swing;    // the i-th: off0 + STEP i, + swing in odd rounds
    __host__ __device__ __forceinline__ DwBandPlaces(const DwBandGeom &g, const DwBandWindow &w, int dg)
        : off0((DEALT ? dg : dg * ND) - w.spare), swing(DEALT ? (dg ^ g.fold) - dg : 0) {}
    __host__ __device__ __forceinline__ int operator()(int i) const { return off0 + STEP * i + ((i & 1) ? swing : 0); }
};
// A stage: group vg of 8 RGN virtual rows, dY blocks yb0 .. yb0 + S32 - 1, x blocks xlo .. xlo + nx - 1 (nx <= 0: no offset of the
// window meets a row in it).
struct DwBandStage {
    int st, vg, yb0, xlo, nx;
};
__host__ __device__ __forceinline__ void dw_band_set_stage(const DwBandGeom &g, int dlo, DwBandStage &s)
{
    s.vg = g.nstep == 1 ? s.st : g.step_magic ? (int)(((unsigned long long)(unsigned)s.st * g.step_magic) >> 32) : s.st / g.nstep;
    s.yb0 = (s.st - s.vg * g.nstep) * g.S32;
    s.xlo = s.yb0 + dlo;
    int xhi = s.xlo + g.S32 + g.ndw - 2;
    // (a block of zeros on both sides of the row: the other half of a pair that is half inside.  Blocks count from the start
    // of each virtual row, of which the last starts seg_blocks into its row)
    const int first = -1 - dw_band_seg_blocks(g), NB32 = (g.L + 31) >> 5;
    s.xlo = s.xlo > first ? s.xlo : first;
    xhi = xhi < NB32 ? xhi : NB32;
    s.nx = xhi - s.xlo + 1;
}
// The block pairs p (dY blocks yb0 + 2 p, + 1) of an offset that meet the row from some virtual row: plo .. phi.
__host__ __device__ __forceinline__ void dw_band_pairs(const DwBandGeom &g, const DwBandWindow &w, int yb0, int offset, int &plo, int &phi)
{
    const int d = w.dlo + offset, NB32 = (g.L + 31) >> 5;
    const int lo = (-yb0 - d - dw_band_seg_blocks(g)) >> 1;              // ceil((-yb0 - d - 1 - seg_blocks) / 2)
    const int rest = dw_band_row_blocks(g) - yb0 + 1, last = (rest < g.S32 ? rest : g.S32) / 2 - 1, hi = (NB32 - 1 - yb0 - d) >> 1;
    plo = lo > 0 ? lo : 0;
    phi = last < hi ? last : hi;
    if ((unsigned)offset >= (unsigned)w.nd) {                            // (in front or behind: active_runs)
        plo = kNoWorkLo;
        phi = kNoWorkHi;
    }
}

// Four consecutive elements at any element-aligned address.
struct __attribute__((packed, aligned(4))) Raw4F { unsigned v[4]; };
struct __attribute__((packed, aligned(2))) Raw4H { unsigned v[2]; };
__device__ __forceinline__ Raw4F load_raw4(const float *p) { return *reinterpret_cast<const Raw4F *>(p); }
__device__ __forceinline__ Raw4H load_raw4(const bf16_t *p) { return *reinterpret_cast<const Raw4H *>(p); }
// moved down by sh elements (0 .. 3), zeros behind; all zeros when zero
__device__ __forceinline__ void fix_raw4(Raw4F &r, int sh, bool zero)
{
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        const bool on = (sh & step) != 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.v[i] = on ? (i + step < 4 ? r.v[i + step] : 0u) : r.v[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = zero ? 0u : r.v[i];
}
__device__ __forceinline__ void fix_raw4(Raw4H &r, int sh, bool zero)
{
    if (sh & 2) { r.v[0] = r.v[1]; r.v[1] = 0u; }
    const int bits = 16 * (sh & 1);
    r.v[0] = __builtin_amdgcn_alignbit(r.v[1], r.v[0], bits);
    r.v[1] = r.v[1] >> bits;
    r.v[0] = zero ? 0u : r.v[0];
    r.v[1] = zero ? 0u : r.v[1];
}
__device__ __forceinline__ void zero_raw4(Raw4F &r, bool zero)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = zero ? 0u : r.v[i];
}
__device__ __forceinline__ void zero_raw4(Raw4H &r, bool zero)
{
    r.v[0] = zero ? 0u : r.v[0];
    r.v[1] = zero ? 0u : r.v[1];
}
// Eight rows x four positions -> per position the eight rows as limbs.
__device__ __forceinline__ void transpose_limbs(const Raw4F (&r)[8], int pos, uintx4 (&out)[3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned p[3];
        split_pair(__uint_as_float(r[2 * i].v[pos]), __uint_as_float(r[2 * i + 1].v[pos]), p);
        out[0][i] = p[0]; out[1][i] = p[1]; out[2][i] = p[2];
    }
}
__device__ __forceinline__ void transpose_limbs(const Raw4H (&r)[8], int pos, uintx4 (&out)[1])
{
    const unsigned sel = (pos & 1) ? 0x07060302u : 0x05040100u;      // the upper or the lower halves of a pair of rows
#pragma unroll
    for (int i = 0; i < 4; ++i) out[0][i] = __builtin_amdgcn_perm(r[2 * i + 1].v[pos >> 1], r[2 * i].v[pos >> 1], sel);
}

// CHAINS (fp32): the products of g.chain stages at a time are summed by themselves (plan_dw_band).  A form of its own: with the registers of its second
// start the others take 3 % longer (B2048 C128 L256 K256 150 / 154 us).
template <typename E, int ND, int DG, bool SPLIT, bool CHAINS = false>
__global__ __launch_bounds__(kDwBandThreads, 2) void dw_band_kernel(const E *__restrict__ x, const E *__restrict__ dy,
                                                                     float *__restrict__ part, E *__restrict__ dw_out,
                                                                     const DwBandGeom g, int slices)
{
    constexpr int NL = Limbs<E>::N;
    constexpr int PB = 16 * NL, BB = dw_band_block_bytes(NL);            // bytes of a position, of a block
    extern __shared__ __align__(16) unsigned char dwb_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x, sl = (int)blockIdx.y;
    const int win = g.rev ? g.nwin - 1 - (int)blockIdx.z : (int)blockIdx.z;
    const int NB32 = (g.L + 31) >> 5;
    constexpr int KS = 4 / DG;
    const int dg = wave & (DG - 1), ks = wave / DG;
    const int RGN = 1 << g.rg_log;
    // This wave's offsets: one of every DG.  (A range of them left the waves with unequal work where the pairs fall with the distance
    // from lag 0; causal filters: the rounds over the groups alternate in direction, so that each wave has near and far ones, and
    // start from the near end, so that the places of the last window that have no offset are far ones.  bf16, both tensors by every
    // thread: a range, whose pairs are nearly the same ones: B3220 C123 L144 K144 75 us, 79 dealt)
    constexpr bool DEALT = SPLIT || NL == 3;
    const DwBandWindow w = dw_band_window(g, win, DEALT);
    const int dlo = w.dlo, nd_here = w.nd;
    const DwBandPlaces<ND, DG, DEALT> place(g, w, dg);
    constexpr int STEP = DwBandPlaces<ND, DG, DEALT>::STEP;
    const size_t CL = (size_t)g.C * (size_t)g.L;
    const E *x_c = x + (size_t)c * (size_t)g.L, *dy_c = dy + (size_t)c * (size_t)g.L;
    const int VR = g.B * g.nseg;

    floatx16 acc[ND], mid[NL == 3 ? ND : 1], low[NL == 3 ? ND : 1];

    typedef DwBandStage Stage;
    // the next stage in which some offset of the window meets a row (nx <= 0: none does); st >= stages: the end
    auto advance = [&](Stage &s) {
        do {
            s.st += (int)gridDim.y;
            if (s.st >= g.stages) return;
            dw_band_set_stage(g, dlo, s);
        } while (s.nx <= 0);
    };
    // Staging: 64 WPR threads bring one group of eight rows, one item of four positions of x and one of dY each (the plan
    // keeps a stage that small); the rows of an item are wave-uniform, so a load is a scalar base and a lane offset.  The
    // items of a stage are loaded while the stage before it is multiplied.
    const int WPR = 4 >> g.rg_log;
    const int rg_ld = wave >> (2 - g.rg_log), it_ld = tid & ((SPLIT ? 32 : 64) * WPR - 1);
    // SPLIT: where a stage is a whole row and either tensor is half a group's items (rows of up to 256 positions in two groups, 512 in one), one
    // half of the waves brings x and the other dY, one item per thread, and the blocks of zeros beside the row are written once.  (Both
    // tensors by every thread: two items for the first of two waves, and an eighth of one, zeros, for the second)
    const bool y_wave = SPLIT && (wave & (WPR - 1)) >= WPR / 2;
    decltype(load_raw4(x)) raw_x[8], raw_y[SPLIT ? 1 : 8];
    auto row_of = [&](int vr, int &off) -> size_t {                      // element offset of (virtual) row vr; off: its first position
        vr = min(vr, VR - 1);
        const int b = g.nseg == 1 ? vr : (int)(((unsigned)vr * g.seg_magic) >> 16);
        off = g.nseg == 1 ? 0 : (vr - b * g.nseg) * g.Lv;
        return (size_t)b * CL;
    };
    auto load_items = [&](const Stage &s) {
        const int it = band_hide(it_ld), vr0 = ((s.vg << g.rg_log) + rg_ld) * 8;
        // (positions outside the row are loaded from inside it and put right below)
        if constexpr (SPLIT) {
            const E *p = (y_wave ? dy_c : x_c) + min(4 * it, g.L - 4);
            if (vr0 + 8 <= VR) {
                p += (size_t)vr0 * CL;
#pragma unroll
                for (int r = 0; r < 8; ++r) raw_x[r] = load_raw4(p + r * CL);
            } else {
#pragma unroll
                for (int r = 0; r < 8; ++r) raw_x[r] = load_raw4(p + (size_t)min(vr0 + r, VR - 1) * CL);
            }
        } else {
            int ux = 32 * s.xlo + min(4 * it, 32 * s.nx - 4), uy = 32 * s.yb0 + min(4 * it, 32 * g.S32 - 4);
            if (g.nseg == 1) {
                ux = max(0, min(ux, g.L - 4));
                uy = min(uy, g.L - 4);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const size_t row = (size_t)min(vr0 + r, VR - 1) * CL;
                    raw_x[r] = load_raw4(x_c + row + ux);
                    raw_y[r] = load_raw4(dy_c + row + uy);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    int off;
                    const size_t row = row_of(vr0 + r, off);
                    raw_x[r] = load_raw4(x_c + row + max(0, min(ux + off, g.L - 4)));
                    raw_y[r] = load_raw4(dy_c + row + max(0, min(uy + off, g.L - 4)));
                }
            }
        }
    };
    // Rows past the batch, positions outside the row, positions of dY that belong to the next virtual row: zeros; a group of
    // four that ends behind its row was loaded from further left.  u: the first position of the item in its virtual row.
    auto put_right = [&](decltype(raw_x) &raw, int vr0, int u, int end) __attribute__((always_inline)) {
        if (SPLIT || g.nseg == 1) {
            const bool zero = u < 0 || u >= g.L;
            const int over = u + 4 - g.L;
            if ((g.L & 3) != 0 && __builtin_amdgcn_ballot_w64(!zero && over > 0) != 0) {
#pragma unroll
                for (int r = 0; r < 8; ++r) fix_raw4(raw[r], !zero && over > 0 ? over : 0, zero);
            } else if (__builtin_amdgcn_ballot_w64(zero) != 0) {
#pragma unroll
                for (int r = 0; r < 8; ++r) zero_raw4(raw[r], zero);
            }
            if (vr0 + 8 > VR) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (vr0 + r >= VR) zero_raw4(raw[r], true);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                int off;
                (void)row_of(vr0 + r, off);
                const int v = u + off;
                const bool zero = vr0 + r >= VR || v < 0 || v >= g.L || u >= end;
                if (__builtin_amdgcn_ballot_w64(zero || v + 4 > g.L) != 0)
                    fix_raw4(raw[r], v + 4 > g.L && v < g.L ? (v + 4 - g.L) & 3 : 0, zero);
            }
        }
    };
    auto store_items = [&](const Stage &s) {
        const int it = band_hide(it_ld), vr0 = ((s.vg << g.rg_log) + rg_ld) * 8;
        unsigned char *base = dwb_smem + rg_ld * ((s.nx + g.S32) * BB);
        auto put = [&](const decltype(raw_x) &raw, unsigned char *dst) __attribute__((always_inline)) {
            const int q = (4 * it) & 31, sw = (q >> 3) & 3;
            dst += ((4 * it) & ~31) * PB;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uintx4 limbs[NL];
                transpose_limbs(raw, j, limbs);
#pragma unroll
                for (int l = 0; l < NL; ++l) *reinterpret_cast<uintx4 *>(dst + ((q + j) ^ sw) * PB + 16 * l) = limbs[l];
            }
        };
        if constexpr (SPLIT) {
            // (the window of x may start behind the row's first block or end before its last)
            put_right(raw_x, vr0, 4 * it, 1 << 30);
            const int blk = it >> 3, to = y_wave ? s.nx + blk : blk - s.xlo;
            if (blk < (y_wave ? g.S32 : NB32) && to >= 0 && (y_wave || to < s.nx)) put(raw_x, base + (to - blk) * BB);
        } else {
            put_right(raw_x, vr0, 32 * s.xlo + 4 * it, 1 << 30);
            put_right(raw_y, vr0, 32 * s.yb0 + 4 * it, g.Lv);
            if (4 * it < 32 * s.nx) put(raw_x, base);
            if (4 * it < 32 * g.S32) put(raw_y, base + s.nx * BB);
        }
    };

    Stage cur;
    cur.st = sl - (int)gridDim.y;
    cur.nx = 0;
    advance(cur);
    for (bool first = true;; first = false) {
#pragma unroll
        for (int i = 0; i < ND; ++i)
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                acc[i][k] = 0.f;
                if constexpr (NL == 3) mid[i][k] = low[i][k] = 0.f;
            }
        int left = CHAINS ? g.chain : 1;
        if (cur.st < g.stages) {
            load_items(cur);
            if constexpr (SPLIT) {
                // (x blocks -1 and NB32; one stage is like the other)
                for (int rg = 0; rg < RGN; ++rg)
                    for (int i = tid; i < 2 * (BB / 16); i += kDwBandThreads) {
                        const int at = (i < BB / 16 ? -1 : NB32) - cur.xlo;
                        if (at >= 0 && at < cur.nx)
                            *reinterpret_cast<uintx4 *>(dwb_smem + rg * ((cur.nx + g.S32) * BB) + at * BB + 16 * (i < BB / 16 ? i : i - BB / 16)) =
                                uintx4{0u, 0u, 0u, 0u};
                    }
            }
        }
        while (cur.st < g.stages && left > 0) {
            const int yb0 = cur.yb0, xlo = cur.xlo, nx = cur.nx;
            const int rg_bytes = (nx + g.S32) * BB;                          // one group of eight rows: x blocks, dY blocks
            __syncthreads();                                                 // everyone is done with the stage before
            store_items(cur);
            __syncthreads();
            advance(cur);
            if constexpr (CHAINS) --left;
            if (cur.st < g.stages && left > 0) load_items(cur);

            int plo[ND], phi[ND];                                            // block pairs p (blocks yb0 + 2 p, + 1) per offset
#pragma unroll
            for (int i = 0; i < ND; ++i) {
                dw_band_pairs(g, w, yb0, place(i), plo[i], phi[i]);
                // (hidden: the compiler would make a second set of loops for waves with an empty place, bf16 119 -> 157
                // registers)
                asm volatile("" : "+s"(plo[i]), "+s"(phi[i]));
            }
            const int ln = band_hide(lane), q = ln & 31, kg = ln >> 5;
            const int lane_off = (q ^ ((q >> 3) & 3)) * PB + kg * BB;
            // pairs p = pa .. pb (those of this wave) for the offsets I0 .. I0 + N - 1
            auto run = [&](auto i0c, auto nc, const unsigned char *xw, const unsigned char *yw, int pa, int pb) {
                constexpr int I0 = decltype(i0c)::value, N = decltype(nc)::value;
                pa += (ks - pa) & (KS - 1);
                if (pa > pb) return;
                const unsigned char *yp = yw + 2 * pa * BB, *xp[2];                      // (of the even and the odd rounds over the groups)
                xp[0] = xw + (2 * pa + place.off0) * BB;
                xp[1] = xp[0] + place.swing * BB;
                uintx4 y[2][NL], xv[2][NL];
                auto read_y = [&](uintx4 (&to)[NL]) {
#pragma unroll
                    for (int l = 0; l < NL; ++l) to[l] = *reinterpret_cast<const uintx4 *>(yp + 16 * l);
                };
                auto read_x = [&](uintx4 (&to)[NL], int i) {
#pragma unroll
                    for (int l = 0; l < NL; ++l) to[l] = *reinterpret_cast<const uintx4 *>(xp[DEALT ? (I0 + i) & 1 : 0] + (I0 + i) * STEP * BB + 16 * l);
                };
                auto multiply = [&](int i, const uintx4 (&a)[NL], const uintx4 (&b)[NL]) {
                    if constexpr (NL == 3) {
                        low[i] = mfma32x32x16(a[2], b[0], low[i]);
                        acc[i] = mfma32x32x16(a[0], b[0], acc[i]);
                        mid[i] = mfma32x32x16(a[1], b[0], mid[i]);
                        low[i] = mfma32x32x16(a[0], b[2], low[i]);
                        mid[i] = mfma32x32x16(a[0], b[1], mid[i]);
                        low[i] = mfma32x32x16(a[1], b[1], low[i]);
                    } else {
                        acc[i] = mfma32x32x16(a[0], b[0], acc[i]);
                    }
                };
                read_y(y[0]);
                read_x(xv[0], 0);
#pragma unroll 1
                for (int p = pa; p <= pb;) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (u == 0 || p <= pb) {
                            const int by = p + KS <= pb ? 2 * KS * BB : 0;   // (past the last pair: the same addresses again)
#pragma unroll
                            for (int i = 0; i < N; ++i) {
                                const int k = u * N + i;
                                if (i + 1 < N) {
                                    read_x(xv[(k + 1) & 1], i + 1);
                                } else {
                                    yp += by;
                                    xp[0] += by;
                                    if constexpr (DEALT) xp[1] += by;
                                    read_y(y[1 - u]);
                                    read_x(xv[(k + 1) & 1], 0);
                                }
                                multiply(I0 + i, xv[k & 1], y[u]);
                            }
                            p += KS;
                        }
                    }
                }
            };
            for (int rg = 0; rg < RGN; ++rg) {
                const unsigned char *xw = dwb_smem + rg * rg_bytes + lane_off + (yb0 + dlo - xlo) * BB;
                const unsigned char *yw = dwb_smem + rg * rg_bytes + lane_off + nx * BB;
                active_runs(plo, phi, [&](auto ac, auto nc, int pa, int pb) { run(ac, nc, xw, yw, pa, pb); });
            }
        }

        // ---- diagonal sums: every wave those of its offsets (e = q' - q + 31 of each), then the two offsets a tap belongs to and the
        // waves' parts of each added in order
        __syncthreads();
        float *img = reinterpret_cast<float *>(dwb_smem) + wave * kDwBandDiag;
        float *taps = reinterpret_cast<float *>(dwb_smem) + 4 * kDwBandDiag;
        constexpr int TW = 64 * ND;
        float *tap = taps + wave * TW;
        // (the cells a diagonal has no entry in stay zero: a sum is 32 columns whatever its length.  A loop over the columns it
        // has, one LDS round trip after the other, took 5 us of a call: B1 C257 L480 K105 bf16 11.7 us)
        // (hidden: what follows from them would stay in registers from one chain to the next)
        const int ld = CHAINS ? band_hide(lane) : lane;
        const float zero = CHAINS ? __int_as_float(band_hide(0)) : 0.f;
        for (int i = ld; i < kDwBandDiag / 4; i += 64) *reinterpret_cast<floatx4 *>(img + 4 * i) = floatx4{zero, zero, zero, zero};
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            // lane (column q, half kg) holds rows q' = 8 (k / 4) + 4 kg + k % 4 in element k
            const int q = ld & 31, kg = ld >> 5;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                float v = acc[i][k];
                if constexpr (NL == 3) v = limb_sum(v, mid[i][k], low[i][k]);
                img[(8 * (k >> 2) + 4 * kg + (k & 3) - q + 31) * kDwBandDiagPitch + q] = v;
            }
            wave_lds_fence();
            if (ld < 63) {
                floatx4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const floatx4 *>(img + ld * kDwBandDiagPitch + 4 * j);
                floatx4 sum = v[0];
#pragma unroll
                for (int j = 1; j < 8; ++j) sum += v[j];
                tap[64 * i + ld] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
            }
            wave_lds_fence();
        }
        __syncthreads();
        // tap T = 0 .. 32 nd_here + 30 of the window is j = 32 dlo - 31 + pad + T; it owns lags j - pad in [32 dlo, 32 dhi), the first
        // and the last window whatever lies beyond (taps no offset reaches are zero)
        const int jw = 32 * dlo - 31 + g.pad;
        const int j_lo = win == 0 ? 0 : 32 * dlo + g.pad, j_hi = win + 1 == g.nwin ? g.K : min(g.K, 32 * (dlo + nd_here - 1) + g.pad);
        float *dst = part + ((size_t)sl * (size_t)g.C + (size_t)c) * (size_t)g.K;
        const bool more = CHAINS && cur.st < g.stages;
        for (int j = max(0, j_lo) + (CHAINS ? band_hide(tid) : tid); j < j_hi; j += kDwBandThreads) {
            const int t = j - jw;
            float sum = 0.f;
            if (t >= 0 && t < 32 * nd_here + 31) {
                // diagonal t % 32 of offset t / 32 and t % 32 + 32 of the one before it; waves (dg, 0), (dg, 1) .. have an offset
#pragma unroll
                for (int h = 1; h >= 0; --h) {
                    const int o = (t >> 5) - h, e = (t & 31) + 32 * h;
                    if (o >= 0 && o < nd_here && e < 63) {
                        const int at_o = o + w.spare, i = DEALT ? at_o / DG : at_o % ND, r = DEALT ? at_o & (DG - 1) : at_o / ND;
                        const int at = (DEALT && (i & 1) ? r ^ g.fold : r) * TW + 64 * i + e;
                        for (int k = 0; k < KS; ++k) sum += taps[k * DG * TW + at];
                    }
                }
            }
            if (dw_out) {                                                // (one slice: one chain)
                st_elem(dw_out + (size_t)c * (size_t)g.K + (size_t)j, sum);
            } else {
                if (CHAINS && !first) sum += dst[j];                    // (what this thread wrote of the chain before)
                dst[j] = sum;
                // (slices beyond those of this launch are part of the workspace's layout: zeros)
                if (!more)
                    for (int o = sl + (int)gridDim.y; o < slices; o += (int)gridDim.y)
                        part[((size_t)o * (size_t)g.C + (size_t)c) * (size_t)g.K + (size_t)j] = 0.f;
            }
        }
        if (!more) break;
        __syncthreads();                                                     // (of tap sums, before the next chain's blocks take their place)
    }
}

}  // namespace dwconv
