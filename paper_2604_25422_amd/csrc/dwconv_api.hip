// C ABI of the gfx950 depthwise 1-D convolution library: argument validation,
// kernel selection and launch.  Declarations and argument contracts are in
// include/dwconv.h; the operator is the one of the paper's Sec. IV-A.
#include "dwconv_host.hip.h"
#include "dwconv_valu.hip.h"

// Partial sums of the weight gradient for callers that cannot hand over a workspace (dwconv_bwd_weight_noalloc):
// one array per GPU, living in the code object's data segment until the process ends.  In host code the name below
// is only a handle for hipGetSymbolAddress; kernels get the device address that call returns.
constexpr size_t kScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace dwhost {

constexpr int kVersion = 101;   // 0.1.1

// Device address of `scratch` on the current device (looked up once per device and kept).
int scratch_pointer(void **out)
{
    static std::mutex mu;
    static std::map<int, void *> per_device;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return DWCONV_ERR_LAUNCH;
    }
    std::lock_guard<std::mutex> lock(mu);
    auto it = per_device.find(dev);
    if (it == per_device.end()) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return DWCONV_ERR_LAUNCH;
        }
        it = per_device.emplace(dev, ptr).first;
    }
    *out = it->second;
    return DWCONV_OK;
}

int check_shape(int B, int C, int L, int K, int pad, int dtype)
{
    if (B < 1 || C < 1 || L < 1 || K < 1) return DWCONV_ERR_SHAPE;
    const unsigned long long n = (unsigned long long)B * (unsigned long long)C;
    if (n > (1ull << 40) || n * (unsigned long long)L > (1ull << 40)) return DWCONV_ERR_SHAPE;
    if ((unsigned long long)C * (unsigned long long)K > (1ull << 40)) return DWCONV_ERR_SHAPE;
    if (pad < 0 || pad > K - 1) return DWCONV_ERR_PAD;
    if (dtype != DWCONV_F32 && dtype != DWCONV_BF16) return DWCONV_ERR_DTYPE;
    return DWCONV_OK;
}

RowsPlan plan_rows(const Shape &s)
{
    RowsPlan r;
    r.on = false; r.batch = false; r.tall = false; r.units = 0; r.nvs = 0;
    r.map = dwconv::RowsMap{0, 0, 0, 0, 0u, 0u};
    const int nd = toeplitz_dmax(s.K, s.pad) - toeplitz_dmin(s.pad) + 1;
    if (s.K < kMfmaMinK || nd < 2) return r;
    const long long es = (long long)elem_size(s.dtype);
    // Sixteen rows per tile (rows of at most 128 positions, either storage type): byte offsets inside a unit stay below
    // the out-of-row marker; the offsets that count are those inside the row (rows_batch_offsets: a filter as long as
    // the row, or longer, is no different from a short one).  Rows that are not whole granules of four must start on a
    // dword (any fp32 row, bf16 rows of even length) and have their kernels for up to six offsets only.
    bool batch = s.L <= dwconv::kRbMaxL && (long long)dwconv::kRbRows * s.C * s.L * es < (1ll << 30);
    if (batch) {
        int bd, bn;
        rows_batch_offsets(s.L, s.K, s.pad, &bd, &bn);
        if ((s.L % 4) != 0) batch = bn <= kMfmaMaxND && (s.dtype == DWCONV_F32 || (s.L % 2) == 0);
        else batch = bn <= kRbMaxND;
    }
    // Virtual rows (whole granules; up to six offsets, fp32 sixteen): where a 1024-position segment of a row would be more than a
    // quarter padding, and positions stay 32-bit.
    const long long halo = s.pad > s.K - 1 - s.pad ? s.pad : s.K - 1 - s.pad;
    // (pitch: whole granules of four; bf16 of eight - rows AND gaps - so that the kernels that load 16 bytes per lane apply;
    // a bf16 row of even length that is not a multiple of eight ends inside its last granule, see rows_granule8_byte_offset)
    const long long gr = s.dtype == DWCONV_F32 ? 4 : 8;
    const long long P = (s.L + gr - 1) / gr * gr + (halo + gr - 1) / gr * gr;
    const long long padded = ((long long)s.L + dwconv::kSegLen - 1) / dwconv::kSegLen * dwconv::kSegLen;
    const long long elems = (long long)s.B * s.C * s.L;
    // (seven to sixteen offsets, fp32: only while the gaps stay below half a row - with a filter as long as the row half of
    // the virtual row is gap, and the tall-row kernels below do better: B3200 C128 L160 K160 fwd 354 us here)
    // (rows that end inside a 16-byte granule - fp32 lengths that are not multiples of four, bf16 lengths that are not
    // multiples of eight: the kernels that load rows straight into LDS, up to six offsets; bf16 rows of odd length start
    // on a dword every other time and are shifted to one, see rows_odd_start: P >= L + 1 + halo leaves room for it)
    const bool vrows = (s.dtype == DWCONV_BF16 || (s.L % 4) == 0 || nd <= kMfmaMaxND) &&
                       (nd <= kMfmaMaxND || (s.dtype == DWCONV_F32 && (s.L % 4) == 0 && nd <= kMfmaMaxNDDw && 2 * P <= 3 * (long long)s.L)) &&
                       4 * padded > 5 * P && elems * es <= (1ll << 30) &&
                       (long long)s.B * P * P < (1ll << 32) && (long long)s.B * P < (1ll << 31);
    if (vrows) {
        r.on = true;
        r.nvs = (int)(((long long)s.B * P + dwconv::kSegLen - 1) / dwconv::kSegLen);
        r.map.P = (int)P; r.map.L = s.L; r.map.CL = s.C * s.L; r.map.Lv = (int)(s.B * P);
        r.map.M = (unsigned)((1ull << 32) / (unsigned long long)P) + 1u;
        r.map.bytes = (unsigned)(elems * es);
    }
    // bf16 rows of 64 to 128 positions in whole 16-byte granules: the virtual-row kernels bring the raw bf16 rows straight
    // into LDS and have a fused backward kernel, which the sixteen-row kernels have up to 48 positions (B8192 C128 L64 K48: 45 us
    // forward, 107 us backward; L60 on the sixteen-row kernels 84 and 170; L48 there 36 and 62)
    if (batch && vrows && s.dtype == DWCONV_BF16 && s.L >= 64 && (s.L % 2) == 0 && (P % 8) == 0) batch = false;
    if (batch) {
        r.on = true; r.batch = true;
        r.units = (s.B + dwconv::kRbRows - 1) / dwconv::kRbRows;
    }
    // Rows of nine to thirty-two blocks with more block offsets than the virtual-row kernels take (filters of the order
    // of the row length), or a batch whose virtual row they cannot address: the band kernels, and weight-gradient slices that
    // follow from units of four rows.  (bf16 up to twenty blocks: longer rows have the slices of long filters.)
    const int m = (s.L + 15) / 16;
    // (rows that are not whole granules: they must start on a dword - any fp32 length, bf16 even lengths)
    const bool tall_rag = (s.L % 4) != 0 && nd > kMfmaMaxND && (s.dtype == DWCONV_F32 || (s.L % 2) == 0);      // (up to six offsets:
                                                                     // the kernels that load rows straight into LDS)
    if (!batch && !vrows && ((s.L % 4) == 0 || tall_rag) && s.L > dwconv::kRbMaxL &&
        m <= (s.dtype == DWCONV_F32 ? 32 : 20) &&
        (long long)dwconv::kRbRows * s.C * s.L * es < (1ll << 30)) {
        r.tall = true;
        r.units = (s.B + dwconv::kRbRows - 1) / dwconv::kRbRows;
    }
    return r;
}

int corr_entry(const void *in, const void *f, void *out, int B, int C, int L, int K, int pad, int dtype, void *stream,
               bool is_dx)
{
    if (!in || !f || !out) return DWCONV_ERR_NULL;
    const int rc = check_shape(B, C, L, K, pad, dtype);
    if (rc != DWCONV_OK) return rc;
    const size_t es = elem_size(dtype);
    if (!aligned_to(in, es) || !aligned_to(f, es) || !aligned_to(out, es)) return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad, dtype};
    const int pad_eff = is_dx ? (K - 1 - pad) : pad;
    const int reverse = is_dx ? 1 : 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dtype == DWCONV_F32) return launch_corr_f32(in, f, out, s, pad_eff, reverse, st);
    return launch_corr_bf16(in, f, out, s, pad_eff, reverse, st);
}

// ------------------------------------------------------------------ weight gradient
// Which filters of more than six block offsets go to dw_band_kernel (us, the register-resident kernels -> dw_band_kernel; K
// causal).  Up to sixteen offsets the register-resident kernels walk 1024-position segments, a wave each, and are the faster
// ones while there are few of them or the batch fills the groups of eight rows that dw_band_kernel contracts badly; it has more
// to do once per workgroup (a stage of eight rows, diagonal sums of 32 x 32 products).
//   fp32, ordinary rows: with 64 segments per channel from eleven offsets (B32 C256 L4096: K = 160 98 -> 91, 226 137 -> 126; B40 C16
//     L2048 K160 14.1 -> 12.1), with 16 of them and 4096 in all from fourteen (B16 C768 L1024: K = 160 39.6 / 44.0, 200 50.5 -> 47.2;
//     B49 C4 L816 K200, 196 in all: 11.3 / 16.0), never below 1024 in all (B250 C2 L883 K144 9.9 / 14.4) or with less than three quarters of
//     the groups of eight (B9 C64 L9016 K160 26 / 37; B13 C31 L9568 24 / 24)
//   fp32, virtual rows: from eleven offsets (B5 C768 L272: K = 118 10.2 / 15.2, 160 15.9 -> 13.6; B256 C128 L400: K = 118 44 / 48,
//     135 55 -> 50) and 1024 segments (B373 C5 L352 K160, 765: 10.3 / 11.8)
//   bf16, rows of whole 16-byte granules that fill their 1024-position segments to three quarters: from twelve offsets with 1024
//     segments, 32 of them per channel or 16 and 4096 in all (B16 C768 L1024 K176 17.4 -> 15.9, B32 C256 L4096 K200 38 -> 33; B8 C256
//     L1024 K176 6.4 / 7.1, B1 C128 L16000 K179 8.7 / 12.9)
//   bf16, other rows of whole granules: from seven offsets with 17 segments per channel (B20 C64 L400 K100 8.7 -> 8.5, B500 C16 L256
//     K100 18.5 -> 9.4; B16 C256 L600 K100 6.9 / 7.8), from eleven with more than 1024 in all (B5 C256 L640 K160 5.8 -> 5.5;
//     B1 C257 L1464 K160 6.2 / 7.6)
//   all with more than sixteen offsets (fp32 B32 C256 L4096 K300 185 -> 140, 4096 1142 -> 782), all bf16 rows of other lengths (L4097
//     K100 309 -> 39), all rows of up to 512 positions that are neither virtual nor below 129 (L256 K256 fp32 182 -> 100)
//   rows of at most 128 positions: bf16 above 112 (L128 K128 59 -> 40, L96 K96 42 / 53; fp32 L128 K128 66 / 92)
static bool dw_takes_band(const Shape &s, const RowsPlan &rp)
{
    const int nd = toeplitz_dmax(s.K, s.pad) - toeplitz_dmin(s.pad) + 1;
    if (rp.tall) return true;
    if (nd <= kMfmaMaxND) return false;
    if (rp.batch) {
        int bd, bn;
        rows_batch_offsets(s.L, s.K, s.pad, &bd, &bn);
        return s.dtype == DWCONV_BF16 && bn > kMfmaMaxND && s.L > 112;
    }
    if (rp.on) return nd >= 11 && (long long)rp.nvs * s.C >= 1024;
    if (nd > kMfmaMaxNDDw || s.L <= 512 * (s.dtype == DWCONV_F32) || (s.dtype == DWCONV_BF16 && (s.L % 8) != 0)) return true;
    const long long segs_per_row = ((long long)s.L + dwconv::kSegLen - 1) / dwconv::kSegLen, segs = s.B * segs_per_row;
    const bool many = segs >= 16 && segs * s.C >= 4096;
    if (s.dtype == DWCONV_F32)
        return segs * s.C >= 1024 && nd >= (segs >= 64 ? 11 : many ? 14 : kMfmaMaxNDDw + 1) && 4ll * s.B >= 3 * ((s.B + 7ll) / 8 * 8);
    if (4ll * s.L >= 3 * segs_per_row * dwconv::kSegLen) return nd >= 12 && segs * s.C >= 1024 && (segs >= 32 || many);
    return segs > 16 || (nd >= 11 && segs * s.C > 1024);
}

// Which of dw_band_kernel's filters go to dw_toep_kernel: by the products of 32 x 32 x 16 that either would form.  dw_toep_kernel
// stages less per product but its tiles are 1024 lags wide: lags beyond the filter, and positions that only the far lags of a tile
// have lost, are multiplied all the same.  dw_band_kernel has groups of eight rows to fill (fewer batch entries: virtual rows, whose
// stages are small), and a stage of its own for every twelve (bf16 sixteen) offsets of 32.  us, dw_band_kernel -> dw_toep_kernel,
// with the ratio of the products:
//   fp32, five batch entries and more: B8 C256 L8192 K8192 (1.12) 792 -> 644, B17 C736 L889 K889 (1.06) 173 -> 130, B161 C46 L1024
//     K1024 (1.25) 104 -> 86, B7 C96 L896 K896 (1.30) 17.6 -> 16.5, B16 C83 L3328 K3328 (1.32) 109 -> 104, B98 C45 L2496 K2496 (1.36) 209 / 232,
//     B284 C103 L768 K768 (1.70) 195 / 308
//   bf16: B8 C256 L8192 K8192 (1.12) 193 -> 131, B12 C355 L1832 K1832 (1.19) 51 -> 40, B25 C328 L1020 K1020 (1.49) 38 -> 29, B25 C32 L1163
//     K1163 (1.52) 17 -> 11; a stage is one row, and a short one has few products: B214 C64 L896 K896 (1.47) 34 / 46, B38 C45 L813 K813
//     (1.55) 11 / 13
//   fewer batch entries, fp32: B4 C672 L1080 K1080 (1.84) 62 -> 54, B1 C365 L5675 K5675 (1.19) 210 -> 73, B1 C396 L1104 K1104 (2.15) 34 -> 10, B2 C608 L416
//     K416 (2.64) 22 -> 12, B4 C71 L912 K912 (1.92) 11.1 / 13.8; bf16: B3 C320 L3968 K3968 (0.92) 80 -> 28, B2 C384 L1150 K1150 (1.62) 16.5 -> 8.3
static bool dw_takes_toep(const Shape &s, const DwPlan &p)
{
    const double lo = std::min(s.pad, s.L - 1), hi = std::min(s.K - 1 - s.pad, s.L - 1);           // lags -lo .. hi
    const double pairs = (lo + hi + 1) * s.L - (lo * (lo + 1) + hi * (hi + 1)) / 2;
    const int nseg = p.bp.g.nseg;
    const double groups = (double)(((long long)s.B * nseg + 7) / 8);
    // (two blocks at a time: half a product lost per offset of 32 at the end of the row, and the offsets at both ends of the filter)
    const double band = groups * (8.0 * pairs / nseg / (1024 * 16) + 0.75 * ((lo + hi + 1) / 32 + 2));
    // Calls that leave compute units idle (at most two workgroups for each) are a chain on a workgroup: here of its batch entries one after the
    // other, 1.2 us each and what they multiply, there of groups of eight at once.  Both as measured over 420 calls of up to 45 us
    // (error 7 % here, 9 % there): fp32 B4 C77 L1023 K1023 11.0 / 19.1, B5 C27 L937 K937 11.8 / 18.0, B2 C69 L946 K946 9.7 / 11.6, but B1 C71 L843 K256
    // 8.8 / 6.8; bf16 B6 C48 L753 K753 7.2 / 11.7, B4 C30 L2496 K717 9.9 / 15.2, B5 C220 L818 K818 8.4 / 10.3, but B5 C100 L1342 K1342 15.8 / 12.3.
    // (Not with fewer than sixteen channels: no layer's, and it is with them that the tests reach the edges of dw_toep_kernel.)
    const double wgs = (double)s.C * p.tp.g.npiece * p.tp.S;
    if (s.C >= 16 && wgs <= 2 * kComputeUnits) {
        const bool f32 = s.dtype == DWCONV_F32;
        const double rows = p.tp.g.rows, chunks = (s.L + p.tp.g.F - 1) / p.tp.g.F, products = s.L / 16.0 + 2;
        const double over = wgs > kComputeUnits ? wgs / kComputeUnits - 1 : 0.0;            // (second workgroups of compute units)
        const double here = f32 ? 3.2 + (p.tp.S > 1 ? 1.6 : 0.0) + rows * (1.2 * chunks + (0.051 + 0.028 * over) * products)
                                : 3.0 + (p.tp.S > 1 ? 1.9 : 0.0) + rows * (0.84 * chunks + (0.014 + 0.006 * over) * products);
        const double stages = (p.bp.g.stages + p.bp.S - 1) / p.bp.S, rounds = (double)s.C * p.bp.g.nwin * p.bp.S / (2 * kComputeUnits);
        const double pairs = stages * p.bp.g.S32 * p.bp.ND * std::max(1.0, rounds);
        const double there = f32 ? 6.6 + (p.bp.S > 1 ? 0.9 : 0.0) + 0.4 * (stages - 1) + 0.056 * pairs + 5.9 * rounds
                                 : 6.1 + (p.bp.S > 1 ? 1.2 : 0.0) + 2.6 * (stages - 1) + 0.011 * pairs + 3.4 * rounds;
        if (here > there) return false;
    }
    const double most = s.dtype == DWCONV_F32 ? (nseg > 2 ? 2.65 : nseg > 1 ? 1.85 : 1.33) : (nseg > 1 ? 2.6 : s.L >= 1000 ? 1.54 : 1.42);
    return p.tp.work <= most * band;
}

// Which fp32 filters of seven and more block offsets go to dw_window_kernel instead of the register-resident kernels of the fp32 instruction (those of
// the band and Toeplitz kernels are asked first): where the products of these, with the padding of rows to regions of 256 positions or of virtual
// rows to their pitch, take longer than its own estimate.  (Both in us at the clock under load; 1.2 and 1.3 are what either takes beyond its
// products.)  us, inputs from memory, before -> here: taken B1407 C162 L256 K123 pad 122 227 -> 133, B3038 C32 L666 K127 pad 63 265 -> 165, B59 C250
// L1333 K86 pad 85 64 -> 47, B1918 C32 L1248 K111 pad 110 191 -> 166, B32 C256 L4096 K128 causal 96 -> 77.  Close above the line (the estimates within a tenth,
// seven offsets on ordinary rows) the mean of 60 calls is 1.10, the best B157 C224 L2384 K84 pad 0 227 -> 172, the worst B209 C256 L999 K88 pad 87 107 ->
// 127; of 61 others above it 1.33, the worst 1.04; of 269 below it 1.03, so that it could lie lower, but not by much (B18 C766 L3761 K120
// 139 / 152, B2670 C32 L880 K77 168 / 185, B18 C276 L1079 K86 29 / 41).
static bool dw_takes_window(const Shape &s, const DwPlan &p, int nd)
{
    const double positions = (double)s.B * s.C * (p.rows.on ? p.rows.map.P : (s.L + 255) / 256 * 256);
    return 1.3 * p.wp.cycles / 2000.0 < 1.2 * positions / 1024.0 * 16 * nd * 32 / (4 * kComputeUnits) / 2100.0;
}

// Slices of the workspace for the filters of dw_band_kernel.  Callers keep workspaces and read slices by these numbers
// (dwconv_bwd_weight_slices), so they stay what they have been although the kernel mostly uses fewer (DwBandPlan::S, chosen from
// the channels, windows and stages there are): a call that takes the gradient sums only those used, dwconv_bwd_weight_partial
// writes zeros to the rest.  About two workgroups per compute unit over channels, windows of offsets and slices, a slice being
// two rows at least; two slices at least and a workspace of at most 64 MiB beyond that.  0: the slices that the segments of the
// row give (times one per started sixteen offsets).
static int dw_band_slices(const Shape &s, const RowsPlan &rp, int nd)
{
    const int nb = (s.L + 15) / 16;
    int dmin = toeplitz_dmin(s.pad), dmax = toeplitz_dmax(s.K, s.pad);
    if (dmin < -(nb - 1)) dmin = -(nb - 1);
    if (dmax > nb - 1) dmax = nb - 1;
    if (rp.tall) {
        // rows of nine to thirty-two blocks: windows of fifteen offsets, each with slices of sixteen rows at least
        const long long nwin = (dmax - dmin + 1 + 14) / 15, units = (s.B + 3) / 4;
        const long long su = (2LL * kComputeUnits + (long long)s.C * nwin - 1) / ((long long)s.C * nwin);
        return (int)(std::min(su, (units + 3) / 4) * nwin);
    }
    if (nd <= mfma_max_nd_dw(s)) return 0;
    if ((s.L % 4) == 0 && s.L <= 8192 && s.K <= 8192) {
        const long long wgs = (dmax - dmin + 1 + 287) / 288;
        long long rs = std::min((2LL * kComputeUnits + s.C * wgs - 1) / (s.C * wgs), std::min(128LL, (s.B + 1LL) / 2));
        while (rs > 1 && 2 * rs * (long long)s.C * s.K * (long long)sizeof(float) > (64ll << 20)) --rs;
        const long long bper = ((s.B + rs - 1) / rs + 1) / 2 * 2;
        return (int)(2 * ((s.B + bper - 1) / bper));
    }
    if ((s.L % (s.dtype == DWCONV_F32 ? 4 : 8)) == 0 && s.L >= kRaggedMinL) {
        const long long items = (long long)s.B * ((s.L + kDwTT - 1) / kDwTT);
        const long long sp = std::min((kTargetWaves / 4 + s.C - 1) / s.C, (items + 3) / 4);
        return (int)(2 * std::max(sp, 1LL));
    }
    return 0;
}

// Depends on the shape only, so stage 1, stage 2 and the workspace query always agree.
DwPlan plan_dw(const Shape &s)
{
    DwPlan p;
    p.kernel = s.K <= 8 ? DW_VALU_K8 : s.K <= 32 ? DW_VALU_K32 : s.K <= 64 ? DW_VALU_K64 : DW_VALU_K256;
    p.rows = plan_rows(s);
    long long tiles = p.rows.on ? p.rows.nvs : ((long long)s.L + kDwTT - 1) / kDwTT;
    if (p.rows.batch) {                                          // units of the weight-gradient kernel, one channel per block
        const int ru = dwconv::rb_dw_unit_rows(s.L, 1);
        tiles = (s.B + ru - 1) / ru;
    }
    long long items = p.rows.on ? tiles : (long long)s.B * tiles;                        // per channel
    int nd = toeplitz_dmax(s.K, s.pad) - toeplitz_dmin(s.pad) + 1;
    if (p.rows.batch) {                                          // (the offsets inside a row are all that count there)
        int bd;
        rows_batch_offsets(s.L, s.K, s.pad, &bd, &nd);
    }
    const bool mfma_shape = p.rows.batch || (s.K >= kMfmaMinK && nd >= 2 && nd <= mfma_max_nd_dw(s) &&
                                             ((s.L % 4) == 0 || ragged_rows_ok(s, nd)) && s.L <= kMfmaMaxL);
    // When the channels alone fill the chip evenly (C = 1, 2 or 3 per compute unit), one block of 16, 8 or 5
    // waves takes a whole channel: no slices, no second stage.
    p.wpb = dwconv::kWavesPerBlock;
    p.single = false;
    p.dw_nc = 1;
    if (mfma_shape && nd <= (s.dtype == DWCONV_F32 ? kMfmaMaxNDWide : kMfmaMaxND) && s.C % kComputeUnits == 0 &&
        s.C / kComputeUnits <= 3 && !(p.rows.batch && (s.L % 4) != 0) && !(p.rows.on && !p.rows.batch && nd > kMfmaMaxND)) {
        int wpb = 16 / (s.C / kComputeUnits);
        // short filters leave the matrix pipe idle, and what then counts is how many bytes the chip has in flight:
        // two rows of 4 KiB per wave are enough with 8 to 12 waves per compute unit (B64 C512 L2048 K7: 82 us against
        // 87 us with 16 waves; bf16 B128 C768 L1024 K32: 59.6 against 60.8 us)
        if (nd <= 3 && s.C / kComputeUnits >= 2) wpb = 4;
        // (sixteen-row units of rows longer than 48 positions need more LDS than sixteen waves have)
        const bool fits = (!p.rows.batch || dwconv::rb_dw_lds_bytes(s.L, nd, wpb, 1) <= kMaxLdsBytes) &&
                          (nd <= kMfmaMaxND || dwconv::dw_direct_lds_bytes(nd, wpb) <= kMaxLdsBytes);
        if (items >= 2 * wpb && fits) { p.wpb = wpb; p.single = true; }
    }
    // Small problems (at most four segments or units per wave of one four-wave workgroup per channel) are bound by
    // launch latency: one workgroup per channel and no second launch there too.
    if (mfma_shape && !p.single && items <= 4 * dwconv::kWavesPerBlock) p.single = true;
    long long groups = s.C;                                      // blocks along the channel axis
    if (p.rows.batch && !p.single && s.C % 2 == 0 && (s.L * (int)elem_size(s.dtype)) % 128 != 0 && s.L <= 48 && (s.L % 4) == 0) {
        // two neighbouring channels per block: rows that are not whole cache lines become pieces that are;
        // a unit is then eight rows of both channels
        p.dw_nc = 2;
        groups = s.C / 2;
        tiles = (s.B + dwconv::kRbRows / 2 - 1) / (dwconv::kRbRows / 2);
        items = tiles;
    }
    long long want = (kTargetWaves / p.wpb + groups - 1) / groups;   // blocks per channel (group)
    if (p.single) want = 1;
    if (want < 1) want = 1;
    if (want > 65535) want = 65535;
    long long spw = (items + want * p.wpb - 1) / (want * p.wpb);
    if (spw < 1) spw = 1;
    const long long per = spw * p.wpb;
    p.segs_per_wave = (int)spw;
    p.items_per_slice = (int)per;
    p.S = (int)((items + per - 1) / per);
    p.band = dw_takes_band(s, p.rows);
    if (p.band && !p.rows.on) {
        const int slices = dw_band_slices(s, p.rows, nd);
        if (slices > 0) { p.S = slices; p.single = false; }
        else if (mfma_shape && nd > kMfmaMaxNDDw) { p.S *= (nd + kMfmaMaxNDDw - 1) / kMfmaMaxNDDw; p.single = false; }
    }
    p.band_fits = (nd > kMfmaMaxND || p.rows.tall) && plan_dw_band(s, p.S, &p.bp);
    p.band = p.band && p.band_fits;
    p.toep = p.band && plan_dw_toep(s, p.S, &p.tp) && dw_takes_toep(s, p);
    p.window = !p.band && !p.rows.batch && nd > kMfmaMaxND && plan_dw_window(s, p.S, &p.wp) && dw_takes_window(s, p, nd);
    // the fused backward kernel of these shapes works on one channel per block: its own slice count
    p.S_fused = p.S;
    if (p.rows.batch && s.L <= dwconv::kRbBwdMaxL) {
        // one wave per (channel, slice), sixteen-row units: about kTargetWaves waves
        long long wantf = kTargetWaves / s.C;
        if (wantf < 1) wantf = 1;
        if (wantf > p.rows.units) wantf = p.rows.units;
        if (wantf > 65535) wantf = 65535;
        const long long upw = (p.rows.units + wantf - 1) / wantf;
        p.S_fused = (int)((p.rows.units + upw - 1) / upw);
    }
    p.tiles_per_row = (int)tiles;
    {
        const long long real_tiles = ((long long)s.L + kDwTT - 1) / kDwTT;
        const long long real_items = (long long)s.B * real_tiles;
        p.valu_tiles_per_row = (int)real_tiles;
        p.valu_items_per_slice = (int)((real_items + p.S - 1) / p.S);
    }
    // the generic kernel on short rows: its items are the tiles of the virtual row of the channel
    p.valu_rows = plan_valu_rows(s);
    if (p.valu_rows.on) {
        p.valu_tiles_per_row = (int)p.valu_rows.tiles;
        p.valu_items_per_slice = (int)((p.valu_rows.tiles + p.S - 1) / p.S);
    }
    return p;
}

size_t dw_workspace_bytes(const Shape &s, const DwPlan &p)
{
    const size_t bytes = (size_t)(p.S > p.S_fused ? p.S : p.S_fused) * (size_t)s.C * (size_t)s.K * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int check_dw_shape(int B, int C, int L, int K, int pad, int dtype)
{
    const int rc = check_shape(B, C, L, K, pad, dtype);
    if (rc != DWCONV_OK) return rc;
    // the slice bookkeeping of stage 1 is 32-bit
    const long long tiles = ((long long)L + kDwTT - 1) / kDwTT;
    if ((long long)B * tiles > 0x3fffffffLL || C > 0x7fffffff / 2) return DWCONV_ERR_SHAPE;
    return DWCONV_OK;
}

template <typename T>
int launch_dw_finalize(const float *part, void *dw, const Shape &s, const DwPlan &p, hipStream_t st)
{
    const size_t CK = (size_t)s.C * (size_t)s.K;
    if (p.S >= 32 && CK <= 16 * 2048) {
        // many slices of few coefficients: the slices in parallel (same order of the sum)
        const size_t nb = (CK + 15) / 16;
        hipLaunchKernelGGL((dwconv::dw_finalize_many_kernel<T>), dim3((unsigned)nb), dim3(256), 0, st, part,
                           static_cast<T *>(dw), p.S, CK);
        return launch_status();
    }
    const size_t blocks = (CK + 255) / 256;
    if (blocks > 0x7fffffffull) return DWCONV_ERR_SHAPE;
    hipLaunchKernelGGL((dwconv::dw_finalize_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, st, part,
                       static_cast<T *>(dw), p.S, CK);
    return launch_status();
}

int check_workspace(const void *ws, size_t ws_bytes, const Shape &s, const DwPlan &p)
{
    if (!ws || !aligned_to(ws, 16) || ws_bytes < dw_workspace_bytes(s, p)) return DWCONV_ERR_WORKSPACE;
    return DWCONV_OK;
}

}  // namespace dwhost

using namespace dwhost;

extern "C" {

int dwconv_fwd(const void *x, const void *w, void *y, int B, int C, int L, int K, int pad_left, int dtype, void *stream)
{
    return corr_entry(x, w, y, B, C, L, K, pad_left, dtype, stream, false);
}

int dwconv_bwd_input(const void *dy, const void *w, void *dx, int B, int C, int L, int K, int pad_left, int dtype,
                     void *stream)
{
    return corr_entry(dy, w, dx, B, C, L, K, pad_left, dtype, stream, true);
}

int dwconv_bwd_weight_partial(const void *x, const void *dy, void *workspace, size_t workspace_bytes, int B, int C,
                              int L, int K, int pad_left, int dtype, void *stream)
{
    if (!x || !dy) return DWCONV_ERR_NULL;
    int rc = check_dw_shape(B, C, L, K, pad_left, dtype);
    if (rc != DWCONV_OK) return rc;
    const size_t es = elem_size(dtype);
    if (!aligned_to(x, es) || !aligned_to(dy, es)) return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    rc = check_workspace(workspace, workspace_bytes, s, p);
    if (rc != DWCONV_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *part = static_cast<float *>(workspace);
    if (dtype == DWCONV_F32) return launch_dw_partial_f32(x, dy, part, nullptr, nullptr, s, p, st);
    return launch_dw_partial_bf16(x, dy, part, nullptr, nullptr, s, p, st);
}

int dwconv_bwd_weight_finalize(const void *workspace, size_t workspace_bytes, void *dw, int B, int C, int L, int K,
                               int pad_left, int dtype, void *stream)
{
    if (!dw) return DWCONV_ERR_NULL;
    int rc = check_dw_shape(B, C, L, K, pad_left, dtype);
    if (rc != DWCONV_OK) return rc;
    if (!aligned_to(dw, elem_size(dtype))) return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    rc = check_workspace(workspace, workspace_bytes, s, p);
    if (rc != DWCONV_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const float *part = static_cast<const float *>(workspace);
    if (dtype == DWCONV_F32) return launch_dw_finalize<float>(part, dw, s, p, st);
    return launch_dw_finalize<bf16_t>(part, dw, s, p, st);
}

int dwconv_bwd_weight(const void *x, const void *dy, void *dw, void *workspace, size_t workspace_bytes, int B, int C,
                      int L, int K, int pad_left, int dtype, void *stream)
{
    if (!x || !dy || !dw) return DWCONV_ERR_NULL;
    int rc = check_dw_shape(B, C, L, K, pad_left, dtype);
    if (rc != DWCONV_OK) return rc;
    const size_t es = elem_size(dtype);
    if (!aligned_to(x, es) || !aligned_to(dy, es) || !aligned_to(dw, es)) return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    rc = check_workspace(workspace, workspace_bytes, s, p);
    if (rc != DWCONV_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *part = static_cast<float *>(workspace);
    DwPlan pf = p;
    rc = (dtype == DWCONV_F32) ? launch_dw_partial_f32(x, dy, part, dw, &pf.S, s, p, st)
                               : launch_dw_partial_bf16(x, dy, part, dw, &pf.S, s, p, st);
    if (rc != DWCONV_OK || pf.S == 0) return rc;
    if (dtype == DWCONV_F32) return launch_dw_finalize<float>(part, dw, s, pf, st);
    return launch_dw_finalize<bf16_t>(part, dw, s, pf, st);
}

int dwconv_bwd_weight_noalloc(const void *x, const void *dy, void *dw, int B, int C, int L, int K, int pad_left,
                              int dtype, void *stream)
{
    if (!x || !dy || !dw) return DWCONV_ERR_NULL;
    int rc = check_dw_shape(B, C, L, K, pad_left, dtype);
    if (rc != DWCONV_OK) return rc;
    const size_t es = elem_size(dtype);
    if (!aligned_to(x, es) || !aligned_to(dy, es) || !aligned_to(dw, es)) return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad_left, dtype};
    if (dw_workspace_bytes(s, plan_dw(s)) > kScratchBytes) return DWCONV_ERR_SCRATCH;
    void *ptr = nullptr;
    rc = scratch_pointer(&ptr);
    if (rc != DWCONV_OK) return rc;
    return dwconv_bwd_weight(x, dy, dw, ptr, kScratchBytes, B, C, L, K, pad_left, dtype, stream);
}

size_t dwconv_noalloc_scratch_bytes(void) { return kScratchBytes; }

int dwconv_bwd(const void *dy, const void *x, const void *w, void *dx, void *dw, void *workspace,
               size_t workspace_bytes, int B, int C, int L, int K, int pad_left, int dtype, void *stream)
{
    if (!dy || !x || !w || !dx || !dw) return DWCONV_ERR_NULL;
    int rc = check_dw_shape(B, C, L, K, pad_left, dtype);
    if (rc != DWCONV_OK) return rc;
    const size_t es = elem_size(dtype);
    if (!aligned_to(dy, es) || !aligned_to(x, es) || !aligned_to(w, es) || !aligned_to(dx, es) || !aligned_to(dw, es))
        return DWCONV_ERR_ALIGN;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    rc = check_workspace(workspace, workspace_bytes, s, p);
    if (rc != DWCONV_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *part = static_cast<float *>(workspace);
    bool wrote_dw = false;
    DwPlan pf = p;
    pf.S = p.S_fused;                                             // slices the fused kernel wrote
    rc = dtype == DWCONV_F32 ? launch_bwd_fused_f32(dy, x, w, dx, part, dw, &wrote_dw, s, p, st)
                             : launch_bwd_fused_bf16(dy, x, w, dx, part, dw, &wrote_dw, s, p, st);
    if (rc >= 0) {
        if (rc != DWCONV_OK || wrote_dw) return rc;
        if (dtype == DWCONV_F32) return launch_dw_finalize<float>(part, dw, s, pf, st);
        return launch_dw_finalize<bf16_t>(part, dw, s, pf, st);
    }
    // shapes and types the fused kernel does not take: the two gradients one after the other
    rc = dwconv_bwd_input(dy, w, dx, B, C, L, K, pad_left, dtype, stream);
    if (rc != DWCONV_OK) return rc;
    return dwconv_bwd_weight(x, dy, dw, workspace, workspace_bytes, B, C, L, K, pad_left, dtype, stream);
}

int dwconv_bwd_is_fused(int B, int C, int L, int K, int pad_left, int dtype)
{
    if (check_dw_shape(B, C, L, K, pad_left, dtype) != DWCONV_OK) return 0;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    const int nd = toeplitz_dmax(K, pad_left) - toeplitz_dmin(pad_left) + 1;
    // sixteen rows per tile, either storage type (its workgroups own four neighbouring channels: with fewer, most of
    // their waves would idle and the two separate kernels are faster - B416666 C1 L48 K33: 298 against 120 us)
    if (p.rows.batch) return (L <= dwconv::kRbBwdMaxL && C >= dwconv::kRbBwdWaves) ? 1 : 0;
    if (p.rows.tall) return 0;
    if (dtype == DWCONV_BF16 && p.rows.on && !p.rows.batch && ((L % 2) != 0 || (p.rows.map.P % 8) != 0)) return 0;
    const bool rows_fit = p.rows.on ? true      // (virtual rows; bf16: of even length, checked above)
                          : dtype == DWCONV_BF16 ? ((L % 8) == 0 || ((L % 2) == 0 && ((L % 4) != 0 ? ragged_rows_fused_ok(s, nd) : true)))
                                                 : ((L % 4) == 0 || ragged_rows_fused_ok(s, nd));
    return (K >= kMfmaMinK && nd >= 2 && nd <= kMfmaMaxND && rows_fit && L <= kMfmaMaxL) ? 1 : 0;
}

int dwconv_bwd_weight_single_pass(int B, int C, int L, int K, int pad_left, int dtype)
{
    if (check_dw_shape(B, C, L, K, pad_left, dtype) != DWCONV_OK) return 0;
    const Shape s{B, C, L, K, pad_left, dtype};
    const DwPlan p = plan_dw(s);
    return (p.single && p.S == 1) ? 1 : 0;
}

int dwconv_bwd_weight_slices(int B, int C, int L, int K, int pad_left, int dtype)
{
    if (check_dw_shape(B, C, L, K, pad_left, dtype) != DWCONV_OK) return 0;
    const Shape s{B, C, L, K, pad_left, dtype};
    return plan_dw(s).S;
}

size_t dwconv_bwd_weight_workspace_bytes(int B, int C, int L, int K, int pad_left, int dtype)
{
    if (check_dw_shape(B, C, L, K, pad_left, dtype) != DWCONV_OK) return 0;
    const Shape s{B, C, L, K, pad_left, dtype};
    return dw_workspace_bytes(s, plan_dw(s));
}

const char *dwconv_status_string(int status)
{
    switch (status) {
    case DWCONV_OK: return "ok";
    case DWCONV_ERR_NULL: return "a required pointer is NULL";
    case DWCONV_ERR_SHAPE: return "B, C, L and K must be >= 1 and B*C*L must fit 2^40 elements";
    case DWCONV_ERR_PAD: return "pad_left must lie in [0, K-1]";
    case DWCONV_ERR_DTYPE: return "dtype must be DWCONV_F32 or DWCONV_BF16";
    case DWCONV_ERR_WORKSPACE: return "workspace is NULL, smaller than dwconv_bwd_weight_workspace_bytes() or not 16-byte aligned";
    case DWCONV_ERR_ALIGN: return "a tensor pointer is not aligned to its element size";
    case DWCONV_ERR_LAUNCH: return "HIP reported an error at kernel launch";
    case DWCONV_ERR_SCRATCH: return "this shape needs more partial-sum space than the library's built-in scratch holds "
                                    "(dwconv_noalloc_scratch_bytes()): use dwconv_bwd_weight with a workspace";
    default: return "unknown status";
    }
}

int dwconv_version(void) { return kVersion; }

}  // extern "C"

