// Launchers of the weight-gradient stage-1 kernels (templates on the storage type; instantiated by
// dwconv_launch_dw_f32.hip and dwconv_launch_dw_bf16.hip).
#pragma once
#include "dwconv_host.hip.h"
#include "dwconv_dw_bf16.hip.h"
#include "dwconv_valu.hip.h"

namespace dwhost {

template <typename T, int KCH>
void launch_dw_partial_valu(const void *x, const void *dy, float *part, const Shape &s, const DwPlan &p, hipStream_t st)
{
    if (p.valu_rows.on) {
        hipLaunchKernelGGL((dwconv::dw_partial_valu_kernel<T, kDwThreads, kDwTT, KCH, true>), dim3((unsigned)s.C, (unsigned)p.S),
                           dim3(kDwThreads), 0, st, static_cast<const T *>(x), static_cast<const T *>(dy), part, 1, s.C,
                           s.L, s.K, s.pad, p.valu_tiles_per_row, p.valu_items_per_slice, p.valu_rows.map);
        return;
    }
    hipLaunchKernelGGL((dwconv::dw_partial_valu_kernel<T, kDwThreads, kDwTT, KCH, false>), dim3((unsigned)s.C, (unsigned)p.S),
                       dim3(kDwThreads), 0, st, static_cast<const T *>(x), static_cast<const T *>(dy), part, s.B, s.C,
                       s.L, s.K, s.pad, p.valu_tiles_per_row, p.valu_items_per_slice, dwconv::RowsMap{0, 0, 0, 0, 0u, 0u});
}

// Rows of at most 128 positions, either storage type: sixteen rows per matrix tile.  dmin / nd: the block offsets inside a
// row (rows_batch_offsets); the kernel is compiled per number of 16-blocks of a row, not per number of offsets.
template <typename T, int W>
int launch_dw_rowbatch_w(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p, int dmin,
                         int nd, hipStream_t st)
{
    // rows of at most 128 positions, either storage type: sixteen rows per matrix tile
    auto launch_rb = [&](auto kernel, int nc) -> int {
        const size_t lds_rb = dwconv::rb_dw_lds_bytes(s.L, nd, W, nc);
        if (lds_rb > kMaxLdsBytes) return -1;
        if (lds_rb > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(s.C / nc), (unsigned)p.S), dim3(64 * W), lds_rb, st,
                           static_cast<const T *>(x), static_cast<const T *>(dy), part, static_cast<T *>(dw_out), s.B,
                           s.C, s.L, s.K, s.pad, dmin, nd, p.tiles_per_row);
        return launch_status();
    };
    // (the kernel is compiled per number of 16-blocks of a row, not per number of block offsets)
    const int m = (s.L + 15) / 16;
    // rows that end inside a granule: the variant with the partial-granule code, four-wave workgroups only (the plan
    // asks for no others there)
    auto rag_rb = [&](auto mc) -> int {
        constexpr int MM = decltype(mc)::value;
        if ((s.L % 4) != 0) {
            if constexpr (W == dwconv::kWavesPerBlock) return launch_rb(dwconv::dw_rowbatch_kernel<T, MM, W, 1, true>, 1);
            else return -1;
        }
        return launch_rb(dwconv::dw_rowbatch_kernel<T, MM, W, 1, false>, 1);
    };
    if constexpr (W == dwconv::kWavesPerBlock) {
        if (p.dw_nc == 2) {
            switch (m) {
            case 1: return launch_rb(dwconv::dw_rowbatch_kernel<T, 1, W, 2, false>, 2);
            case 2: return launch_rb(dwconv::dw_rowbatch_kernel<T, 2, W, 2, false>, 2);
            case 3: return launch_rb(dwconv::dw_rowbatch_kernel<T, 3, W, 2, false>, 2);
            default: return -1;
            }
        }
    }
    switch (m) {
    case 1: return rag_rb(std::integral_constant<int, 1>{});
    case 2: return rag_rb(std::integral_constant<int, 2>{});
    case 3: return rag_rb(std::integral_constant<int, 3>{});
    case 4: return rag_rb(std::integral_constant<int, 4>{});
    case 5: return rag_rb(std::integral_constant<int, 5>{});
    case 6: return rag_rb(std::integral_constant<int, 6>{});
    case 7: return rag_rb(std::integral_constant<int, 7>{});
    case 8: return rag_rb(std::integral_constant<int, 8>{});
    default: return -1;
    }
}

template <typename T>
int launch_dw_rowbatch(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p, hipStream_t st)
{
    int dmin, nd;
    rows_batch_offsets(s.L, s.K, s.pad, &dmin, &nd);
    switch (p.wpb) {
    case 4: return launch_dw_rowbatch_w<T, 4>(x, dy, part, dw_out, s, p, dmin, nd, st);
    case 5: return launch_dw_rowbatch_w<T, 5>(x, dy, part, dw_out, s, p, dmin, nd, st);
    case 8: return launch_dw_rowbatch_w<T, 8>(x, dy, part, dw_out, s, p, dmin, nd, st);
    case 16: return launch_dw_rowbatch_w<T, 16>(x, dy, part, dw_out, s, p, dmin, nd, st);
    default: return -1;
    }
}

// One stage-1 launch on the matrix cores.  dw_out != nullptr only for single-slice plans.
template <typename T, int ND, int W>
int launch_dw_partial_mfma_ndw(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                               int dmin, hipStream_t st)
{
    if constexpr (std::is_same<T, float>::value) {
        // fp32 rows go from memory straight into LDS
        constexpr size_t lds = dwconv::dw_direct_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (p.rows.on) {
            auto kernel = dwconv::dw_partial_direct_kernel<ND, W, true>;
            if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
            hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                               static_cast<const float *>(x), static_cast<const float *>(dy), part,
                               static_cast<float *>(dw_out), 1, s.C, s.L, s.K, s.pad, dmin, p.tiles_per_row, p.rows.map);
        } else {
            auto kernel = dwconv::dw_partial_direct_kernel<ND, W, false>;
            if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
            hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                               static_cast<const float *>(x), static_cast<const float *>(dy), part,
                               static_cast<float *>(dw_out), s.B, s.C, s.L, s.K, s.pad, dmin, p.tiles_per_row, p.rows.map);
        }
    } else if (bf16_odd_rows(s, x, dy)) {
        // bf16 rows that do not all start on a dword: the same kernels on rows shifted to the dword in which they start
        // (four waves whatever the plan says: workgroups of more are compiled for the aligned forms only).  Vector-ALU
        // kernel -> here: B32 C256 L4097 K64 159 -> 27 us, B4096 C128 L199 K48 618 -> 86 us, B50000 C128 L9 K9 359 -> 147 us
        if constexpr (W != dwconv::kWavesPerBlock) {
            return launch_dw_partial_mfma_ndw<T, ND, dwconv::kWavesPerBlock>(x, dy, part, dw_out, s, p, dmin, st);
        } else {
            constexpr size_t lds = dwconv::dw_bf16_lds_bytes(ND, W);
            static_assert(lds <= 64 * 1024, "LDS budget");
            auto go = [&](auto kernel, int B, int segs) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                                   static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(dy), part,
                                   static_cast<bf16_t *>(dw_out), B, s.C, s.L, s.K, s.pad, dmin, segs, p.rows.map, aligned_to(x, 4) ? 0 : 1);
            };
            if (p.rows.on) go(dwconv::dw_partial_bf16_kernel<ND, W, true, true>, 1, p.tiles_per_row);
            // (a shifted row may reach one position into a segment more)
            else go(dwconv::dw_partial_bf16_kernel<ND, W, false, true>, s.B, (s.L + 1 + dwconv::kSegLen - 1) / dwconv::kSegLen);
        }
    } else if (p.rows.on && (s.L % 2) == 0 && (p.rows.map.P % 8) == 0 && aligned_to(x, 4) && aligned_to(dy, 4)) {
        // bf16 short rows of even length (they start on a dword): the virtual row of a channel on the bf16 matrix instruction,
        // raw rows straight into LDS (B4096 C128 L200 K48: 247 -> 88 us against the widening kernel below)
        auto kernel = dwconv::dw_partial_bf16_kernel<ND, W, true>;
        constexpr size_t lds = dwconv::dw_bf16_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                           static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(dy), part,
                           static_cast<bf16_t *>(dw_out), 1, s.C, s.L, s.K, s.pad, dmin, p.tiles_per_row, p.rows.map, 0);
    } else if (p.rows.on) {
        // bf16 short rows (longer than 64 positions): the virtual row of a channel, widened to fp32 through registers
        auto kernel = dwconv::dw_partial_mfma_kernel<T, ND, W, true>;
        constexpr size_t lds = dwconv::dw_mfma_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st, static_cast<const T *>(x),
                           static_cast<const T *>(dy), part, static_cast<T *>(dw_out), 1, s.C, s.L, s.K, s.pad, dmin,
                           p.tiles_per_row, p.rows.map);
    } else if ((s.L % 2) == 0 && aligned_to(x, 4) && aligned_to(dy, 4)) {
        // bf16 rows that start on a dword: raw rows straight into LDS, bf16 matrix instruction
        auto kernel = dwconv::dw_partial_bf16_kernel<ND, W>;
        constexpr size_t lds = dwconv::dw_bf16_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st,
                           static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(dy), part,
                           static_cast<bf16_t *>(dw_out), s.B, s.C, s.L, s.K, s.pad, dmin, p.tiles_per_row, dwconv::RowsMap{0, 0, 0, 0, 0u, 0u}, 0);
    } else {
        auto kernel = dwconv::dw_partial_mfma_kernel<T, ND, W, false>;
        constexpr size_t lds = dwconv::dw_mfma_lds_bytes(ND, W);
        static_assert(lds <= kMaxLdsBytes, "LDS budget");
        if (lds > 64 * 1024 && !allow_large_lds(kernel)) return -1;
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.S), dim3(64 * W), lds, st, static_cast<const T *>(x),
                           static_cast<const T *>(dy), part, static_cast<T *>(dw_out), s.B, s.C, s.L, s.K, s.pad, dmin,
                           p.tiles_per_row, p.rows.map);
    }
    return launch_status();
}

template <typename T, int ND>
int launch_dw_partial_mfma_nd(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                              int dmin, hipStream_t st)
{
    switch (p.wpb) {
    case 4: return launch_dw_partial_mfma_ndw<T, ND, 4>(x, dy, part, dw_out, s, p, dmin, st);
    case 5: return launch_dw_partial_mfma_ndw<T, ND, 5>(x, dy, part, dw_out, s, p, dmin, st);
    case 8: return launch_dw_partial_mfma_ndw<T, ND, 8>(x, dy, part, dw_out, s, p, dmin, st);
    case 16: return launch_dw_partial_mfma_ndw<T, ND, 16>(x, dy, part, dw_out, s, p, dmin, st);
    default: return -1;
    }
}

// Returns -1 when the shape or the pointers do not fit the matrix-core kernel.
template <typename T>
int launch_dw_partial_mfma(const void *x, const void *dy, float *part, void *dw_out, const Shape &s, const DwPlan &p,
                           hipStream_t st)
{
    const int dmin = toeplitz_dmin(s.pad), dmax = toeplitz_dmax(s.K, s.pad);
    const int nd = dmax - dmin + 1;
    // (rows of at most 128 positions: the sixteen-row kernel needs rows that start on a dword, nothing more)
    if (p.rows.batch) return (aligned_to(x, 4) && aligned_to(dy, 4)) ? launch_dw_rowbatch<T>(x, dy, part, dw_out, s, p, st) : -1;
    if (s.K < kMfmaMinK || nd < 2 || nd > mfma_max_nd_dw(s) || s.L > kMfmaMaxL) return -1;
    // whole granules of four elements; otherwise only the kernels that load rows straight into LDS apply (see ragged_rows_ok)
    const bool granular = (s.L % 4) == 0 && aligned_to(x, 4 * sizeof(T)) && aligned_to(dy, 4 * sizeof(T));
    // (bf16 virtual rows of even length: launch_dw_partial_mfma_ndw takes them on the kernel that loads raw rows into LDS)
    // (fp32 virtual rows of any length, up to six offsets: the kernel that loads rows straight into LDS)
    const bool rows_direct_bf16 = sizeof(T) == 2 && p.rows.on && (s.L % 2) == 0 && (p.rows.map.P % 8) == 0;
    const bool rows_direct_f32 = sizeof(T) == 4 && p.rows.on && nd <= kMfmaMaxND;
    const bool rows_direct = (rows_direct_bf16 || rows_direct_f32) && aligned_to(x, 4) && aligned_to(dy, 4);
    if (bf16_odd_rows(s, x, dy)) {
        // (rows of one to three positions are all gap as virtual rows: B61773 C32 L1 K2 21 us on the vector-ALU kernel, 32 us here;
        // with one tap there are no gaps: B30000 C64 L1 K1 2457 -> 27 us)
        if (nd > kMfmaMaxND || !bf16_odd_rows_ok(s, x, dy, p.rows) || (p.rows.on && s.L < 4 && s.K > 1)) return -1;
    } else if (!granular && !rows_direct && (!ragged_rows_ok(s, nd) || p.rows.on || !aligned_to(x, 4) || !aligned_to(dy, 4))) return -1;
    if constexpr (std::is_same<T, float>::value) {
        if (nd > kMfmaMaxND) return launch_dw_partial_wide_f32(x, dy, part, dw_out, s, p, dmin, nd, st);
    } else {
        if (nd > kMfmaMaxND) return launch_dw_partial_wide_bf16(x, dy, part, dw_out, s, p, dmin, nd, st);
    }
    switch (nd) {
    case 2: return launch_dw_partial_mfma_nd<T, 2>(x, dy, part, dw_out, s, p, dmin, st);
    case 3: return launch_dw_partial_mfma_nd<T, 3>(x, dy, part, dw_out, s, p, dmin, st);
    case 4: return launch_dw_partial_mfma_nd<T, 4>(x, dy, part, dw_out, s, p, dmin, st);
    case 5: return launch_dw_partial_mfma_nd<T, 5>(x, dy, part, dw_out, s, p, dmin, st);
    case 6: return launch_dw_partial_mfma_nd<T, 6>(x, dy, part, dw_out, s, p, dmin, st);
    default: return -1;
    }
}

template <typename T>
int launch_dw_partial(const void *x, const void *dy, float *part, void *dw_out, int *slices, const Shape &s,
                      const DwPlan &p, hipStream_t st)
{
    // dw_out: where a single-slice matrix-core launch may put the gradient itself (nullptr: always write part, all p.S slices);
    // *slices tells the caller how many slices of part hold the sums (0: dw_out holds the gradient).
    if constexpr (std::is_same<T, float>::value) {
        if (p.window) {
            // (a caller that takes the gradient needs no more slices than the launch uses)
            const int used = dw_out ? p.wp.S : p.S;
            void *to = p.wp.S == 1 ? dw_out : nullptr;
            if (slices) *slices = to ? 0 : used;
            return launch_dw_window_f32(x, dy, part, to, p.wp, used, st);
        }
    }
    void *direct = (p.single && p.S == 1) ? dw_out : nullptr;
    int rc = p.band ? -1 : launch_dw_partial_mfma<T>(x, dy, part, direct, s, p, st);
    if (slices) *slices = direct ? 0 : p.S;
    if (rc < 0 && p.band_fits) {
        // (a caller that takes the gradient needs no more slices than the launch uses)
        const int mine = p.toep ? p.tp.S : p.bp.S, used = dw_out ? mine : p.S;
        direct = mine == 1 ? dw_out : nullptr;
        if (slices) *slices = direct ? 0 : used;
        if (p.toep) {
            if constexpr (std::is_same<T, float>::value) rc = launch_dw_toep_f32(x, dy, part, direct, p.tp, used, st);
            else rc = launch_dw_toep_bf16(x, dy, part, direct, p.tp, used, st);
        } else {
            if constexpr (std::is_same<T, float>::value) rc = launch_dw_band_f32(x, dy, part, direct, p.bp, used, st);
            else rc = launch_dw_band_bf16(x, dy, part, direct, p.bp, used, st);
        }
    }
    if (rc >= 0) return rc;
    if (slices) *slices = p.S;
    switch (p.kernel) {
    case DW_VALU_K8: launch_dw_partial_valu<T, 8>(x, dy, part, s, p, st); break;
    case DW_VALU_K32: launch_dw_partial_valu<T, 32>(x, dy, part, s, p, st); break;
    case DW_VALU_K64: launch_dw_partial_valu<T, 64>(x, dy, part, s, p, st); break;
    case DW_VALU_K256: launch_dw_partial_valu<T, 256>(x, dy, part, s, p, st); break;
    }
    return launch_status();
}

}  // namespace dwhost
