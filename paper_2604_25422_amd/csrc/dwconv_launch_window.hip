// Launcher of the forward / input-gradient kernel that keeps its inputs in registers (dwconv_window.hip.h).
#include "dwconv_window.hip.h"
#include "dwconv_host.hip.h"

namespace dwhost {

// False: the kernel does not apply, or does not pay.
bool plan_corr_window(const Shape &s, int pad_eff, int reverse, WindowPlan *p)
{
    dwconv::WindowGeom &g = p->g;
    // (byte offsets inside a unit stay below the out-of-row marker.  Calls of fewer than four million positions never fill the chip: below)
    const long long positions = (long long)s.B * s.C * s.L;
    if (s.dtype != DWCONV_F32 || s.L <= dwconv::kRbMaxL || 64ll * s.C * s.L >= (1ll << 30) || positions < (4ll << 20)) return false;
    g.B = s.B; g.C = s.C; g.L = s.L; g.K = s.K; g.pad = pad_eff; g.reverse = reverse;
    const int nch = (s.L + 31) / 32;
    // the q that hold taps and meet the row, the first one odd; chunks shifted against the pieces where that leaves fewer of them
    int NW = 100;
    for (int phi = 0; phi < 32; phi += 4) {
        int lo = (phi - pad_eff - 31 + 15) >> 4, hi = (int)((s.K + 14ll + phi - pad_eff) >> 4);
        lo = std::max(lo, -2 * nch);
        hi = std::min(hi, 2 * nch);
        if ((lo & 1) == 0) --lo;
        const int nw = (hi - lo + 2) / 2;
        if (nw < NW) { NW = nw; g.phi = phi; g.q0 = lo; g.qn = hi - lo + 1; }
    }
    if (NW > 9) return false;
    NW = std::max(NW, 4);
    p->NW = NW;
    const int w0 = (g.q0 + 1) >> 1, G = 2;
    // Pieces of a row, waves of a workgroup and units of a wave: the least of what a wave has to do in the rounds it takes (cycles of its
    // SIMD).  A step is 24 NW products and some 300 vector instructions, one that only brings chunks has the latencies and half of those; a
    // wave alone on its SIMD takes a third longer than its share of two.  These, 8000 for the start of a workgroup and 1.06 for one unit a wave are a
    // fit to some sixty calls; the last one is not the same everywhere (pieces of 1024, one unit, and of 512, two: B32 C256 L4096 K128 82 / 67 us,
    // but of 400 calls those with one unit gain as much over the kernels before as the others).
    const int per_cu = 4 * dwconv::kWinPerSimd;
    const double step = 384.0 * NW + 1000.0;
    double best = 0.0, crowded = 1.0;
    for (int np = 1; np <= 12 && np <= (s.L + 63) / 64; ++np) {
        const int P = ((s.L + np - 1) / np + 63) / 64 * 64, NP = (s.L + P - 1) / P;
        if (NP != np) continue;
        const long long cols = (long long)s.B * NP, units = (cols + 15) / 16;
        if (units * 16 * NP >= (1ll << 32)) return false;
        const int clo = NP > 1 ? w0 : 0;
        const int need = clo - w0 - NW - G + 2, s_first = std::min(0, need > 0 ? (need + G - 1) / G : -((-need) / G));
        const int ns = (P + 63) / 64;
        const double unit = ns * step - 1100.0 * s_first;
        for (int waves = 4; waves >= 2; waves -= 2) {
            const int lds = dwconv::win_lds_bytes(3, NW, waves);
            const long long slots = (long long)kComputeUnits * std::min(per_cu / waves, (int)(kMaxLdsBytes / lds));
            for (int rounds = 1; rounds <= 3; ++rounds) {
                const long long want = std::max(1ll, rounds * slots / s.C);
                const long long r = (units + waves * want - 1) / (waves * want), gy = (units + waves * r - 1) / (waves * r);
                const long long wgs = s.C * gy, full = (wgs + slots - 1) / slots;
                const double resident = (double)std::min(wgs, slots) * std::min((long long)waves, units) / (4.0 * kComputeUnits);
                const double cost = full * (r * unit * (r == 1 ? 1.06 : 1.0) * (0.6 + 0.7 * resident) + 8000.0);
                if (best == 0.0 || cost < best * 0.99) {
                    best = cost;
                    g.NP = NP; g.P = P; g.np_magic = NP > 1 ? (unsigned)((1ull << 32) / (unsigned)NP) + 1u : 0u;
                    g.units = (int)units; g.s_first = s_first; g.ns = ns;
                    g.clo = clo; g.chi = NP > 1 ? 1 << 28 : (s.L + g.phi + 31) / 32 - 1;
                    p->gy = (int)gy;
                    g.waves = waves;
                    const int on_cu = (int)((std::min(wgs, slots) + kComputeUnits - 1) / kComputeUnits) * (int)std::min((long long)waves, units);
                    crowded = (0.6 + 0.7 * ((on_cu + 3) / 4)) / (0.6 + 0.7 * resident);
                }
                if (r == 1) break;
            }
        }
    }
    // Where at least 0.6 of that is steps that a full chip could not do without: pieces of few columns, waves without a unit and the chunks in front
    // of a piece cost more than corr_band_kernel's barriers (us, the kernels before / here, inputs from memory: B2 C712 L4000 K208 24 / 31, B96 C352 L304
    // K230 35 / 45; further lines in corr_takes_window).
    p->cycles = best;
    const double need = positions / (1024.0 * 1024.0) * step / best;
    p->share = need / crowded;
    return need >= 0.60;
}

int launch_corr_window_f32(const void *in, const void *f, void *out, const Shape &s, WindowPlan p, hipStream_t st)
{
    p.g.lines = (s.L % 32) == 0 && aligned_to(out, 128);
    auto go = [&](auto kernel, int NW) -> int {
        hipLaunchKernelGGL(kernel, dim3((unsigned)s.C, (unsigned)p.gy), dim3(64u * (unsigned)p.g.waves), dwconv::win_lds_bytes(3, NW, p.g.waves), st,
                           static_cast<const float *>(in), static_cast<const float *>(f), static_cast<float *>(out), p.g);
        return launch_status();
    };
    switch (p.NW) {
    case 4: return go(dwconv::corr_window_kernel<4, 6>, 4);
    case 5: return go(dwconv::corr_window_kernel<5, 6>, 5);
    case 6: return go(dwconv::corr_window_kernel<6, 8>, 6);
    case 7: return go(dwconv::corr_window_kernel<7, 8>, 7);
    case 8:
        if (p.g.chi < 8) return go(dwconv::corr_window_kernel<8, 8>, 8);
        return go(dwconv::corr_window_kernel<8, 10>, 8);
    case 9:
        if (p.g.chi < 8) return go(dwconv::corr_window_kernel<9, 8>, 9);
        return go(dwconv::corr_window_kernel<9, 10>, 9);
    default: return DWCONV_ERR_LAUNCH;                                   // (never planned)
    }
}

}  // namespace dwhost
