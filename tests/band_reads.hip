// Follows the operand addresses of the kernels for long filters on the host, with the plans and the walk the kernels use themselves:
// every operand a wave reads from LDS must lie in what its stage has put there, and every product must be one of a place that has
// work, formed once.  Built and run by tests/test_band_reads_cpu.py; prints the first fault of a shape and returns 1.
#include "../paper_2604_25422_amd/csrc/dwconv_plan_band.hip"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

using namespace dwhost;

static int planned = 0;
static bool fault(const char *kernel, const Shape &s, const char *what, long long v, long long lo, long long hi)
{
    printf("%s %s B%d C%d L%d K%d pad%d: %s %lld, expected %lld .. %lld\n", kernel, s.dtype == DWCONV_F32 ? "f32" : "bf16", s.B, s.C, s.L, s.K,
           s.pad, what, v, lo, hi);
    return false;
}

// One window of dw_band_kernel, one stage of it: the blocks every wave reads.
template <int ND, int DG, bool DEALT>
static bool dw_band_stage(const Shape &s, const dwconv::DwBandGeom &g, const dwconv::DwBandWindow &w, const dwconv::DwBandStage &st)
{
    constexpr int KS = 4 / DG;
    std::vector<int> formed(w.nd, 0), due(w.nd, 0);
    bool ok = true;
    for (int wave = 0; wave < 4; ++wave) {
        const int dg = wave & (DG - 1), ks = wave / DG;
        const dwconv::DwBandPlaces<ND, DG, DEALT> place(g, w, dg);
        int plo[ND], phi[ND];
        for (int i = 0; i < ND; ++i) {
            dwconv::dw_band_pairs(g, w, st.yb0, place(i), plo[i], phi[i]);
            if (ks == 0 && (unsigned)place(i) < (unsigned)w.nd) due[place(i)] = std::max(0, phi[i] - plo[i] + 1);
        }
        dwconv::active_runs(plo, phi, [&](auto ac, auto nc, int pa, int pb) {
            constexpr int I0 = decltype(ac)::value, N = decltype(nc)::value;
            pa += (ks - pa) & (KS - 1);
            for (int p = pa; p <= pb && ok; p += KS)
                for (int i = I0; i < I0 + N && ok; ++i) {
                    const int o = place(i), xb = st.yb0 + w.dlo + o + 2 * p - st.xlo;
                    if (o < 0 || o >= w.nd) ok = fault("dw_band", s, "product of offset", o, 0, w.nd - 1);
                    else if (xb < 0 || xb + 1 >= st.nx) ok = fault("dw_band", s, "block of x", xb, 0, st.nx - 2);
                    else if (p < 0 || 2 * p + 1 >= g.S32) ok = fault("dw_band", s, "block of dY", 2 * p, 0, g.S32 - 2);
                    else ++formed[o];
                }
        });
    }
    for (int o = 0; o < w.nd && ok; ++o)
        if (formed[o] != due[o]) ok = fault("dw_band", s, "products", formed[o], due[o], due[o]);
    return ok;
}

template <int ND, int DG>
static bool dw_band_form(const Shape &s, const DwBandPlan &p)
{
    const bool dealt = p.split || s.dtype == DWCONV_F32;
    const dwconv::DwBandGeom &g = p.g;
    for (int win = 0; win < g.nwin; ++win) {
        const dwconv::DwBandWindow w = dwconv::dw_band_window(g, win, dealt);
        // (the stages of one group of rows: the others are like them)
        for (int st = 0; st < g.nstep; ++st) {
            dwconv::DwBandStage stage;
            stage.st = st;
            dwconv::dw_band_set_stage(g, w.dlo, stage);
            if (stage.nx <= 0) continue;
            const size_t bytes = (size_t)(1 << g.rg_log) * (size_t)(stage.nx + g.S32) * dwconv::dw_band_block_bytes(s.dtype == DWCONV_F32 ? 3 : 1);
            if (bytes > p.lds) return fault("dw_band", s, "bytes of a stage", (long long)bytes, 0, (long long)p.lds);
            if (!(dealt ? dw_band_stage<ND, DG, true>(s, g, w, stage) : dw_band_stage<ND, DG, false>(s, g, w, stage))) return false;
        }
    }
    return true;
}

static bool check_dw_band(const Shape &s)
{
    DwBandPlan p;
    if (!plan_dw_band(s, 1 << 20, &p)) return true;
    ++planned;
    if (s.dtype == DWCONV_F32) {
        // a chain of additions is no longer than with two rounds of workgroups, as far as stages and 16 MiB of partial sums go
        const long long wgs = (long long)s.C * p.g.nwin, slices = std::max(1ll, std::min({(1024 + wgs - 1) / wgs, (16ll << 20) / (4ll * s.C * s.K), (long long)p.g.stages}));
        const long long all = (p.g.stages + p.S - 1ll) / p.S, chain = p.g.chain > 0 ? std::min((long long)p.g.chain, all) : all, most = (p.g.stages + slices - 1) / slices;
        if (chain < 1 || chain > most) return fault("dw_band", s, "stages of a chain", chain, 1, most);
    }
    switch (8 * p.ND + p.g.dg_log) {
    case 8: return dw_band_form<1, 1>(s, p);
    case 16: return dw_band_form<2, 1>(s, p);
    case 17: return dw_band_form<2, 2>(s, p);
    case 18: return dw_band_form<2, 4>(s, p);
    case 24: return dw_band_form<3, 1>(s, p);
    case 25: return dw_band_form<3, 2>(s, p);
    case 26: return dw_band_form<3, 4>(s, p);
    case 34: return dw_band_form<4, 4>(s, p);
    default: return fault("dw_band", s, "form", 8 * p.ND + p.g.dg_log, 8, 34);
    }
}

// An item and a chunk of corr_band_kernel: the blocks of the window and the taps every wave reads.
template <int T>
static bool corr_band_item(const Shape &s, const BandPlan &p, const dwconv::BandStage &st)
{
    const dwconv::BandGeom &g = p.g;
    const int NL = s.dtype == DWCONV_F32 ? 3 : 1, BS = dwconv::band_block_bytes(NL), KS = dwconv::kBandWaves / g.TG, NBk = 1 << g.nb_log;
    const int blocks = st.n8 / 4, TP = dwconv::band_tap_dwords(g.F), tiles = g.PB >> g.nb_log;
    const int granules = p.few ? dwconv::kBandPrefetchF32Few : dwconv::band_prefetch(NL);
    if (blocks * BS > g.pitch) return fault("corr_band", s, "bytes of a window", blocks * BS, 0, g.pitch);
    if (g.RW * st.n8 > granules * dwconv::kBandThreads) return fault("corr_band", s, "granules of a window", g.RW * st.n8, 0, granules * dwconv::kBandThreads);
    std::vector<int> formed(tiles, 0), due(tiles, 0);
    bool ok = true;
    for (int wave = 0; wave < dwconv::kBandWaves; ++wave) {
        const int tg = wave % g.TG, ks = wave / g.TG;
        int tile[T], lo[T], hi[T];
        for (int t = 0; t < T; ++t) {
            tile[t] = dwconv::band_tile(g, tg, t);
            dwconv::band_tile_range(g, st, tile[t], lo[t], hi[t]);
            if (ks == 0 && dwconv::band_has_tile(g, st.p0, tile[t])) due[tile[t]] += std::max(0, hi[t] - lo[t] + 1);
        }
        dwconv::active_runs(lo, hi, [&](auto t0c, auto nc, int ea, int eb) {
            constexpr int T0 = decltype(t0c)::value, N = decltype(nc)::value;
            ea += (st.e_lo + ks - ea) & (KS - 1);
            for (int e = ea; e <= eb && ok; e += KS) {
                // dwords of a tap operand: either copy, lanes 0 .. 31 and halves 0, 1
                const int a = 16 * e + g.pad - st.j0 + dwconv::kBandTapMargin, d0 = (a - 31) >> 1, d1 = ((a + 8 + 1) >> 1) + 3;
                if (d0 < 0 || d1 >= TP) ok = fault("corr_band", s, "dwords of taps from", d0, 0, TP - 1 - (d1 - d0));
                for (int t = T0; t < T0 + N && ok; ++t) {
                    const int b0 = st.p0 - st.wb0 + (tile[t] << g.nb_log) + (e >> 1), b1 = b0 + NBk - 1;
                    if (!dwconv::band_has_tile(g, st.p0, tile[t])) ok = fault("corr_band", s, "product of tile", tile[t], 0, tiles - 1);
                    else if (b0 < 0 || b1 >= blocks) ok = fault("corr_band", s, "block of the window", b0 < 0 ? b0 : b1, 0, blocks - 1);
                    else ++formed[tile[t]];
                }
            }
        });
    }
    for (int t = 0; t < tiles && ok; ++t)
        if (formed[t] != due[t]) ok = fault("corr_band", s, "products", formed[t], due[t], due[t]);
    // (tiles are dealt once, spare ones excepted)
    for (int t = 0; t < tiles && ok; ++t) {
        int n = 0;
        for (int tg = 0; tg < g.TG; ++tg)
            for (int i = 0; i < T; ++i) n += dwconv::band_tile(g, tg, i) == t;
        if (n != 1) ok = fault("corr_band", s, "waves of a tile", n, 1, 1);
    }
    return ok;
}

static bool check_corr_band(const Shape &s)
{
    for (int reverse = 0; reverse < 2; ++reverse) {
        BandPlan p;
        if (!plan_corr_band(s, reverse ? s.K - 1 - s.pad : s.pad, reverse, &p)) continue;
        ++planned;
        for (int piece = 0; piece < p.g.NP; ++piece)
            for (int j0 = 0; j0 < s.K; j0 += p.g.F) {
                dwconv::BandStage st{};
                st.j0 = j0;
                st.p0 = piece * p.g.PB;
                if (!dwconv::band_set_window(p.g, st)) continue;
                if (!(p.T == 1 ? corr_band_item<1>(s, p, st) : p.T == 2 ? corr_band_item<2>(s, p, st) : corr_band_item<4>(s, p, st))) return false;
            }
    }
    return true;
}

// A piece and a chunk of dw_toep_kernel: the blocks of X and the taps every wave reads.
template <int T>
static bool dw_toep_stage(const Shape &s, const DwToepPlan &p, int p0, const dwconv::DwToepStage &st)
{
    const dwconv::DwToepGeom &g = p.g;
    const int NL = s.dtype == DWCONV_F32 ? 3 : 1, BS = dwconv::band_block_bytes(NL), KS = dwconv::kBandWaves, blocks = st.n8 / 4, TP = dwconv::band_tap_dwords(g.F);
    if (blocks * BS > g.tap_off) return fault("dw_toep", s, "bytes of a window", blocks * BS, 0, g.tap_off);
    if (st.n8 > dwconv::kToepX * dwconv::kToepThreads) return fault("dw_toep", s, "granules of a window", st.n8, 0, dwconv::kToepX * dwconv::kToepThreads);
    if (g.F > 8 * dwconv::kToepY * dwconv::kToepThreads) return fault("dw_toep", s, "positions of a chunk", g.F, 0, 8 * dwconv::kToepY * dwconv::kToepThreads);
    int formed[T] = {}, due[T] = {};
    bool ok = true;
    for (int ks = 0; ks < KS; ++ks) {
        int lo[T], hi[T];
        for (int t = 0; t < T; ++t) {
            dwconv::dw_toep_tile_range(g, st, p0 + 32 * t, lo[t], hi[t]);
            due[t] = std::max(0, hi[t] - lo[t] + 1);
        }
        dwconv::active_runs(lo, hi, [&](auto t0c, auto nc, int ea, int eb) {
            constexpr int T0 = decltype(t0c)::value, N = decltype(nc)::value;
            ea += (st.e_lo + ks - ea) & (KS - 1);
            for (int e = ea; e <= eb && ok; e += KS) {
                const int a = 16 * e - st.t0 + dwconv::kBandTapMargin, d0 = (a - 31 + 1) >> 1, d1 = ((a + 8 + 1) >> 1) + 3;
                if (d0 < 0 || d1 >= TP) ok = fault("dw_toep", s, "dwords of taps from", d0, 0, TP - 1 - (d1 - d0));
                for (int t = T0; t < T0 + N && ok; ++t) {
                    const int b0 = p0 + 32 * t - st.wb0 + (e >> 1), b1 = b0 + 31;
                    if (b0 < 0 || b1 >= blocks) ok = fault("dw_toep", s, "block of the window", b0 < 0 ? b0 : b1, 0, blocks - 1);
                    else ++formed[t];
                }
            }
        });
    }
    for (int t = 0; t < T && ok; ++t)
        if (formed[t] != due[t]) ok = fault("dw_toep", s, "products", formed[t], due[t], due[t]);
    return ok;
}

static bool check_dw_toep(const Shape &s)
{
    DwToepPlan p;
    if (!plan_dw_toep(s, 1 << 20, &p)) return true;
    ++planned;
    const dwconv::DwToepGeom &g = p.g;
    // fp32: chains of about the root of the products an element sums on a wave
    const double root = std::max(s.B < 5 ? 4.0 : 8.0, std::sqrt((double)g.rows * s.L / 64));
    if (s.dtype == DWCONV_F32 && (g.run > 4 * root || g.run < 4 * (root - 1) || (g.run & 3) != 0))
        return fault("dw_toep", s, "e of a chain", g.run, (long long)(4 * (root - 1)), (long long)(4 * root));
    for (int piece = 0; piece < g.npiece; ++piece)
        for (int t0 = 0; t0 < s.L; t0 += g.F) {
            dwconv::DwToepStage st{};
            st.t0 = t0;
            const int p0 = g.blk0 + piece * 32 * p.T;
            if (!dwconv::dw_toep_set_window(g, p0, 32 * p.T, st)) continue;
            if (!(p.T == 1 ? dw_toep_stage<1>(s, p, p0, st) : dw_toep_stage<2>(s, p, p0, st))) return false;
        }
    return true;
}

// Shapes over the range of the kernels: causal, nearly causal, centred, anti-causal and any other pad, few and many batch entries.
static Shape draw(std::mt19937 &rng)
{
    auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
    auto spread = [&](double lo, double hi) { return (int)(lo * std::pow(hi / lo, (rng() % 100001u) / 100000.0)); };
    Shape s;
    s.B = upto(3) ? spread(1, 12) : spread(1, 3000);
    s.C = spread(1, 1000);
    s.L = spread(8, 9000);
    s.K = upto(4) ? std::min(s.L, spread(66, 9000)) : spread(66, 12000);
    switch (upto(6)) {
    case 0: s.pad = s.K - 1; break;
    case 1: s.pad = 0; break;
    case 2: s.pad = (s.K - 1) / 2; break;
    case 3: s.pad = s.K - 1 - upto(std::max(1, s.K / 4)); break;
    case 4: s.pad = upto(std::max(1, s.K / 4)); break;
    default: s.pad = upto(s.K); break;
    }
    s.dtype = upto(2) ? DWCONV_F32 : DWCONV_BF16;
    return s;
}

int main(int argc, char **argv)
{
    // kernel seed count, or kernel - and lines "B C L K pad dtype" on standard input
    if (argc < 3) return 2;
    bool (*check)(const Shape &) = nullptr;
    if (!strcmp(argv[1], "dw_band")) check = check_dw_band;
    if (!strcmp(argv[1], "corr_band")) check = check_corr_band;
    if (!strcmp(argv[1], "dw_toep")) check = check_dw_toep;
    if (!check) return 2;
    int bad = 0;
    if (!strcmp(argv[2], "-")) {
        Shape s;
        while (scanf("%d %d %d %d %d %d", &s.B, &s.C, &s.L, &s.K, &s.pad, &s.dtype) == 6) bad += !check(s);
    } else {
        std::mt19937 rng((unsigned)atoi(argv[2]));
        for (int i = 0, n = argc > 3 ? atoi(argv[3]) : 1; i < n && bad < 20; ++i) bad += !check(draw(rng));
    }
    printf("%d shapes planned, %d at fault\n", planned, bad);
    return bad ? 1 : 0;
}
