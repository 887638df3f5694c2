"""corr_window_kernel (fp32 forward and input gradient, filters of about 65 to 260 taps, calls that fill the chip) and dw_window_kernel (weight
gradient, about 65 to 130 taps): against the oracle on small integers, on values that need all three limbs and at the edges of the range, bit for
bit; and which calls go to them."""
import pytest
import torch

from _parity import empty_device, small_ints, to_device
from paper_2604_25422_amd import binding
from paper_2604_25422_amd.workloads import as_f32_numpy
from test_exact_gpu import _kernels, _same, test_exact_fp32_needs_every_limb
from test_limits_gpu import PAIRS

pytestmark = pytest.mark.gpu

# every form of the kernel (chunks a tile reads, chunks in registers), rows in one piece and in several, waves of one unit and of more, rows that end
# inside a granule, units that the batch does not fill
SHAPES = [
    (374, 160, 180, 75, 20), (482, 128, 179, 81, 40), (159, 96, 824, 97, 0), (42, 128, 2263, 88, 44), (188, 160, 320, 108, 54), (388, 131, 249, 108, 54),
    (49, 128, 1996, 106, 53), (19, 256, 2478, 110, 0), (871, 64, 228, 134, 77), (158, 131, 625, 160, 80), (94, 131, 888, 133, 129), (137, 64, 1343, 141, 0),
    (817, 64, 248, 191, 95), (793, 64, 247, 171, 0), (62, 96, 2128, 189, 0), (81, 64, 2169, 189, 87), (190, 160, 352, 211, 0), (189, 131, 310, 218, 109),
    (19, 256, 2536, 212, 106), (158, 96, 638, 196, 86), (288, 96, 376, 237, 118), (801, 64, 249, 226, 113), (46, 256, 992, 255, 0), (191, 64, 874, 241, 240),
    (511, 128, 255, 250, 125), (512, 128, 256, 256, 255),
    (124, 256, 252, 79, 39), (861, 64, 230, 67, 33), (39, 192, 1273, 67, 33), (162, 128, 768, 75, 25), (166, 128, 557, 69, 34), (54, 160, 1276, 102, 51),
    (314, 64, 542, 99, 49), (313, 128, 315, 129, 22), (628, 96, 176, 137, 68), (210, 96, 553, 130, 0), (267, 192, 246, 163, 81), (477, 64, 237, 162, 81),
    (27, 192, 2077, 162, 81), (478, 64, 242, 199, 99), (430, 128, 192, 207, 103), (49, 256, 933, 192, 129), (103, 192, 547, 229, 228),
]
# ... directions that go to it, where not both do (159: us of corr_mfma_kernel / here, forward 33 / 35, input gradient 31 / 35)
WAYS = {(159, 96, 824, 97, 0): 0, (871, 64, 228, 134, 77): 1, (793, 64, 247, 171, 0): 1}


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,C,L,K,p", SHAPES)
def test_exact_corr_window(oracle_mod, B, C, L, K, p, offset):
    print(f"case window B{B} C{C} L{L} K{K} p{p} offset {offset}", flush=True)
    tdt, what = torch.float32, f"B{B} C{C} L{L} K{K} p{p} offset {offset}"
    x, w = small_ints((B, C, L), 71, 3, tdt), small_ints((C, K), 72, 3, tdt)
    xd, wd = to_device(x, offset), to_device(w, offset)
    y, dx = empty_device((B, C, L), tdt, offset), empty_device((B, C, L), tdt, offset)
    names = _kernels(lambda: binding.dwconv_fwd(xd, wd, p, out=y)) + _kernels(lambda: binding.dwconv_bwd_input(xd, wd, p, out=dx))
    assert len(names) == 2 and sum("corr_window_kernel" in n for n in names) == WAYS.get((B, C, L, K, p), 2), names
    xn, wn = as_f32_numpy(x), as_f32_numpy(w)
    _same("fwd", y, oracle_mod.fwd(xn, wn, p)[0], tdt, what)
    _same("dx", dx, oracle_mod.bwd_input(xn, wn, p)[0], tdt, what)


@pytest.mark.parametrize("B,C,L,K,p,window", [(600, 64, 520, 97, 48, False), (500, 64, 688, 80, 40, False), (600, 64, 544, 97, 48, False), (600, 64, 520, 110, 55, True)])
def test_seven_offsets_on_virtual_rows(oracle_mod, B, C, L, K, p, window):
    """Rows of more than 512 positions keep the register-resident kernel at seven block offsets where it is the faster one (us, of whole lines 49 / 52);
    more offsets do not."""
    print(f"case window B{B} C{C} L{L} K{K} p{p}", flush=True)
    x, w = small_ints((B, C, L), 75, 3, torch.float32), small_ints((C, K), 76, 3, torch.float32)
    xd, wd = x.cuda(), w.cuda()
    y = torch.empty_like(xd)
    names = _kernels(lambda: binding.dwconv_fwd(xd, wd, p, out=y))
    assert len(names) == 1 and ("corr_window_kernel" in names[0]) == window, names
    _same("fwd", y, oracle_mod.fwd(as_f32_numpy(x), as_f32_numpy(w), p)[0], torch.float32, f"B{B} C{C} L{L} K{K} p{p}")


@pytest.mark.parametrize("B,C,L,K,p", [(62, 64, 2251, 114, 65), (512, 128, 256, 256, 255)])
def test_every_limb_corr_window(B, C, L, K, p):
    test_exact_fp32_needs_every_limb(B, C, L, K, p)


def test_non_finite_values_stay_where_the_definition_puts_them():
    """An infinity or NaN reaches outputs of its own row up to 63 positions beyond what the definition says, and the other outputs are what they are
    without it; sums above 10^19 are as good as any."""
    B, C, L, K, p = 62, 64, 2251, 114, 65
    g = torch.Generator(device="cuda").manual_seed(5)
    x, w = torch.randn(B, C, L, generator=g, device="cuda"), torch.randn(C, K, generator=g, device="cuda")
    clean = binding.dwconv_fwd(x, w, p)
    for at, v in ((700, float("inf")), (0, float("nan")), (L - 1, float("-inf"))):
        bad = x.clone()
        bad[30, 7, at] = v
        y = binding.dwconv_fwd(bad, w, p)
        lo, hi = max(0, at - (K - 1 - p) - 63), min(L, at + p + 64)
        touched = torch.zeros_like(y, dtype=torch.bool)
        touched[30, 7, lo:hi] = True
        assert torch.equal(y[~touched], clean[~touched])
        assert not torch.isfinite(y[30, 7, max(0, at - (K - 1 - p)):min(L, at + p + 1)]).any()
    big = binding.dwconv_fwd(x * 2.0 ** 100, w, p)
    assert torch.equal(big, clean * 2.0 ** 100)


def _shifted(v, o, out):                                 # v[t + o], zeros outside the row
    L = v.shape[-1]
    a, b = max(0, -o), min(L, L - o)
    out.zero_()
    if a < b:
        out[..., a:b] = v[..., a + o:b + o]
    return out


# ... with every limb of the rows, tap by tap - a tap's product is now the first and now the last of a tile, and the first and the last tile of
# a step alone in it - and of the taps, position by position.  And the same bits again from normal data, where a product that is not there yet
# would be there another time.  (The last two calls: rows whose last step is one tile.)
@pytest.mark.parametrize("B,C,L,K,p", SHAPES + [(857, 96, 144, 160, 159), (528, 96, 272, 145, 0)])
def test_every_limb_of_rows_and_taps_corr_window(B, C, L, K, p):
    print(f"case window every limb B{B} C{C} L{L} K{K} p{p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x, w = torch.randn(B, C, L, generator=g, device="cuda"), torch.randn(C, K, generator=g, device="cuda")
    if (B, C, L, K, p) in SHAPES:
        names = _kernels(lambda: (binding.dwconv_fwd(x, w, p), binding.dwconv_bwd_input(x, w, p)))
        assert len(names) == 2 and sum("corr_window_kernel" in n for n in names) == WAYS.get((B, C, L, K, p), 2), names
    y, want, one_w, one_x = torch.empty_like(x), torch.empty_like(x), torch.zeros_like(w), torch.zeros_like(x)
    for j in sorted({*range(0, K, 11), max(p - 1, 0), p, min(p + 1, K - 1), K - 1}):
        one_w.zero_()
        one_w[:, j] = 1.0
        for call, o in ((binding.dwconv_fwd, j - p), (binding.dwconv_bwd_input, p - j)):      # y[t] takes x[t + o]
            call(x, one_w, p, out=y)
            assert torch.equal(y, _shifted(x, o, want)), f"{call.__name__} tap {j}: {int((y != want).sum())} outputs differ"
    t = torch.arange(L, device="cuda")
    for u in sorted({0, 1, L // 3, L // 2, L - 17, L - 1}):
        one_x.zero_()
        one_x[:, :, u] = 1.0
        for call, sign in ((binding.dwconv_fwd, -1), (binding.dwconv_bwd_input, 1)):          # tap p + sign (t - u) reaches position t
            j = p + sign * (t - u)
            rows = torch.where((j >= 0) & (j < K), w[:, j.clamp(0, K - 1)], torch.zeros((), device="cuda"))
            call(one_x, w, p, out=y)
            assert torch.equal(y, rows.expand(B, C, L)), f"{call.__name__} position {u}: outputs differ"
    for call in (binding.dwconv_fwd, binding.dwconv_bwd_input):
        first = call(x, w, p)
        for _ in range(4):
            assert torch.equal(call(x, w, p), first), f"{call.__name__}: other bits"


# Calls that the kernel could make and leaves to others, and their neighbours: seven and eight block offsets where memory is near (off cache lines and
# not), virtual rows, rows of three steps off half cache lines, pieces of few steps and workgroups that crowd some SIMDs
@pytest.mark.parametrize("B,C,L,K,p,window", [
    (139, 96, 896, 75, 37, False), (109, 256, 1082, 80, 40, True), (84, 32, 7952, 79, 39, False), (234, 64, 1184, 107, 0, True),
    (1075, 194, 185, 70, 35, False), (374, 160, 180, 75, 20, True), (373, 160, 176, 68, 34, True), (277, 128, 498, 143, 71, False), (94, 651, 208, 181, 90, False),
    (62, 64, 2251, 114, 65, False),
])
def test_which_calls_corr_window_takes(oracle_mod, B, C, L, K, p, window):
    print(f"case window B{B} C{C} L{L} K{K} p{p}", flush=True)
    x, w = small_ints((B, C, L), 75, 3, torch.float32), small_ints((C, K), 76, 3, torch.float32)
    xd, wd = x.cuda(), w.cuda()
    y = torch.empty_like(xd)
    names = _kernels(lambda: binding.dwconv_fwd(xd, wd, p, out=y))
    assert len(names) == 1 and ("corr_window_kernel" in names[0]) == window, names
    _same("fwd", y, oracle_mod.fwd(as_f32_numpy(x), as_f32_numpy(w), p)[0], torch.float32, f"B{B} C{C} L{L} K{K} p{p}")


# Rows in one piece and in several that end inside a granule, in one unit a wave and more
EDGE = [(49, 128, 1996, 106, 53), (314, 64, 542, 99, 49), (512, 128, 256, 256, 255), (313, 128, 315, 129, 22)]


@pytest.mark.parametrize("B,C,L,K,p", EDGE)
def test_non_finite_values_of_corr_window(B, C, L, K, p):
    """An infinity or NaN reaches outputs of its own row up to 63 positions beyond what the definition says, and the other outputs are what they are
    without it; among operands of one sign an infinity stays one; sums above 10^19 are as good as any."""
    print(f"case window not finite B{B} C{C} L{L} K{K} p{p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x, w = torch.randn(B, C, L, generator=g, device="cuda"), torch.randn(C, K, generator=g, device="cuda")
    for call, before, behind in ((binding.dwconv_fwd, K - 1 - p, p), (binding.dwconv_bwd_input, p, K - 1 - p)):
        names = _kernels(lambda: call(x, w, p))
        assert "corr_window_kernel" in names[0], names
        clean = call(x, w, p)
        for at, v in ((L // 2 + 3, float("inf")), (0, float("nan")), (L - 1, float("-inf"))):
            bad = x.clone()
            bad[B // 2, 7, at] = v
            y = call(bad, w, p)
            touched = torch.zeros_like(y, dtype=torch.bool)
            touched[B // 2, 7, max(0, at - before - 63):min(L, at + behind + 64)] = True
            assert torch.equal(y[~touched], clean[~touched])
            assert not torch.isfinite(y[B // 2, 7, max(0, at - before):min(L, at + behind + 1)]).any()
            if at != 0:
                bad = x.abs()
                bad[B // 2, 7, at] = v
                y = call(bad, w.abs() + 0.5, p)
                assert (y[B // 2, 7, max(0, at - before):min(L, at + behind + 1)] == v).all()
        assert torch.equal(call(x * 2.0 ** 100, w, p), clean * 2.0 ** 100)


def _top_of_the_range(B, C, L, K, p, dw):
    u, j = L // 2, p + 20 if p + 20 < K else p - 20
    x, w, dy = torch.zeros(B, C, L, device="cuda"), torch.zeros(C, K, device="cuda"), torch.zeros(B, C, L, device="cuda")
    for a, b in PAIRS:
        x[:, :, u], w[:, j], dy[0, :, u + 3] = a, b, b                          # one product per output, one pair per coefficient
        exp = (torch.tensor([a], dtype=torch.float32).double() * torch.tensor([b], dtype=torch.float32).double()).float().cuda()
        if dw:                                                                  # dw[j] takes dy[u + 3] x[u + 3 + j - p]
            cases = [(binding.dwconv_bwd_weight(x, dy, K, p), (slice(None), p - 3))]
        else:
            cases = [(binding.dwconv_fwd(x, w, p), (slice(None), slice(None), u - j + p)), (binding.dwconv_bwd_input(x, w, p), (slice(None), slice(None), u + j - p))]
        for got, at in cases:
            want = torch.zeros_like(got)
            want[at] = exp
            assert not torch.isnan(got).any(), f"{a!r} x {b!r}: a NaN from finite inputs"
            assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.equal(got.sign(), want.sign()), f"{a!r} x {b!r}"
            # (three limbs per operand, the products of the small ones left out: 2^-24 of the product, and roundings of the sums)
            fin = torch.isfinite(want)
            assert float(((got[fin].double() - want[fin].double()).abs() / want[fin].double().abs().clamp_min(1e-30)).max()) <= 2.0 ** -22, f"{a!r} x {b!r}"


@pytest.mark.parametrize("B,C,L,K,p", EDGE)
def test_products_at_the_top_of_the_range_corr_window(B, C, L, K, p):
    print(f"case window top of the range B{B} C{C} L{L} K{K} p{p}", flush=True)
    _top_of_the_range(B, C, L, K, p, False)


# dw_window_kernel (fp32 weight gradient, at most five 32-blocks): four and five offsets, rows in one piece and in several, one slice and more,
# rows that end inside a granule, units that the batch does not fill
DW_SHAPES = [
    (179, 256, 240, 85, 84), (128, 256, 348, 96, 95), (56, 256, 780, 104, 52), (148, 256, 272, 118, 117), (58, 256, 541, 111, 55), (57, 256, 566, 113, 56),
    (349, 128, 244, 119, 118), (463, 128, 192, 125, 96), (96, 256, 817, 89, 59), (31, 255, 2836, 85, 84), (32, 250, 2848, 87, 0), (32, 250, 1840, 121, 0),
    (42, 255, 1305, 104, 52), (42, 255, 1281, 101, 50), (41, 250, 2096, 127, 126), (191, 128, 848, 112, 56), (64, 128, 2617, 124, 123), (192, 128, 886, 123, 122),
    (89, 256, 1029, 95, 94), (93, 250, 1264, 86, 85), (460, 64, 526, 83, 82), (38, 256, 1796, 117, 0),
]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,C,L,K,p", DW_SHAPES)
def test_exact_dw_window(oracle_mod, B, C, L, K, p, offset):
    print(f"case dw window B{B} C{C} L{L} K{K} p{p} offset {offset}", flush=True)
    tdt, what = torch.float32, f"B{B} C{C} L{L} K{K} p{p} offset {offset}"
    assert 9 * B * L < 2 ** 24
    x, dy = small_ints((B, C, L), 73, 3, tdt), small_ints((B, C, L), 74, 3, tdt)
    xd, dyd = to_device(x, offset), to_device(dy, offset)
    dw = torch.empty(C, K, device="cuda")
    names = _kernels(lambda: binding.dwconv_bwd_weight(xd, dyd, K, p, out=dw))
    ref = oracle_mod.bwd_weight(as_f32_numpy(x), as_f32_numpy(dy), K, p)[0]
    _same("dw", dw, ref, tdt, what)
    assert "dw_window_kernel" in names[0], names
    if offset == 0:
        # the partial sums alone: every slice of the workspace is written, and their sum is the gradient
        ws = binding.new_workspace(xd, K, p)
        ws.fill_(255)
        S = binding.dwconv_bwd_weight_slices(B, C, L, K, p, binding.F32)
        binding.dwconv_bwd_weight_partial(xd, dyd, K, p, workspace=ws)
        _same("partial", ws.view(torch.float32)[:S * C * K].view(S, C, K).sum(0), ref, tdt, what)


# Rows in one piece and in several, rows that end inside a granule
DW_EDGE = [(179, 256, 240, 85, 84), (58, 256, 541, 111, 55), (41, 250, 2096, 127, 126), (89, 256, 1029, 95, 94)]


@pytest.mark.parametrize("B,C,L,K,p", DW_EDGE)
def test_every_limb_dw_window(B, C, L, K, p):
    test_exact_fp32_needs_every_limb(B, C, L, K, p)


@pytest.mark.parametrize("B,C,L,K,p", DW_EDGE)
def test_non_finite_values_of_dw_window(B, C, L, K, p):
    """Other channels keep their bits, also where the value stands next to them in memory; the coefficients that the definition reaches are not finite, and
    an infinity among operands of one sign stays one."""
    print(f"case dw window not finite B{B} C{C} L{L} K{K} p{p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dy = torch.randn(B, C, L, generator=g, device="cuda"), torch.randn(B, C, L, generator=g, device="cuda")
    names = _kernels(lambda: binding.dwconv_bwd_weight(x, dy, K, p))
    assert "dw_window_kernel" in names[0], names
    clean = binding.dwconv_bwd_weight(x, dy, K, p)
    others = [c for c in range(C) if c != 7]
    for at, v in ((L // 2 + 3, float("inf")), (0, float("nan")), (L - 1, float("-inf"))):
        for which, jlo, jhi in (("x", at + p - L + 1, at + p), ("dy", p - at, p - at + L - 1)):
            jlo, jhi = max(jlo, 0), min(jhi, K - 1)
            bad = [x.clone(), dy.clone()]
            bad[which == "dy"][B - 1, 7, at] = v
            dw = binding.dwconv_bwd_weight(*bad, K, p)
            assert torch.equal(dw[others], clean[others]), f"{which}: another channel changed"
            assert not torch.isfinite(dw[7, jlo:jhi + 1]).any()
            if at != 0:
                bad = [x.abs(), dy.abs() + 0.5]
                bad[which == "dy"][B - 1, 7, at] = v
                assert (binding.dwconv_bwd_weight(*bad, K, p)[7, jlo:jhi + 1] == v).all()
    assert torch.equal(binding.dwconv_bwd_weight(x * 2.0 ** 100, dy, K, p), clean * 2.0 ** 100)


@pytest.mark.parametrize("B,C,L,K,p", DW_EDGE)
def test_products_at_the_top_of_the_range_dw_window(B, C, L, K, p):
    print(f"case dw window top of the range B{B} C{C} L{L} K{K} p{p}", flush=True)
    _top_of_the_range(B, C, L, K, p, True)
