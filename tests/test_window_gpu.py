"""corr_window_kernel (fp32 forward and input gradient, filters of about 65 to 260 taps, calls that fill the chip) and dw_window_kernel (weight
gradient, about 65 to 130 taps) against the oracle, bit for bit on small integers and on values that need all three limbs."""
import pytest
import torch

from _parity import empty_device, small_ints, to_device
from paper_2604_25422_amd import binding
from paper_2604_25422_amd.workloads import as_f32_numpy
from test_exact_gpu import _kernels, _same, test_exact_fp32_needs_every_limb

pytestmark = pytest.mark.gpu

# every form of the kernel (chunks a tile reads, chunks in registers), rows in one piece and in several, waves of one unit and of more, rows that end
# inside a granule, units that the batch does not fill
SHAPES = [
    (124, 256, 252, 79, 39), (861, 64, 230, 67, 33), (39, 192, 1273, 67, 33), (162, 128, 768, 75, 25), (166, 128, 557, 69, 34),
    (42, 128, 2263, 88, 44), (188, 160, 320, 108, 54), (388, 131, 249, 108, 54), (49, 128, 1996, 106, 53), (54, 160, 1276, 102, 51), (314, 64, 542, 99, 49),
    (313, 128, 315, 129, 22), (628, 96, 176, 137, 68), (158, 131, 625, 160, 80), (94, 131, 888, 133, 129), (137, 64, 1343, 141, 0), (210, 96, 553, 130, 0),
    (817, 64, 248, 191, 95), (267, 192, 246, 163, 81), (477, 64, 237, 162, 81), (62, 96, 2128, 189, 0), (81, 64, 2169, 189, 87), (27, 192, 2077, 162, 81),
    (478, 64, 242, 199, 99), (430, 128, 192, 207, 103), (190, 160, 352, 211, 0), (189, 131, 310, 218, 109), (19, 256, 2536, 212, 106), (158, 96, 638, 196, 86),
    (49, 256, 933, 192, 129), (288, 96, 376, 237, 118), (801, 64, 249, 226, 113), (46, 256, 992, 255, 0), (191, 64, 874, 241, 240), (511, 128, 255, 250, 125),
    (512, 128, 256, 256, 255), (103, 192, 547, 229, 228),
]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,C,L,K,p", SHAPES)
def test_exact_corr_window(oracle_mod, B, C, L, K, p, offset):
    print(f"case window B{B} C{C} L{L} K{K} p{p} offset {offset}", flush=True)
    tdt, what = torch.float32, f"B{B} C{C} L{L} K{K} p{p} offset {offset}"
    x, w = small_ints((B, C, L), 71, 3, tdt), small_ints((C, K), 72, 3, tdt)
    xd, wd = to_device(x, offset), to_device(w, offset)
    y, dx = empty_device((B, C, L), tdt, offset), empty_device((B, C, L), tdt, offset)
    names = _kernels(lambda: binding.dwconv_fwd(xd, wd, p, out=y)) + _kernels(lambda: binding.dwconv_bwd_input(xd, wd, p, out=dx))
    assert len(names) == 2 and all("corr_window_kernel" in n for n in names), names
    xn, wn = as_f32_numpy(x), as_f32_numpy(w)
    _same("fwd", y, oracle_mod.fwd(xn, wn, p)[0], tdt, what)
    _same("dx", dx, oracle_mod.bwd_input(xn, wn, p)[0], tdt, what)


# ... with every limb of the rows, tap by tap: a tap's product is now the first and now the last of a tile, and the first and the last tile of
# a step alone in it.  And the same bits again from normal data, where a product that is not there yet would be there another time.
@pytest.mark.parametrize("B,C,L,K,p", SHAPES + [(857, 96, 144, 160, 159), (528, 96, 272, 145, 0)])
def test_every_tap_alone_corr_window(B, C, L, K, p):
    print(f"case window tap by tap B{B} C{C} L{L} K{K} p{p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(B, C, L, generator=g, device="cuda")
    y, want = torch.empty_like(x), torch.zeros_like(x)
    for j in sorted({*range(0, K, 11), max(p - 1, 0), p, min(p + 1, K - 1), K - 1}):
        w = torch.zeros(C, K, device="cuda"); w[:, j] = 1.0
        for call, o in ((binding.dwconv_fwd, j - p), (binding.dwconv_bwd_input, p - j)):      # y[t] takes x[t + o]
            a, b = max(0, -o), min(L, L - o)
            call(x, w, p, out=y)
            want.zero_()
            if a < b:
                want[..., a:b] = x[..., a + o:b + o]
            assert torch.equal(y, want), f"{call.__name__} tap {j}: {int((y != want).sum())} outputs differ"
    w = torch.randn(C, K, generator=g, device="cuda")
    for call in (binding.dwconv_fwd, binding.dwconv_bwd_input):
        first = call(x, w, p)
        for _ in range(4):
            assert torch.equal(call(x, w, p), first), f"{call.__name__}: other bits"


# Calls that the kernel could make and leaves to others, and their neighbours: seven and eight block offsets where memory is near (off cache lines and
# not), virtual rows, rows of three steps off half cache lines, pieces of few steps and workgroups that crowd some SIMDs
@pytest.mark.parametrize("B,C,L,K,p,window", [
    (600, 64, 520, 97, 48, False), (500, 64, 688, 80, 40, False), (600, 64, 520, 110, 55, True), (139, 96, 896, 75, 37, False), (109, 256, 1082, 80, 40, True),
    (84, 32, 7952, 79, 39, False), (374, 160, 180, 75, 20, False), (373, 160, 176, 68, 34, True), (277, 128, 498, 143, 71, False), (94, 651, 208, 181, 90, False),
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


# dw_window_kernel (fp32 weight gradient, at most five 32-blocks): four and five offsets, rows in one piece and in several, one slice and more,
# rows that end inside a granule, units that the batch does not fill
DW_SHAPES = [
    (179, 256, 240, 85, 84), (128, 256, 348, 96, 95), (56, 256, 780, 104, 52), (148, 256, 272, 118, 117), (58, 256, 541, 111, 55), (57, 256, 566, 113, 56),
    (349, 128, 244, 119, 118), (463, 128, 192, 125, 96), (89, 256, 1029, 95, 94), (93, 250, 1264, 86, 85), (460, 64, 526, 83, 82), (38, 256, 1796, 117, 0), (32, 250, 1840, 121, 0),
    (42, 255, 1305, 104, 52), (42, 255, 1281, 101, 50), (41, 250, 2096, 127, 126), (191, 128, 848, 112, 56), (64, 128, 2617, 124, 123), (192, 128, 886, 123, 122),
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
    if offset == 0:
        assert "dw_window_kernel" in names[0], names
        # the partial sums alone: every slice of the workspace is written, and their sum is the gradient
        ws = binding.new_workspace(xd, K, p)
        ws.fill_(255)
        S = binding.dwconv_bwd_weight_slices(B, C, L, K, p, binding.F32)
        binding.dwconv_bwd_weight_partial(xd, dyd, K, p, workspace=ws)
        _same("partial", ws.view(torch.float32)[:S * C * K].view(S, C, K).sum(0), ref, tdt, what)


@pytest.mark.parametrize("B,C,L,K,p", [(179, 256, 240, 85, 84), (58, 256, 541, 111, 55)])
def test_every_limb_dw_window(B, C, L, K, p):
    test_exact_fp32_needs_every_limb(B, C, L, K, p)
