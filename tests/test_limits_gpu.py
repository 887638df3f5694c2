"""Edges of the contract in include/dwconv.h: tensors above 2^32 bytes (64-bit row offsets next to 32-bit
segment walks) and non-finite inputs (the matrix-core kernels multiply the zero taps of their edge Toeplitz blocks
and the zero-filled halos, where the definition of Sec. IV-A skips the term)."""
import numpy as np
import pytest
import torch

from paper_2604_25422_amd import binding
from paper_2604_25422_amd.workloads import as_f32_numpy

pytestmark = pytest.mark.gpu


def _device_ints(shape, seed, lim, tdt):
    """Seeded integers in [-lim, lim], drawn on the device batch by batch (the tensor is larger than 4 GiB)."""
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    out = torch.empty(shape, dtype=tdt, device="cuda")
    step = max(1, (1 << 28) // (shape[1] * shape[2]))
    for a in range(0, shape[0], step):
        n = min(step, shape[0] - a)
        out[a:a + n] = torch.randint(-lim, lim + 1, (n,) + tuple(shape[1:]), generator=g, dtype=torch.int8, device="cuda").to(tdt)
    return out


# (B, C, L, K, pad_left, storage, lim): x and dY are integers in [-lim, lim], w in [-3, 3]; every sum stays
# below 2^24, so the comparison with the oracle is exact.  Rows (fwd, dX) of the first, a middle and the last batch
# and the channels 0, C/2 and C-1 (dW, over all batches) are checked: the first and last bytes of the tensor, and
# element offsets on both sides of 2^31 and 2^32.
@pytest.mark.parametrize("B,C,L,K,p,dtype,lim", [
    (1100, 1024, 2048, 32, 31, "bf16", 2),       # 4.6 GB per tensor: register-resident filters, bf16 matrix instruction
    (600, 1024, 2048, 64, 63, "f32", 3),         # 5.0 GB per tensor: headline class, one workgroup per channel for dW
    (190000, 128, 48, 48, 24, "f32", 1),         # 4.7 GB per tensor: the paper's rows, sixteen to a matrix tile
    (50, 96, 300000, 7, 3, "f32", 1),            # 5.8 GB per tensor: rows of 1.2 MB, 293 segments each
])
def test_tensors_above_4_GiB(oracle_mod, B, C, L, K, p, dtype, lim):
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    es = 4 if dtype == "f32" else 2
    assert B * C * L * es > 1 << 32 and lim * lim * B * L < 1 << 24 and 3 * lim * K < 1 << 24
    print(f"case above 4 GiB {dtype} B{B} C{C} L{L} K{K} p{p}: {B * C * L * es / 2 ** 30:.2f} GiB per tensor", flush=True)
    x = _device_ints((B, C, L), 61, lim, tdt)
    dy = _device_ints((B, C, L), 62, lim, tdt)
    g = torch.Generator(device="cpu"); g.manual_seed(63)
    w = torch.randint(-3, 4, (C, K), generator=g, dtype=torch.int32).to(tdt)
    wd = w.cuda()
    y = binding.dwconv_fwd(x, wd, p)
    dx = binding.dwconv_bwd_input(dy, wd, p)
    dw = binding.dwconv_bwd_weight(x, dy, K, p)
    torch.cuda.synchronize()
    dx_f = torch.empty_like(dx)
    _, dw_f = binding.dwconv_bwd(dy, x, wd, p, out_dx=dx_f)
    torch.cuda.synchronize()
    assert torch.equal(dx_f, dx), "dwconv_bwd: dx differs from dwconv_bwd_input"
    del dx_f
    wn = as_f32_numpy(w)
    bsel = [0, B // 2, B - 1]
    xs = as_f32_numpy(x[bsel].cpu()); dys = as_f32_numpy(dy[bsel].cpu())
    ref, _ = oracle_mod.fwd(xs, wn, p)
    assert torch.equal(y[bsel].cpu(), torch.from_numpy(ref).float().to(tdt)), "fwd differs on the sampled batches"
    ref, _ = oracle_mod.bwd_input(dys, wn, p)
    assert torch.equal(dx[bsel].cpu(), torch.from_numpy(ref).float().to(tdt)), "dX differs on the sampled batches"
    csel = [0, C // 2, C - 1]
    xc = as_f32_numpy(x[:, csel].contiguous().cpu()); dyc = as_f32_numpy(dy[:, csel].contiguous().cpu())
    ref, _ = oracle_mod.bwd_weight(xc, dyc, K, p)
    assert np.all(np.abs(ref) < 2.0 ** 24)
    exp = torch.from_numpy(ref).float().to(tdt)
    assert torch.equal(dw[csel].cpu(), exp), "dW differs on the sampled channels"
    assert torch.equal(dw_f[csel].cpu(), exp), "dW of dwconv_bwd differs on the sampled channels"


# Non-finite inputs.  The contract (include/dwconv.h): an Inf or NaN at position u of row (b, c) reaches, besides the
# outputs the definition gives it, at most the outputs of the same row within 63 positions of those and the last 63
# positions of row (b - 1, c) / the first 63 of row (b + 1, c) (short rows of a channel are processed end to end); no
# other channel is touched.  In the weight gradient it may reach every coefficient of its channel and no other channel.
# (B, C, L, K, pad_left, storage): one shape per kernel family (those that take large calls only, corr_window_kernel and dw_window_kernel: in
# test_window_gpu.py, with the top of the range and the infinities).
NONFINITE = [
    (2, 3, 2600, 64, 63, "f32"), (2, 3, 2600, 64, 20, "f32"), (2, 3, 2600, 7, 3, "f32"), (2, 3, 2600, 130, 129, "f32"),
    (2, 3, 2608, 64, 63, "bf16"), (2, 3, 2608, 200, 100, "bf16"),
    (40, 4, 48, 48, 24, "f32"), (40, 4, 48, 48, 24, "bf16"), (60, 4, 200, 31, 15, "f32"),
    (2, 3, 1024, 700, 699, "f32"), (2, 3, 1024, 700, 350, "bf16"),
    (2, 3, 1001, 9, 4, "f32"), (2, 3, 1001, 300, 299, "f32"),
    # ... dw_toep_kernel with several chunks of a row
    (2, 3, 4100, 900, 899, "f32"), (2, 3, 9000, 1500, 700, "bf16"),
]
SLOP = 63


@pytest.mark.parametrize("B,C,L,K,p,dtype", NONFINITE)
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_non_finite_inputs_stay_where_the_contract_says(B, C, L, K, p, dtype, bad):
    print(f"case non-finite {bad} {dtype} B{B} C{C} L{L} K{K} p{p}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cpu"); g.manual_seed(77)
    x = torch.randn((B, C, L), generator=g).to(tdt); dy = torch.randn((B, C, L), generator=g).to(tdt)
    w = torch.randn((C, K), generator=g).to(tdt)
    w[w == 0] = 1.0
    b0, c0 = B - 1, 1
    for u in (0, L // 2 + 3, L - 1):
        xb = x.clone(); xb[b0, c0, u] = bad
        dyb = dy.clone(); dyb[b0, c0, u] = bad
        xd, xbd, dyd, dybd, wd = x.cuda(), xb.cuda(), dy.cuda(), dyb.cuda(), w.cuda()
        y0 = binding.dwconv_fwd(xd, wd, p); y1 = binding.dwconv_fwd(xbd, wd, p)
        d0 = binding.dwconv_bwd_input(dyd, wd, p); d1 = binding.dwconv_bwd_input(dybd, wd, p)
        g0 = binding.dwconv_bwd_weight(xd, dyd, K, p); g1 = binding.dwconv_bwd_weight(xbd, dyd, K, p)
        g2 = binding.dwconv_bwd_weight(xd, dybd, K, p)
        torch.cuda.synchronize()
        # fwd: x[u] enters y[t] for t = u - j + p, j = 0..K-1;  dX: dy[u] enters dx[s] for s = u + j - p
        for name, clean, dirty, lo, hi in (("fwd", y0, y1, u + p - K + 1, u + p), ("dx", d0, d1, u - p, u - p + K - 1)):
            lo_d, hi_d = max(lo, 0), min(hi, L - 1)
            same = torch.ones((B, C, L), dtype=torch.bool)
            same[b0, c0, max(lo - SLOP, 0):min(hi + SLOP, L - 1) + 1] = False
            same[b0 - 1, c0, max(L - SLOP, 0):] = False          # (b0 is the last batch: no row after it)
            assert torch.equal(clean.cpu()[same], dirty.cpu()[same]), f"{name}: position {u} reached outside its footprint"
            assert torch.isfinite(clean).all()
            assert not torch.isfinite(dirty[b0, c0, lo_d:hi_d + 1]).any(), f"{name}: position {u} must poison [{lo_d}, {hi_d}]"
        # dW: other channels keep their bits; the coefficients the definition reaches are not finite
        for name, dirty, jlo, jhi in (("dw (x)", g1, u + p - L + 1, u + p), ("dw (dy)", g2, p - u, p - u + L - 1)):
            other = [c for c in range(C) if c != c0]
            assert torch.equal(g0[other], dirty[other]), f"{name}: another channel changed"
            jl, jh = max(jlo, 0), min(jhi, K - 1)
            assert not torch.isfinite(dirty[c0, jl:jh + 1]).any(), f"{name}: coefficients [{jl}, {jh}] must not be finite"


# fp32 operands at the top of their range on the kernels that work on limbs of them (filters of more than six block offsets):
# every output is one product, so it must be what the definition gives - infinite exactly where the product is, never NaN, the
# product itself otherwise, up to the last float, also where the rounding of a first limb goes past it.
# (one chunk of taps and several, one tile per wave and two; windows of offsets and rows cut into virtual rows for dW)
BIG = [(2, 3, 2048, 300, 299), (6, 3, 256, 256, 100), (40, 2, 160, 100, 50), (1, 1, 8192, 8192, 4000), (9, 2, 1024, 700, 0)]
TOP = 2.0 ** 100 * (1 + 2.0 ** -8 + 2.0 ** -9)         # first limb above it, second limb negative
PAIRS = [(TOP, 2.0 ** 100), (-TOP, 2.0 ** 100), (TOP, TOP), (2.0 ** 63 * (2 - 2.0 ** -8), 2.0 ** 63 * (2 - 2.0 ** -8)),
         (2.0 ** 64, 2.0 ** 64 * (1 - 2.0 ** -24)), (3.4028234663852886e38, 1.0), (1.0, -3.4028234663852886e38), (3.4028234663852886e38, 2.0)]


@pytest.mark.parametrize("B,C,L,K,p", BIG)
def test_products_at_the_top_of_the_range(B, C, L, K, p):
    u, j = L // 2, p + 20 if p + 20 < K else p - 20
    for a, b in PAIRS:
        print(f"case top of the range B{B} C{C} L{L} K{K} p{p}: {a!r} x {b!r}", flush=True)
        x = torch.zeros(B, C, L); x[:, :, u] = a
        w = torch.zeros(C, K); w[:, j] = b
        dy = torch.zeros(B, C, L); dy[0, :, u + 3] = b                          # one pair per coefficient
        exp = (torch.tensor([a], dtype=torch.float32).double() * torch.tensor([b], dtype=torch.float32).double()).float()[0]
        want_y = torch.zeros(B, C, L); want_y[:, :, u - j + p] = exp             # y[t] takes x[t + j - p]
        want_dx = torch.zeros(B, C, L); want_dx[:, :, u + j - p] = exp
        want_dw = torch.zeros(C, K)
        if 0 <= p - 3 < K:
            want_dw[:, p - 3] = exp                                              # dw[j] takes dy[u + 3] x[u + 3 + j - p]
        y = binding.dwconv_fwd(x.cuda(), w.cuda(), p).cpu()
        dx = binding.dwconv_bwd_input(x.cuda(), w.cuda(), p).cpu()
        dw = binding.dwconv_bwd_weight(x.cuda(), dy.cuda(), K, p).cpu()
        for name, got, want in (("fwd", y, want_y), ("dx", dx, want_dx), ("dw", dw, want_dw)):
            assert not torch.isnan(got).any(), f"{name}: a NaN from finite inputs"
            assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.equal(got.sign(), want.sign()), name
            # (three limbs per operand, the products of the small ones left out: 2^-24 of the product, and roundings of the sums)
            fin = torch.isfinite(want)
            err = ((got[fin].double() - want[fin].double()).abs() / want[fin].double().abs().clamp_min(1e-30)).max()
            assert float(err) <= 2.0 ** -22, (name, float(err))


# An infinity among operands of one sign: the outputs it enters are that infinity (all taps in one chunk; the zero taps that fill up a
# chunk make the outputs at its edges NaN; the weight gradient on dw_band_kernel: on dw_toep_kernel the zeros beside a chunk of dY make
# NaN of the lags that reach the infinity from there)
@pytest.mark.parametrize("B,C,L,K,p", BIG[:3])
def test_infinity_on_the_limb_kernels(B, C, L, K, p):
    g = torch.Generator(device="cpu"); g.manual_seed(5)
    u = L // 2
    x = torch.rand(B, C, L, generator=g); x[B - 1, 1, u] = float("inf")
    w = torch.rand(C, K, generator=g) + 0.5
    y = binding.dwconv_fwd(x.cuda(), w.cuda(), p).cpu()
    lo, hi = max(u + p - K + 1, 0), min(u + p, L - 1)
    assert (y[B - 1, 1, lo:hi + 1] == float("inf")).all()
    assert torch.isfinite(y[:, [0] + list(range(2, C))]).all()
    dy = torch.rand(B, C, L, generator=g) + 0.5
    dw = binding.dwconv_bwd_weight(x.cuda(), dy.cuda(), K, p).cpu()
    jlo, jhi = max(u + p - L + 1, 0), min(u + p, K - 1)
    assert (dw[1, jlo:jhi + 1] == float("inf")).all()
    x[B - 1, 1, u] = 1.0
    w[1, K // 2] = float("-inf")
    x += 0.5
    y = binding.dwconv_fwd(x.cuda(), w.cuda(), p).cpu()
    t0, t1 = max(p - K // 2, 0), min(L - 1 + p - K // 2, L - 1)
    assert (y[:, 1, t0:t1 + 1] == float("-inf")).all()


# More channels than a grid dimension holds workgroups of 256 threads (2^24), and a filter of more windows of block offsets than its third
# dimension holds (65535), which dw_toep_kernel takes in two launches of its pieces: what is beyond a grid is launched separately.
def test_band_kernels_with_2_to_the_24_channels():
    B, C, L, K, p = 1, (1 << 24) + 3, 9, 97, 40
    tdt = torch.bfloat16
    x = _device_ints((B, C, L), 71, 2, tdt).view(B, C, L)
    dy = _device_ints((B, C, L), 72, 2, tdt).view(B, C, L)
    w = _device_ints((1, C, K), 73, 2, tdt)[0]
    y = binding.dwconv_fwd(x, w, p)
    dx = binding.dwconv_bwd_input(dy, w, p)
    dw = binding.dwconv_bwd_weight(x, dy, K, p)
    torch.cuda.synchronize()
    sel = torch.tensor([0, 1, 5_000_000, (1 << 24) - 257, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, C - 1], device="cuda")
    xs, ds, ws = x[0, sel].double().cpu(), dy[0, sel].double().cpu(), w[sel].double().cpu()
    want_y, want_dx, want_dw = torch.zeros_like(xs), torch.zeros_like(xs), torch.zeros_like(ws)
    for t in range(L):
        for u in range(L):
            j = u - t + p                                    # y[t] takes x[u] w[j]
            want_y[:, t] += xs[:, u] * ws[:, j]
            want_dx[:, u] += ds[:, t] * ws[:, j]
            want_dw[:, j] += ds[:, t] * xs[:, u]
    for name, got, want in (("fwd", y[0, sel], want_y), ("dx", dx[0, sel], want_dx), ("dw", dw[sel], want_dw)):
        assert torch.equal(got.cpu(), want.to(tdt)), name


def test_weight_gradient_with_more_than_65535_windows():
    B, C, K = 1, 1, 23_100_001
    L, p = K, K - 1
    x = _device_ints((B, C, L), 81, 3, torch.float32)
    dy = torch.zeros(B, C, L, device="cuda")
    u = L - 5
    dy[0, 0, u] = 1.0                                        # dw[j] = x[u + j - p]
    want = torch.zeros(C, K, device="cuda")
    want[0, p - u:] = x[0, 0, :u + K - p]
    dw = binding.dwconv_bwd_weight(x, dy, K, p)             # (a workspace of 87 GB that this call does not touch)
    torch.cuda.synchronize()
    assert torch.equal(dw, want)
    torch.cuda.empty_cache()
