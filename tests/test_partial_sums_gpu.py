"""Rounding of the fp32 sums of the weight gradient of long filters (Sec. IV-C/D, the intermediate tensor) before anything else is rounded."""
import numpy as np
import pytest
import torch

from paper_2604_25422_amd import binding

pytestmark = pytest.mark.gpu


# dw_toep_kernel, one tile of lags per workgroup and two, one batch entry and several, one slice and several.  An element of a slice sums
# N = B L / 64 products of the instruction on each of four waves, in chains of n of them that are added to a total of M = N / n: with random
# operands an addition at the size s of its sum errs by up to 2^-24 s, 2^-24 s / sqrt(3) in the root mean square, and the sums grow with
# the root of their length, so the relative error is 2^-24 sqrt((n + M) / 6).  Chains may be twice as long as sqrt(N), the best
# (one chain of all N: two to three times as much).
@pytest.mark.parametrize("B,C,L,K,p", [(8, 256, 8192, 8192, 8191), (91, 96, 1810, 1810, 1809), (32, 256, 4096, 1024, 1023), (1, 224, 5952, 5952, 5951), (1, 544, 6988, 6988, 3494),
                                       (12, 355, 1832, 1832, 916)])
def test_bf16_sums_of_long_filters(B, C, L, K, p):
    print(f"case partial sums bf16 B{B} C{C} L{L} K{K} p{p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(11)
    x, dy = (torch.randn(B, C, L, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    S = binding.dwconv_bwd_weight_slices(B, C, L, K, p, binding.BF16)
    part = binding.dwconv_bwd_weight_partial(x, dy, K, p)[:4 * S * C * K].view(torch.float32).view(S, C, K)
    sel = [0, C // 2, C - 1]
    got = part[:, sel].double().sum(0).cpu().numpy()
    xs, ds = x[:, sel].double().cpu().numpy(), dy[:, sel].double().cpu().numpy()
    n = 1 << (2 * L - 1).bit_length()
    corr = np.fft.irfft((np.fft.rfft(xs, n) * np.conj(np.fft.rfft(ds, n))).sum(0), n)          # lag o at o mod n
    lo, hi = max(0, p - L + 1), min(K, p + L)
    ref = np.zeros((len(sel), K))
    ref[:, lo:hi] = corr[:, (np.arange(lo, hi) - p) % n]
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    bound = 2.0 ** -24 * (2.5 * (B * L / 64) ** 0.5 / 6) ** 0.5
    print(f"error {err:.3e}, bound {bound:.3e}", flush=True)
    assert err <= bound
