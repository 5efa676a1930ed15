"""fp32 calibration with more key blocks per head than the forward's limit of
4,096, which the calibration does not have: masses and normalisers, with and
without room for the latter, on sampled query blocks against 64-bit sums of the
same scores.  Bars: relative 1e-4 on masses (scores below 30 carry at most 30 x
2^-21 of absolute rounding, twice over), 1e-4 on lse."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

# (heads, d, block_q, block_k, N): ragged, one and four blocks past the limit
CASES = [(2, 64, 128, 32, 131_160), (1, 64, 64, 64, 262_150)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_f32_calibration_past_4096_blocks(case):
    from paper_2608_12032_amd import losa as L
    H, d, Cq, Ck, N = case
    n_pad = L.padded_len(N, Cq, Ck)
    n_q, n_k = n_pad // Cq, n_pad // Ck
    assert n_k > 4096
    print(f"[gpu-many-key-blocks] H={H} blocks={Cq}x{Ck} N={N} n_k={n_k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(41)
    q, k = (torch.randn((1, H, n_pad, d), generator=g, device="cuda") for _ in range(2))
    scale = 1.0 / math.sqrt(d)
    mass, lse = L.losa_calibrate_mass(q, k, N, Cq, Ck)
    mass2, _ = L.losa_calibrate_mass(q, k, N, Cq, Ck, want_lse=False)
    torch.cuda.synchronize()
    for m in (mass, mass2):
        assert (m.double().sum(3) - 1.0).abs().max().item() <= 1e-5
    assert torch.isneginf(lse[:, :, N:]).all()
    for h in range(H):
        for i in (0, 1, n_q // 2, n_q - 2, n_q - 1):
            rows = slice(i * Cq, min(N, (i + 1) * Cq))
            s = (q[0, h, rows].double() @ k[0, h].double().t()) * scale
            s[:, N:] = -math.inf
            want = torch.softmax(s, 1).view(-1, n_k, Ck).sum(2).mean(0)
            for m in (mass, mass2):
                assert ((m[0, h, i].double() - want).abs() <= 1e-4 * want).all(), (h, i)
            assert (lse[0, h, rows].double() - torch.logsumexp(s, 1)).abs().max().item() <= 1e-4
