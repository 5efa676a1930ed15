"""Selection where its search can go wrong: rows of equal masses (the cut by
index), masses that differ only in their lowest bits (every stage of the
search), more and fewer than 64 blocks with the cut's bits, masses over 1, infinite,
negative and NaN ones, rows that never reach tau, and each width of a row's bit
mask, both rules, against the oracle.  The masses are exact sums in fp64 and in
units of 2^-56 of the threshold's power of two, so the sets must be equal, with
no exemption.  Then masses and thresholds scaled down together."""
from fractions import Fraction

import numpy as np
import pytest
import torch

from oracle import losa_oracle as O

pytestmark = pytest.mark.gpu

N_K = [1, 7, 8, 63, 64, 65, 256, 257, 700, 1024, 1025, 4096]
KINDS = ["equal", "low-bits", "two-levels", "large", "corrupt", "short", "random"]


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2608_12032_amd import losa
    return losa


def masses(kind, rows, n_k, rng):
    m = np.zeros((rows, n_k), np.float32)
    for r in range(rows):
        if kind == "equal":            # multiples of 2^-20: every sum is exact
            m[r] = max(1, (1 << 20) // n_k) * 2.0 ** -20
        elif kind == "low-bits":       # one value and its next neighbours
            x = np.float32(max(1, (1 << 14) // n_k) * 2.0 ** -14)
            m[r] = x * (1 + rng.integers(0, 4, n_k) * 2.0 ** -22).astype(np.float32)
        elif kind == "two-levels":     # a few heavy blocks, the rest alike
            m[r] = 2.0 ** -14
            m[r, rng.permutation(n_k)[:max(1, n_k // 9)]] = 2.0 ** -5
        elif kind == "large":          # not normalised
            m[r] = rng.choice([0.25, 1.0, 3.0, 1e30, np.inf], n_k, p=[.8, .1, .05, .03, .02])
        elif kind == "corrupt":
            m[r] = 2.0 ** -9
            m[r, rng.random(n_k) < 0.2] = np.nan
            m[r, rng.random(n_k) < 0.2] = -3.0
            m[r, rng.random(n_k) < 0.3] = 0.0
        elif kind == "short":          # sums to half of the smallest tau used
            m[r] = 2.0 ** -2 / n_k if n_k & (n_k - 1) == 0 else 2.0 ** -16
        else:                          # exponents over 20 octaves, 8-bit mantissas
            m[r] = rng.integers(128, 256, n_k) * 2.0 ** -rng.integers(12, 32, n_k).astype(np.float64)
    return m


@pytest.mark.parametrize("kind", KINDS)
def test_selection_search(L, kind):
    rng = np.random.default_rng(40 + KINDS.index(kind))
    for n_k in N_K:
        # 128 x 32 blocks (64 x 64 for counts that are no multiple of four)
        Cq, Ck = (128, 32) if n_k % 4 == 0 else (64, 64)
        N = n_k * Ck - (5 if n_k > 1 else 0)
        n_q, H = n_k * Ck // Cq, 1 if n_k > 1000 else 2
        print(f"[gpu-select-search] {kind} n_k={n_k} rows={H * n_q}", flush=True)
        m = masses(kind, H * n_q, n_k, rng)
        mt = torch.from_numpy(m.reshape(1, H, n_q, n_k)).cuda()
        m64 = np.where(m > 0, m, 0).astype(np.float64).reshape(1, H, n_q, n_k)
        for tau in (0.5, 0.75, 1.0 - 2.0 ** -10):
            rp, ci = L.losa_select_blocks(mt, N, Cq, Ck, tau)
            got = rp.cpu().numpy()
            want_rp, want_ci, _ = O.select_blocks(np.minimum(m64, 2.0 ** 100), N, Cq, Ck, tau)
            assert np.array_equal(got, want_rp), (n_k, tau)
            assert np.array_equal(ci[:got[-1]].cpu().numpy(), want_ci), (n_k, tau)
        for k in (1, max(1, n_k // 3), n_k + 3):
            rp, ci = L.losa_select_blocks_topk(mt, N, Cq, Ck, k)
            got = rp.cpu().numpy()
            want_rp, want_ci, _ = O.select_blocks_topk(m64, N, Cq, Ck, k)
            assert np.array_equal(got, want_rp), (n_k, k)
            assert np.array_equal(ci[:got[-1]].cpu().numpy(), want_ci), (n_k, k)


@pytest.mark.parametrize("kind", [k for k in KINDS if k != "large"])
@pytest.mark.parametrize("down", [20, 47, 100])
def test_small_masses_and_threshold(L, kind, down):
    """Masses that do not sum to one, and a threshold as small as they are: the
    rule only compares sums, so masses and threshold scaled by a power of two
    keep the same sets."""
    rng = np.random.default_rng(60 + KINDS.index(kind))
    for n_k in (7, 64, 257, 1025, 4096):
        Cq, Ck = (128, 32) if n_k % 4 == 0 else (64, 64)
        N = n_k * Ck - 5
        n_q = n_k * Ck // Cq
        print(f"[gpu-select-search] small {kind} 2^-{down} n_k={n_k} rows={n_q}", flush=True)
        m = np.ldexp(masses(kind, n_q, n_k, rng), -down).astype(np.float32)
        mt = torch.from_numpy(m.reshape(1, 1, n_q, n_k)).cuda()
        m64 = np.where(m > 0, m, 0).astype(np.float64).reshape(1, 1, n_q, n_k)
        for tau in (0.5, 0.75, 1.0 - 2.0 ** -10):
            t = float(np.ldexp(np.float32(tau), -down))
            rp, ci = L.losa_select_blocks(mt, N, Cq, Ck, t)
            got = rp.cpu().numpy()
            want_rp, want_ci, _ = O.select_blocks(m64, N, Cq, Ck, t)
            assert np.array_equal(got, want_rp), (n_k, tau)
            assert np.array_equal(ci[:got[-1]].cpu().numpy(), want_ci), (n_k, tau)


# (blocks, mass of each, tau): the first ceil(tau / mass) of them, by whole-number
# arithmetic on the fp32 values; the last one is below the normal range
EQUAL = [(1000, 1e-18, 5e-16), (4096, 1e-17, 1e-14), (1000, 1e-16, 5e-14), (48, 1e-18, 1.5e-17),
         (4096, 1e-12, 1e-9), (1024, 1e-10, 1e-7), (3, 1e-38, 1.5e-38), (1000, 2e-45, 1e-42)]


@pytest.mark.parametrize("n_k,m,tau", EQUAL)
def test_equal_tiny_masses(L, n_k, m, tau):
    m, tau = Fraction(float(np.float32(m))), Fraction(float(np.float32(tau)))
    want = -(-tau // m)
    assert 0 < want < n_k
    Cq, Ck = (128, 32) if n_k % 4 == 0 else (64, 64)
    rows = n_k * Ck // Cq
    mt = torch.full((1, 1, rows, n_k), float(m), dtype=torch.float32, device="cuda")
    rp, ci = L.losa_select_blocks(mt, n_k * Ck, Cq, Ck, float(tau))
    torch.cuda.synchronize()
    assert torch.equal(rp.cpu(), (torch.arange(rows + 1) * want).int())
    assert torch.equal(ci[:rows * want].cpu(), torch.arange(want, dtype=torch.int32).repeat(rows))
