"""Selection where its search can go wrong: rows of equal masses (the cut by
index), masses that differ only in their lowest bits (every stage of the
search), more and fewer than 64 blocks with the cut's bits, masses over 1, infinite,
negative and NaN ones, rows that never reach tau, and each width of a row's bit
mask, both rules, against the oracle.  The masses are exact sums in fp64 and in
units of 2^-56, so the sets must be equal, with no exemption."""
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
