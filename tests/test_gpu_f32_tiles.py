"""fp32 kernels at the edges of their tiles.

The attention kernel works on tiles of two groups of 16 rows, 256 at a time, and
on tiles of one for a rest of 128 of the former or fewer (at d = 64 then
throughout); its eight waves share a row's 32-key sub-tiles.  The masses come from block statistics in
the construction step's output (two floats per query and key block, the query
blocks in up to two parts) where there are no more key blocks than floats in a
row of it, and else from a kernel that splits a row's key blocks over
workgroups when the normalisers have room (the caller's lse, or that output)
and sweeps the keys itself when they have none.  Each combination of tile height, head size, block
shape and ragged length, with fewer, as many and more sub-tiles than waves,
against the oracle on every row.  Bars: the fp32 path's (1e-4 on outputs and
masses, 1e-3 on lse)."""
import numpy as np
import pytest
import torch

from oracle import losa_oracle as O

pytestmark = pytest.mark.gpu

# (heads, d, block_q, block_k, N): 16-row tiles, then 32-row ones, both, and more
# key blocks than the statistics have room for
CASES = [(2, 64, 64, 64, 33), (2, 128, 128, 128, 257), (3, 128, 64, 32, 289), (2, 64, 128, 32, 480),
         (12, 64, 64, 64, 385), (10, 128, 128, 128, 511), (9, 128, 128, 32, 487),
         (17, 64, 128, 128, 256), (14, 128, 64, 64, 321), (9, 64, 64, 64, 950),
         (22, 128, 128, 32, 380), (1, 64, 64, 32, 2100), (1, 64, 64, 32, 2040),
         (2, 64, 64, 32, 1020), (2, 64, 64, 32, 1060), (2, 64, 64, 64, 4090)]


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2608_12032_amd import losa
    return losa


def f64(x):
    return x.detach().double().cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_f32_tiles(L, case):
    H, d, Cq, Ck, N = case
    n_pad = O.padded_len(N, Cq, Ck)
    n_q, n_k = n_pad // Cq, n_pad // Ck
    print(f"[gpu-f32-tiles] H={H} d={d} blocks={Cq}x{Ck} N={N}", flush=True)
    g = torch.Generator().manual_seed(700 + CASES.index(case))
    q, k, v = (torch.randn((1, H, n_pad, d), generator=g) * 1.3 for _ in range(3))
    q, k, v = q.cuda(), k.cuda(), v.cuda()     # padding rows hold values too
    scale = 1.0 / np.sqrt(d)
    qh, kh, vh = f64(q), f64(k), f64(v)
    m_ref, l_ref = O.block_masses(qh, kh, N, Cq, Ck, scale)

    mass, lse = L.losa_calibrate_mass(q, k, N, Cq, Ck)
    mass2, none = L.losa_calibrate_mass(q, k, N, Cq, Ck, want_lse=False)
    o, mass3, lse3 = L.losa_construct(q, k, v, N, Cq, Ck, want_lse=True)
    torch.cuda.synchronize()
    assert none is None
    for m in (mass, mass2, mass3):
        assert np.abs(f64(m) - m_ref).max() <= 1e-4
        assert np.abs(f64(m).sum(3) - 1.0).max() <= 1e-5
    for x in (lse, lse3):
        assert np.abs(f64(x)[:, :, :N] - l_ref[:, :, :N]).max() <= 1e-3
        assert np.all(np.isneginf(f64(x)[:, :, N:]))
    d_ref, _ = O.dense_attention(qh, kh, vh, N, scale)
    assert np.abs(f64(o)[:, :, :N] - d_ref[:, :, :N]).max() <= 1e-4
    assert np.all(f64(o)[:, :, N:] == 0)
    x = q.clone()                              # the output over an input
    o2, mass4 = L.losa_construct(x, k, v, N, Cq, Ck, out=x)
    torch.cuda.synchronize()
    assert torch.equal(o2, o) and np.abs(f64(mass4) - m_ref).max() <= 1e-4

    # a support with empty, single-block and full rows, repeated and stray ids
    rng = np.random.default_rng(800 + CASES.index(case))
    rows = []
    for r in range(H * n_q):
        ids = rng.permutation(n_k)[:[0, 1, n_k, max(1, n_k // 2)][r % 4]]
        rows.append(np.concatenate([ids, ids[:1], [-1, n_k + 1]]) if r % 3 == 0 else ids)
    rp = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    s, ls = L.losa_sparse_attn_fwd(q, k, v, N, Cq, Ck, torch.from_numpy(rp).cuda(),
                                   torch.from_numpy(ci).cuda(), want_lse=True)
    torch.cuda.synchronize()
    s_ref, ls_ref = O.sparse_attention(qh, kh, vh, N, Cq, Ck, scale, rp, ci)
    assert np.abs(f64(s)[:, :, :N] - s_ref[:, :, :N]).max() <= 1e-4
    assert np.all(f64(s)[:, :, N:] == 0)
    real = np.isfinite(ls_ref[:, :, :N])
    assert np.array_equal(real, np.isfinite(f64(ls)[:, :, :N]))
    assert np.abs(f64(ls)[:, :, :N][real] - ls_ref[:, :, :N][real]).max() <= 1e-3


@pytest.mark.parametrize("d,C,N,top", [(64, 64, 1000, 8), (64, 64, 4000, 8), (128, 128, 4096, 6)])
def test_construction_mass_rounding(L, d, C, N, top):
    """Masses of peaked rows whose scores (multiples of 1/16, in log2 units) fp32
    holds exactly, so that only exponentials and sums round.  A mass is a mean of
    products of a block's sum, 2^x and 1 / normaliser: a dozen roundings of 2^-24
    at most (a few ulps of the exponentials among them) between a term and the
    result.  Independent and uniform, their root mean square is sqrt(12 / 3) 2^-24
    = 2^-23.  (Kept as an fp32 logarithm of 16 to 64, the sum alone is off by up to
    2^-21 to 2^-19 ln 2.)"""
    n_pad = O.padded_len(N, C, C)
    n_k = n_pad // C
    print(f"[gpu-f32-tiles] mass rounding d={d} block={C} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(17)
    q, k = (torch.randint(-top, top + 1, (1, 2, n_pad, d), generator=g, device="cuda") / 4.0
            for _ in range(2))
    _, mass = L.losa_construct(q, k, k, N, C, C, scale=float(np.log(2.0)))  # ln 2 log2 e = 1 in fp32
    s = (q[:, :, :N].double() @ k.double().transpose(2, 3).contiguous()) * np.log(2.0)
    s[:, :, :, N:] = -np.inf
    p = torch.softmax(s, 3).view(1, 2, N, n_k, C).sum(4)
    p = torch.nn.functional.pad(p, (0, 0, 0, n_pad - N)).view(1, 2, n_k, C, n_k).sum(3)
    want = p / (N - C * torch.arange(n_k, device="cuda")).clamp(max=C)[:, None]
    rel = ((mass.double() - want) / want)[want > 1e-30]
    print(f"[gpu-f32-tiles] relative error {rel.square().mean().sqrt().item():.2e}, "
          f"largest {rel.abs().max().item():.2e}", flush=True)
    assert rel.square().mean().sqrt().item() <= 2.0 ** -23
