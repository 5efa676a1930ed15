"""bf16 forward in calls of few and of many query blocks (fewer and more than the
GPU's CUs, and both sides of the rule that gives a call a row order).
Rows with no, one, an odd and an even number of blocks, repeated and stray ids,
32-key blocks that do not fill the pipeline's passes, a ragged last block; the
construction step equals the sparse forward over a full support bitwise,
whether its heads are worked through together or one at a time.  Bars: the bf16 path's."""
import numpy as np
import pytest
import torch

from oracle import losa_oracle as O

pytestmark = pytest.mark.gpu

# (heads, d, block_q, block_k, N): a few rows, and just below and above 256 (512
# at d = 64 with 64-row blocks), at fewer and more than 512 padded keys
CASES = [(2, 128, 128, 128, 385), (2, 128, 128, 128, 384), (51, 128, 128, 128, 577),
         (52, 128, 128, 128, 577), (51, 64, 128, 128, 600), (52, 64, 128, 128, 600),
         (2, 128, 128, 32, 490), (52, 64, 128, 32, 530), (28, 128, 64, 64, 570),
         (29, 128, 64, 64, 570), (56, 64, 64, 32, 545), (57, 64, 64, 32, 545),
         (3, 128, 64, 32, 640)]


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2608_12032_amd import losa
    return losa


def f64(x):
    return x.detach().double().cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_key_split(L, case):
    H, d, Cq, Ck, N = case
    n_pad = O.padded_len(N, Cq, Ck)
    n_q, n_k = n_pad // Cq, n_pad // Ck
    n_kv = -(-N // Ck)
    print(f"[gpu-key-split] H={H} d={d} blocks={Cq}x{Ck} N={N} rows={H * n_q}", flush=True)
    g = torch.Generator().manual_seed(300 + CASES.index(case))
    q, k, v = ((torch.randn((1, H, n_pad, d), generator=g) * 1.3).bfloat16().cuda()
               for _ in range(3))              # padding rows hold values too
    scale = 1.0 / np.sqrt(d)
    rng = np.random.default_rng(310 + CASES.index(case))
    rows = []
    for r in range(H * n_q):
        ids = rng.permutation(n_kv)[:[0, 1, 2, 3, n_kv, max(1, n_kv // 2)][r % 6]]
        rows.append(np.concatenate([ids, ids[:1], [-1, n_k + 1]]) if r % 5 == 0 else ids)
    rp = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    o, lse = L.losa_sparse_attn_fwd(q, k, v, N, Cq, Ck, torch.from_numpy(rp).cuda(),
                                    torch.from_numpy(ci).cuda(), want_lse=True)
    torch.cuda.synchronize()
    some = np.unique(np.concatenate([np.arange(min(12, H * n_q)), [H * n_q - 1],
                                     rng.integers(0, H * n_q, 30)]))
    ref, lref = O.sparse_attention(f64(q), f64(k), f64(v), N, Cq, Ck, scale, rp, ci,
                                   rows_subset=some)
    errs = []
    for r in some:
        h, i = divmod(int(r), n_q)
        real = slice(i * Cq, min(N, (i + 1) * Cq))
        errs.append(np.abs(f64(o[0, h, real]) - ref[0, h, real]).ravel())
        lg, lr = f64(lse[0, h, real]), lref[0, h, real]
        assert np.array_equal(np.isfinite(lg), np.isfinite(lr))
        assert np.all(np.abs(lg[np.isfinite(lr)] - lr[np.isfinite(lr)]) <= 1e-3)
    errs = np.concatenate(errs)
    assert errs.max() <= 2e-2 and errs.mean() <= 2e-3, (errs.max(), errs.mean())
    assert np.all(f64(o[0, :, N:]) == 0) and np.all(np.isneginf(f64(lse[0, :, N:])))

    full = torch.arange(n_kv, dtype=torch.int32).repeat(H * n_q).cuda()
    frp = (torch.arange(H * n_q + 1) * n_kv).int().cuda()
    sparse = L.losa_sparse_attn_fwd(q, k, v, N, Cq, Ck, frp, full)
    dense, mass = L.losa_construct(q, k, v, N, Cq, Ck)
    one = torch.empty(L.workspace_bytes(4, L.LOSA_DTYPE_BF16, 1, 1, N, d, Cq, Ck),
                      dtype=torch.uint8, device="cuda")
    dense1, mass1 = L.losa_construct(q, k, v, N, Cq, Ck, workspace=one)  # a head at a time
    torch.cuda.synchronize()
    assert torch.equal(dense, sparse)
    assert torch.equal(dense, dense1) and torch.equal(mass, mass1)
    m_ref, _ = O.block_masses(f64(q[:, :2]), f64(k[:, :2]), N, Cq, Ck, scale)
    assert np.abs(f64(mass[:, :2]) - m_ref).max() <= 1e-4


@pytest.mark.parametrize("H,N", [(2, 600), (40, 1000)])   # few rows and many
def test_output_over_v(L, H, N):
    """o written over v gives what separate buffers give, in both calls."""
    n_pad = O.padded_len(N, 128, 128)
    n = n_pad // 128
    g = torch.Generator().manual_seed(77)
    q, k, v = (torch.randn((1, H, n_pad, 128), generator=g).bfloat16().cuda() for _ in range(3))
    rp = (torch.arange(H * n + 1) * n).int().cuda()
    ci = torch.arange(n, dtype=torch.int32).repeat(H * n).cuda()
    want = L.losa_sparse_attn_fwd(q, k, v, N, 128, 128, rp, ci)
    for call in (lambda x: L.losa_sparse_attn_fwd(q, k, x, N, 128, 128, rp, ci, out=x),
                 lambda x: L.losa_sparse_attn_fwd_noalloc(q, k, x, N, 128, 128, rp, ci, out=x),
                 lambda x: L.losa_construct(q, k, x, N, 128, 128, out=x)[0]):
        x = v.clone()
        got = call(x)
        torch.cuda.synchronize()
        assert got.data_ptr() == x.data_ptr() and torch.equal(got, want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("H,N", [(2, 600), (40, 1000)])   # few rows and many
def test_output_over_q(L, H, N, dtype):
    """o written over q gives what separate buffers give, in every forward call."""
    n_pad = O.padded_len(N, 128, 128)
    n = n_pad // 128
    print(f"[gpu-key-split] o over q, {H} heads, {dtype}", flush=True)
    g = torch.Generator().manual_seed(78)
    q, k, v = (torch.randn((1, H, n_pad, 128), generator=g).to(dtype).cuda() for _ in range(3))
    rp = (torch.arange(H * n + 1) * n).int().cuda()
    ci = torch.arange(n, dtype=torch.int32).repeat(H * n).cuda()
    want = L.losa_sparse_attn_fwd(q, k, v, N, 128, 128, rp, ci)
    for call in (lambda x: L.losa_sparse_attn_fwd(x, k, v, N, 128, 128, rp, ci, out=x),
                 lambda x: L.losa_sparse_attn_fwd_noalloc(x, k, v, N, 128, 128, rp, ci, out=x),
                 lambda x: L.losa_construct(x, k, v, N, 128, 128, out=x)[0]):
        x = q.clone()
        got = call(x)
        torch.cuda.synchronize()
        assert got.data_ptr() == x.data_ptr() and torch.equal(got, want)


@pytest.mark.parametrize("H,Cq,Ck,N,d", [(48, 128, 128, 1000, 128), (64, 64, 64, 500, 128),
                                         (32, 128, 128, 1000, 128), (32, 64, 32, 500, 64)])
def test_order_rule(L, H, Cq, Ck, N, d):
    """The largest call whose rows run in id order (64-row blocks at d = 128: 512
    rows, else 256; or one that has a dispatch order like the next) against the first
    H heads of one head more, which gets an order: the same bits."""
    n_pad = O.padded_len(N, Cq, Ck)
    n_q, n_k = n_pad // Cq, n_pad // Ck
    print(f"[gpu-key-split] order rule: {H * n_q} rows", flush=True)
    g = torch.Generator().manual_seed(90 + H)
    q, k, v = (torch.randn((1, H + 1, n_pad, d), generator=g).bfloat16().cuda() for _ in range(3))
    keep = torch.rand(((H + 1) * n_q, n_k), generator=g) < 0.5
    rp = torch.zeros((H + 1) * n_q + 1, dtype=torch.int32)
    rp[1:] = keep.sum(1).cumsum(0)
    ci = keep.nonzero()[:, 1].int().cuda()
    got = []
    for h in (H, H + 1):
        o, lse = L.losa_sparse_attn_fwd(*(x[:, :h].contiguous() for x in (q, k, v)), N, Cq, Ck,
                                        rp[:h * n_q + 1].cuda(), ci, want_lse=True)
        got.append((o[:, :H], lse[:, :H]))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
