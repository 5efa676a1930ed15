"""A head's results do not depend on what else is in the call: one head alone,
and the same head among many, give the same bits, in every entry point that
works per head.  Calls of few query blocks and of many (more than the GPU's CUs
and, for fp32, more and fewer than whole rounds of its tiles)."""
import pytest
import torch

from oracle import losa_oracle as O

pytestmark = pytest.mark.gpu

# (heads, d, block_q, block_k, N, dtype)
CASES = [(52, 128, 128, 128, 577, "bf16"), (52, 64, 128, 32, 530, "bf16"),
         (60, 64, 64, 64, 570, "bf16"), (40, 128, 64, 32, 545, "bf16"),
         (9, 64, 64, 64, 1024, "f32"), (12, 64, 64, 64, 385, "f32"),
         (10, 128, 128, 128, 511, "f32"), (22, 128, 128, 32, 380, "f32")]


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2608_12032_amd import losa
    return losa


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_head_alone(L, case):
    H, d, Cq, Ck, N, dtype = case
    n_pad = O.padded_len(N, Cq, Ck)
    n_q, n_k = n_pad // Cq, n_pad // Ck
    print(f"[gpu-call-size] H={H} d={d} blocks={Cq}x{Ck} N={N} {dtype}", flush=True)
    g = torch.Generator().manual_seed(500 + CASES.index(case))
    q, k, v = (torch.randn((1, H, n_pad, d), generator=g) for _ in range(3))
    if dtype == "bf16":
        q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    keep = torch.rand((H * n_q, n_k), generator=g) < 0.6
    keep[:, -(-N // Ck):] = False
    rp = torch.zeros(H * n_q + 1, dtype=torch.int32)
    rp[1:] = keep.sum(1).cumsum(0)
    ci = keep.nonzero()[:, 1].int()

    def every(h0, h1):
        x = [t[:, h0:h1].contiguous() for t in (q, k, v)]
        r = rp[h0 * n_q:h1 * n_q + 1]
        o, lse = L.losa_sparse_attn_fwd(*x, N, Cq, Ck, (r - r[0]).int().cuda(),
                                        ci[r[0]:r[-1]].contiguous().cuda(), want_lse=True)
        return (o, lse, *L.losa_construct(*x, N, Cq, Ck, want_lse=True),
                *L.losa_calibrate_mass(*x[:2], N, Cq, Ck),
                *L.losa_calibrate_mass(*x[:2], N, Cq, Ck, two_sweep=True))

    whole = every(0, H)
    for h in (0, H // 2, H - 1):
        for a, b in zip(every(h, h + 1), whole):
            torch.cuda.synchronize()
            assert torch.equal(a[:, 0], b[:, h]), h


@pytest.mark.parametrize("d,C,N", [(128, 128, 640), (64, 64, 576), (64, 128, 1000)])
def test_infinite_value(L, d, C, N):
    """An infinite value of a kept key makes its rows' output column infinite, and
    nothing else, in rows of an even and an odd number of blocks."""
    n_pad = O.padded_len(N, C, C)
    n = n_pad // C
    print(f"[gpu-call-size] infinite value d={d} block={C} N={N}", flush=True)
    g = torch.Generator().manual_seed(70 + d + C)
    q, k, v = (torch.randn((1, 2, n_pad, d), generator=g).bfloat16() for _ in range(3))
    lens = [1 + r % n for r in range(2 * n)]
    rp = torch.tensor([0] + lens).cumsum(0).int().cuda()
    ci = torch.cat([torch.arange(x) for x in lens]).int().cuda()
    want = L.losa_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), N, C, C, rp, ci)
    for j in range(n):                       # one key of block j
        w = v.clone()
        w[:, :, j * C + 7, 5] = float("inf")
        got = L.losa_sparse_attn_fwd(q.cuda(), k.cuda(), w.cuda(), N, C, C, rp, ci)
        torch.cuda.synchronize()
        x = want.clone()
        for r, m in enumerate(lens):
            if m > j:
                h, i = divmod(r, n)
                x[0, h, i * C:min(N, (i + 1) * C), 5] = float("inf")
        assert torch.equal(got[:, :, :N], x[:, :, :N]), j
