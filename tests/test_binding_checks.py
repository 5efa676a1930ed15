"""The Python binding rejects bad tensor arguments before any pointer reaches
the library (which cannot tell a host pointer, a wrong element type or a short
buffer from a valid one).  The host-tensor cases run on the CPU; the rest need
device tensors and are marked gpu (nothing is launched in them)."""
import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def L():
    from paper_2608_12032_amd import losa
    return losa


def test_host_tensors_are_rejected(L):
    q = torch.zeros((1, 2, 128, 128), dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="must live on"):
        L.losa_calibrate_mass(q, q, 100, 128)
    with pytest.raises(ValueError, match="must live on"):
        L.losa_sparse_attn_fwd(q, q, q, 100, 128, 128, torch.zeros(3, dtype=torch.int32),
                               torch.zeros(4, dtype=torch.int32))
    mass = torch.zeros((1, 2, 1, 1))
    with pytest.raises(ValueError, match="must live on"):
        L.losa_select_blocks(mass, 100, 128, 128, 0.99)


def test_sizes_held_in_arrays_and_tensors(L):
    """Whatever ctypes takes as an int is a size: an array, or a tensor that
    holds another value at the next call."""
    def args(n):
        return 2, L.LOSA_DTYPE_BF16, 1, 2, n, 64, 64, 64

    for n in (300, np.int64(300), np.array(300), torch.tensor(300)):
        assert L._need(*args(n)) == L.workspace_bytes(*args(300))
    n = torch.tensor(300)
    for value in (300, 3000):
        n.fill_(value)
        assert L._need(*args(n)) == L.workspace_bytes(*args(value))


@pytest.mark.gpu
def test_device_argument_checks(L):
    dev = "cuda"
    B, H, N, d, C = 1, 2, 200, 128, 128
    Np = L.padded_len(N, C, C)
    q = torch.zeros((B, H, Np, d), dtype=torch.bfloat16, device=dev)
    n_q = Np // C
    rp = torch.zeros(B * H * n_q + 1, dtype=torch.int32, device=dev)
    ci = torch.zeros(B * H * n_q * n_q, dtype=torch.int32, device=dev)
    mass = torch.zeros((B, H, n_q, n_q), dtype=torch.float32, device=dev)
    cases = [
        # N_pad of q does not match N and the block sizes
        (lambda: L.losa_calibrate_mass(q, q, N + 128, C), ValueError, "N_pad"),
        # k of another dtype, v of another shape
        (lambda: L.losa_calibrate_mass(q, q.float(), N, C), TypeError, "k must be"),
        (lambda: L.losa_sparse_attn_fwd(q, q, q[:, :1].contiguous(), N, C, C, rp, ci),
         ValueError, "v must have shape"),
        # a non-contiguous operand
        (lambda: L.losa_sparse_attn_fwd(q, q.transpose(2, 3).contiguous().transpose(2, 3), q,
                                        N, C, C, rp, ci), ValueError, "contiguous"),
        # CSR of the wrong type or too short
        (lambda: L.losa_sparse_attn_fwd(q, q, q, N, C, C, rp.long(), ci), TypeError, "row_ptr"),
        (lambda: L.losa_sparse_attn_fwd(q, q, q, N, C, C, rp[:-1], ci), ValueError, "row_ptr"),
        # output buffers of the wrong shape / a short workspace
        (lambda: L.losa_sparse_attn_fwd(q, q, q, N, C, C, rp, ci, out=q[:, :1].contiguous()),
         ValueError, "out must have shape"),
        (lambda: L.losa_sparse_attn_fwd(q, q, q, N, C, C, rp, ci,
                                        workspace=torch.empty(16, dtype=torch.uint8, device=dev)),
         ValueError, "workspace holds"),
        (lambda: L.losa_calibrate_mass(q, q, N, C, mass=mass[:, :1].contiguous()), ValueError,
         "mass must have shape"),
        # masses whose shape does not match N and the block sizes
        (lambda: L.losa_select_blocks(mass, N + 256, C, C, 0.99), ValueError,
         "mass must have shape"),
        (lambda: L.losa_select_blocks(mass.double(), N, C, C, 0.99), TypeError, "mass must be"),
        (lambda: L.losa_block_recall(mass, N, C, C, rp[:1], ci), ValueError, "row_ptr"),
    ]
    for fn, exc, msg in cases:
        with pytest.raises(exc, match=msg):
            fn()
