"""The work a program gives this library, as cases that can be timed and compared.

A case is one call (or one layer's short series of calls) through the public
binding `paper_2608_12032_amd.losa`, with buffers and workspaces that such a
program keeps between calls.  `op` says what is called:

  reuse    one later denoising step: the sparse forward over a frozen support
           (entry "workspace": losa_sparse_attn_fwd, "noalloc": the entry point
           without a workspace)
  build    the construction step: dense attention and exact block masses
  track    masses of a later step and the recall of the frozen support on them
           (sweeps: 1 with a workspace, 2 without)
  select   the shortest-prefix rule on given masses (rule "topk": fixed ratio)
  layer    one layer's cycle: construction, selection and `steps` reuse steps

Inputs are the seeded synthetic video tensors of `workload`, T x Hg x Wg tokens.
Supports that a call takes as given are formed here in plain torch from the
construction step's masses; q, k and v of a reuse step have drifted from it.
"""
import math

import torch

from paper_2608_12032_amd import losa
from paper_2608_12032_amd.workload import Workload, cast, drift_, make_state

DEFAULTS = {"op": "reuse", "dtype": "bf16", "B": 1, "H": 12, "d": 128, "T": 21, "Hg": 30, "Wg": 52,
            "bq": 128, "bk": 128, "theta": 0.99, "alpha_lo": 1.5, "alpha_hi": 1.5, "sigma": 0.02,
            "steps": 1, "entry": "workspace", "sweeps": 1, "rule": "mass"}


def listed():
    def case(name, **kw):
        return dict(DEFAULTS, name=name, **kw)

    cog = {"H": 48, "d": 64, "T": 13, "Wg": 45, "alpha_lo": 0.8, "alpha_hi": 2.0}
    hunyuan = {"H": 24, "T": 33, "Hg": 45, "Wg": 80}
    return [
        # the tiny fp32 workload, a whole layer: what a check or a first integration runs
        case("tiny-f32-layer", op="layer", dtype="f32", H=2, d=64, T=4, Hg=16, Wg=16, bq=64,
             bk=64, sigma=0.05, steps=3),
        # one latent frame at 480p (a still, or the first chunk of a streamed video)
        case("frame-reuse", T=1),
        # a short clip with both guidance branches and the paper's 128 x 32 blocks, a whole layer
        case("clip-layer-c32", op="layer", B=2, T=5, bk=32, steps=2),
        # Wan2.1-1.3B, 81 frames at 480p: the step that runs 49 times per layer and sample
        case("wan-reuse"),
        # the same with the paper's rectangular blocks
        case("wan-reuse-c32", bk=32),
        # the same with very local attention and a lower threshold (density sweep's sparsest point)
        case("wan-reuse-local", alpha_lo=3.0, alpha_hi=3.0, theta=0.95),
        # its construction step
        case("wan-build", op="build"),
        # CogVideoX-5B: 48 heads of 64, ragged length
        case("cog-reuse", **cog),
        # recall tracking of the frozen support at a later step
        case("cog-track", op="track", **cog),
        # HunyuanVideo, 129 frames at 720p: the largest
        case("hunyuan-reuse", **hunyuan),
        # its selection with 32-key blocks: 22,296 rows of 3,716 masses
        case("hunyuan-select-c32", op="select", bk=32, **hunyuan),
        # fp32 inputs at an ordinary size, a whole layer, ragged length
        case("clip-f32-layer", op="layer", dtype="f32", H=4, T=3, Hg=29, Wg=51),
    ]


def draw(rng):
    """One more case: sizes over the whole range, in proportion to how often a program makes the call."""
    c = dict(DEFAULTS)
    c["op"] = rng.choice(["reuse"] * 5 + ["build", "build", "layer", "layer", "track", "select"])
    c["dtype"] = rng.choice(["bf16"] * 4 + ["f32"])
    c["d"] = rng.choice([64, 128])
    c["bq"] = rng.choice([128, 128, 64])
    c["bk"] = rng.choice([c["bq"], c["bq"], 32])
    c["B"] = rng.choice([1, 1, 2])
    c["H"] = rng.choice([2, 4, 6, 12, 16, 24, 30, 48])
    c["theta"] = rng.choice([0.95, 0.99, 0.99, 0.999])
    c["alpha_lo"] = c["alpha_hi"] = round(rng.uniform(0.5, 3.0), 2)
    c["sweeps"] = rng.choice([1, 1, 2])
    c["rule"] = rng.choice(["mass", "mass", "topk"])
    # scores of a whole call: 1e6 to 4e10 (fp32 and the one-sweep statistics: less)
    most = 10.0 if c["dtype"] == "f32" and c["op"] != "select" else 10.6
    scores = 10 ** rng.uniform(6.0, most)
    n = min(120_000, max(200, int(math.sqrt(scores / (c["B"] * c["H"])))))
    while -(-n // c["bk"]) > 4000:
        n //= 2
    c["T"] = min(33, max(1, round((n / 1500) * rng.uniform(0.7, 1.4))))
    c["Hg"] = max(3, round(math.sqrt(n / c["T"]) * rng.uniform(0.6, 0.9)))
    c["Wg"] = max(3, n // (c["T"] * c["Hg"]))
    c["steps"] = rng.choice([1, 2, 3]) if c["op"] == "layer" else 1
    if c["op"] == "reuse" and c["B"] * c["H"] * n * c["d"] * 2 < 100 << 20:
        c["entry"] = rng.choice(["workspace", "noalloc"])
    return c


def _workload(c, seed):
    alpha = ("uniform", c["alpha_lo"], c["alpha_hi"])
    return Workload("case", B=c["B"], H=c["H"], d=c["d"], dtype=c["dtype"],
                    grid=(c["T"], c["Hg"], c["Wg"]), block=c["bq"], tau=c["theta"],
                    alpha=c["alpha_lo"] if c["alpha_lo"] == c["alpha_hi"] else alpha, noise=0.5,
                    sigma=c["sigma"], reuse=c["steps"], seed=100_000 + 1000 * seed,
                    block_k=c["bk"] if c["bk"] != c["bq"] else 0)


def _blocks(c):
    n = c["T"] * c["Hg"] * c["Wg"]
    n_pad = -(-n // max(c["bq"], c["bk"])) * max(c["bq"], c["bk"])
    return n, n_pad, n_pad // c["bq"], n_pad // c["bk"]


def _chunks(c, compute, stride=1):
    """Ranges of query blocks whose scores fit about 2 GiB."""
    n, n_pad, n_q, _ = _blocks(c)
    per = max(1, (1 << 31) // (n_pad * (c["bq"] // stride) * torch.finfo(compute).bits // 8))
    return [(i, min(n_q, i + per)) for i in range(0, n_q, per)]


def _scores(c, qh, kh, i0, i1, compute, stride=1):
    """Scaled scores of query blocks i0..i1 of one head, padding keys at -inf, and which rows are real."""
    n, n_pad, _, _ = _blocks(c)
    rows = torch.arange(i0 * c["bq"], i1 * c["bq"], stride, device=qh.device)
    s = (qh[rows].to(compute) @ kh.to(compute).t()) * (1.0 / math.sqrt(c["d"]))
    s[:, n:] = -math.inf
    return s, rows < n


def _masses(c, q, k, compute, stride=1):
    """Exact block masses [B, H, n_q, n_k] over every `stride`-th query."""
    n, n_pad, n_q, n_k = _blocks(c)
    out = torch.zeros(c["B"], c["H"], n_q, n_k, dtype=compute, device=q.device)
    for b in range(c["B"]):
        for h in range(c["H"]):
            for i0, i1 in _chunks(c, compute, stride):
                s, ok = _scores(c, q[b, h], k[b, h], i0, i1, compute, stride)
                p = torch.softmax(s, 1).view(-1, n_k, c["bk"]).sum(2) * ok[:, None]
                count = ok.view(i1 - i0, -1).sum(1).clamp(min=1)
                out[b, h, i0:i1] = p.view(i1 - i0, -1, n_k).sum(1) / count[:, None]
    return out


def _keep(c, mass):
    """Which key blocks each row keeps: the shortest prefix whose mass reaches theta."""
    n, _, n_q, n_k = _blocks(c)
    theta = float(torch.tensor(c["theta"], dtype=torch.float32))
    m, order = torch.sort(mass.reshape(-1, n_k).double(), dim=1, descending=True, stable=True)
    taken = (m.cumsum(1) < theta).sum(1) + 1
    keep = torch.zeros(m.shape, dtype=torch.bool, device=m.device)
    keep.scatter_(1, order, torch.arange(n_k, device=m.device)[None, :] < taken[:, None])
    keep[:, -(-n // c["bk"]):] = False
    return keep


def _frozen(c, q, k):
    """The frozen support of a construction step and the masses it came from (from a sample
    of the queries where the score matrix is very large)."""
    n = _blocks(c)[0]
    stride = 8 if c["B"] * c["H"] * n * n > 3e10 else 1
    mass = _masses(c, q, k, torch.float32, stride)
    return mass, _keep(c, mass)


def _csr(keep):
    row_ptr = torch.zeros(keep.shape[0] + 1, dtype=torch.int32, device=keep.device)
    row_ptr[1:] = keep.sum(1).cumsum(0)
    return row_ptr, keep.nonzero()[:, 1].to(torch.int32).contiguous()


def _inputs(c, seed):
    """q, k, v of the construction step, then of each later step."""
    w = _workload(c, seed)
    state = make_state(w, "cuda")
    steps = [cast(state, w)]
    for t in range(1, c["steps"] + 1 if c["op"] in ("reuse", "track", "layer") else 1):
        steps.append(cast(drift_(state, w, t), w))
    return steps


def _room(which, c, code):
    n = _blocks(c)[0]
    need = losa.workspace_bytes(which, code, c["B"], c["H"], n, 1 if which in (1, 3) else c["d"],
                                c["bq"], c["bk"])
    return torch.empty(need, dtype=torch.uint8, device="cuda") if need else None


def prepare(case, seed):
    c = case
    n, n_pad, n_q, n_k = _blocks(c)
    op, rows = c["op"], c["B"] * c["H"] * n_q
    code = losa.LOSA_DTYPE_F32 if c["dtype"] == "f32" else losa.LOSA_DTYPE_BF16
    steps = _inputs(c, seed)
    st = {"case": c, "N": n, "steps": steps}
    if op != "build":
        st["ws_select"], st["ws_recall"] = _room(1, c, code), _room(3, c, code)
    if op in ("reuse", "track", "select"):
        mass, keep = _frozen(c, *steps[0][:2])
        if op == "select":
            st["mass"], st["k"] = mass, max(1, int(keep.sum()) // rows)
            st["steps"] = None
        else:
            st["row_ptr"], st["col_idx"] = _csr(keep)
            st["steps"] = steps[1:]
        del mass, keep
    if op in ("select", "layer"):
        st["row_ptr"] = torch.full((rows + 1,), -1, dtype=torch.int32, device="cuda")
        st["col_idx"] = torch.full((rows * n_k,), -1, dtype=torch.int32, device="cuda")
    if op in ("build", "layer"):
        st["ws_build"] = _room(4, c, code)
        st["dense"] = torch.empty_like(steps[0][0])
    if op in ("build", "layer", "track"):
        st["mass"] = torch.empty(c["B"], c["H"], n_q, n_k, device="cuda")
    if op == "track":
        st["lse"] = torch.empty(c["B"], c["H"], n_pad, device="cuda")
        st["ws_mass"] = _room(0, c, code) if c["sweeps"] == 1 else None
    if op in ("reuse", "layer"):
        st["out"] = [torch.empty_like(steps[0][0]) for _ in range(c["steps"])]
        st["ws_fwd"] = _room(2, c, code) if c["entry"] == "workspace" else None
    return st


def _reuse(st, i, qkv):
    c = st["case"]
    if c["entry"] == "noalloc":
        return losa.losa_sparse_attn_fwd_noalloc(*qkv, st["N"], c["bq"], c["bk"], st["row_ptr"],
                                                 st["col_idx"], out=st["out"][i])
    return losa.losa_sparse_attn_fwd(*qkv, st["N"], c["bq"], c["bk"], st["row_ptr"], st["col_idx"],
                                     out=st["out"][i], workspace=st["ws_fwd"])


def run(state):
    st, c = state, state["case"]
    n, bq, bk, op = st["N"], c["bq"], c["bk"], c["op"]
    if op == "reuse":
        return {"out": _reuse(st, 0, st["steps"][0])}
    if op == "build":
        o, mass = losa.losa_construct(*st["steps"][0], n, bq, bk, out=st["dense"], mass=st["mass"],
                                      workspace=st["ws_build"])
        return {"dense": o, "mass": mass}
    if op == "track":
        q, k, _ = st["steps"][0]
        mass, lse = losa.losa_calibrate_mass(q, k, n, bq, bk, mass=st["mass"], lse=st["lse"],
                                             workspace=st["ws_mass"], two_sweep=c["sweeps"] == 2)
        rows, heads = losa.losa_block_recall(mass, n, bq, bk, st["row_ptr"], st["col_idx"],
                                             workspace=st["ws_recall"])
        return {"mass": mass, "lse": lse, "recall_rows": rows, "recall_heads": heads}
    if op == "select":
        kept = {"row_ptr": st["row_ptr"], "col_idx": st["col_idx"], "workspace": st["ws_select"]}
        if c["rule"] == "topk":
            row_ptr, col_idx = losa.losa_select_blocks_topk(st["mass"], n, bq, bk, st["k"], **kept)
        else:
            row_ptr, col_idx = losa.losa_select_blocks(st["mass"], n, bq, bk, c["theta"], **kept)
        return {"row_ptr": row_ptr, "col_idx": col_idx}
    o, mass = losa.losa_construct(*st["steps"][0], n, bq, bk, out=st["dense"], mass=st["mass"],
                                  workspace=st["ws_build"])
    losa.losa_select_blocks(mass, n, bq, bk, c["theta"], row_ptr=st["row_ptr"],
                            col_idx=st["col_idx"], workspace=st["ws_select"])
    return {"dense": o, "mass": mass,
            "reuse": [_reuse(st, i, qkv) for i, qkv in enumerate(st["steps"][1:])]}


def work(case):
    """Each input read once, each output written once; the products over the kept blocks."""
    c = case
    n, n_pad, n_q, n_k = _blocks(c)
    bh, el = c["B"] * c["H"], 4 if c["dtype"] == "f32" else 2
    tensor, mass, lse = bh * n_pad * c["d"] * el, 4 * bh * n_q * n_k, 4 * bh * n_pad
    dense = 4 * bh * n * n * c["d"]
    if c["op"] == "build":
        return {"bytes": 4 * tensor + mass, "flops": dense}
    q, k = _inputs(dict(c, op="build"), 1)[0][:2]
    keep = _frozen(c, q, k)[1]
    csr = 4 * (bh * n_q + 1 + int(keep.sum()))
    size_q = torch.full((n_q,), c["bq"], device="cuda")
    size_q[-1] -= n_pad - n
    size_k = (n - c["bk"] * torch.arange(n_k, device="cuda")).clamp(0, c["bk"])
    pairs = float((keep.view(bh, n_q, n_k) * size_q[:, None].double() * size_k.double()).sum())
    sparse = 4 * c["d"] * pairs
    if c["op"] == "select":
        return {"bytes": mass + csr, "flops": 0}
    if c["op"] == "track":
        return {"bytes": 2 * tensor + mass + lse + csr + 4 * bh * (n_q + 1), "flops": dense / 2}
    one = {"bytes": 4 * tensor + csr, "flops": sparse}
    if c["op"] == "reuse":
        return one
    return {"bytes": 4 * tensor + mass + csr + c["steps"] * one["bytes"],
            "flops": dense + c["steps"] * one["flops"]}


def tolerance(case):
    """Selection from given masses is exact.  fp32: rounding of scores and sums (measured 3e-6 to
    6e-6 against 64 bits on outputs, up to 1e-6 on masses).  bf16: half an ulp of the output and of
    each probability that enters P V (measured 2.3e-3).  Four times what was measured."""
    if case["op"] == "select":
        return "exact"
    if case["op"] == "track":
        return {"rel": 1e-5, "max": 1e-3}
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 2e-3}
    return {"rel": 1e-2, "max": 0.1}


def _attention(c, qkv, keep=None):
    """Attention in 64 bits over the kept blocks (all valid keys without `keep`)."""
    n, n_pad, n_q, n_k = _blocks(c)
    q, k, v = qkv
    out = torch.zeros(q.shape, dtype=torch.float64, device=q.device)
    for b in range(c["B"]):
        for h in range(c["H"]):
            for i0, i1 in _chunks(c, torch.float64):
                s, ok = _scores(c, q[b, h], k[b, h], i0, i1, torch.float64)
                if keep is not None:
                    r0 = (b * c["H"] + h) * n_q
                    row = keep[r0 + i0:r0 + i1].repeat_interleave(c["bk"], 1)
                    s.view(i1 - i0, c["bq"], n_pad).masked_fill_(~row[:, None, :], -math.inf)
                p = torch.softmax(s, 1).nan_to_num_(0.0)
                out[b, h, i0 * c["bq"]:i1 * c["bq"]] = (p @ v[b, h].double()) * ok[:, None]
    return out


def exact(case, seed):
    """What `run` returns, in 64 bits with plain torch."""
    c = case
    n, n_pad, n_q, n_k = _blocks(c)
    if c["op"] == "select" or c["B"] * c["H"] * n * n * (1 + c["steps"]) > 6e10:
        return None
    steps = _inputs(c, seed)
    if c["op"] == "reuse":
        return {"out": _attention(c, steps[1], _frozen(c, *steps[0][:2])[1])}
    if c["op"] == "track":
        q, k = steps[1][:2]
        keep = _frozen(c, *steps[0][:2])[1]
        mass = _masses(c, q, k, torch.float64)
        lse = torch.full((c["B"], c["H"], n_pad), -math.inf, dtype=torch.float64, device="cuda")
        for b in range(c["B"]):
            for h in range(c["H"]):
                for i0, i1 in _chunks(c, torch.float64):
                    s, ok = _scores(c, q[b, h], k[b, h], i0, i1, torch.float64)
                    lse[b, h, i0 * c["bq"]:i1 * c["bq"]] = torch.where(ok, torch.logsumexp(s, 1),
                                                                       -math.inf)
        kept = mass.view(-1, n_k) * keep
        rows_valid = (n - c["bq"] * torch.arange(n_q, device="cuda")).clamp(0, c["bq"]).double()
        num = (kept.sum(1).view(c["B"], c["H"], n_q) * rows_valid).sum(2)
        den = (mass.sum(3) * rows_valid).sum(2)
        return {"mass": mass, "lse": lse, "recall_rows": kept.sum(1), "recall_heads": num / den}
    mass = _masses(c, *steps[0][:2], torch.float64)
    dense = _attention(c, steps[0])
    if c["op"] == "build":
        return {"dense": dense, "mass": mass}
    keep = _keep(c, mass)
    return {"dense": dense, "mass": mass, "reuse": [_attention(c, x, keep) for x in steps[1:]]}
