"""The calls a program makes through this package's public entry points, as cases to be timed.

A case is one pass of one of five kinds:
  prefill  the attention of one layer over a prompt: sample the layer's permutation, (rotate K,) stochastic attention
  train    forward and backward of one single-path layer
  gated    the gated sum of the stochastic and the sliding-window branch, forward or forward and backward
  layer    the dual-path layer with its gate projections, forward and backward
  decode   one generated token per sequence against the K/V caches
Training and prefill draw a fresh permutation for every pass, as a program does for every layer and step.
Tensors are N(0, 1), gate weights N(0, 1/dm): what the repository's tests and benchmark use.
"""
import math

import torch

from paper_2604_00754_amd import binding as sa

# (query heads, KV heads, head size) of the configurations in synth.WORKLOADS
HEADS = [(32, 8, 128), (32, 4, 128), (12, 12, 64), (16, 16, 64)]


def _case(kind, B, heads, n, w, **more):
    c = {"kind": kind, "B": B, "Hq": heads[0], "Hkv": heads[1], "d": heads[2], "n": n, "w": w, "dtype": "bf16", "per_head_perm": False,
         "rope": False, "backward": False, "gate_per_dim": False, "varlen": False, "len": n}
    c.update(more)
    return c


def listed():
    grouped8, grouped4, small12, wide16 = HEADS
    cases = [
        # the fp32 configuration of the benchmark definition: the smallest call, used to check models
        ("f32_forward_1k", _case("prefill", 1, (2, 2, 64), 1024, 64, dtype="f32", per_head_perm=True)),
        # the same precision in a training step, at a length off every tile edge
        ("f32_train_2k", _case("train", 2, (8, 8, 64), 2039, 128, dtype="f32", backward=True)),
        # a token generated early in a conversation: few rows filled of a cache laid out for 32K
        ("decode_early", _case("decode", 1, grouped8, 32768, 1, len=1100)),
        # the token after the long prompt
        ("decode_32k", _case("decode", 1, grouped8, 32768, 1)),
        # a serving batch whose sequences have different lengths
        ("decode_batch", _case("decode", 16, grouped8, 8192, 1, varlen=True)),
        # an ordinary prompt of odd length, RoPE on original positions
        ("prefill_short", _case("prefill", 1, grouped8, 1531, 512, rope=True)),
        # the headline prefill
        ("prefill_32k", _case("prefill", 1, grouped8, 32768, 512)),
        # the longest prefill: positions no longer fit 16 bits
        ("prefill_128k", _case("prefill", 1, grouped4, 131072, 1024, rope=True)),
        # pre-training forward (evaluation of the loss): one permutation per head
        ("gated_forward_2k", _case("gated", 8, small12, 2048, 128, per_head_perm=True)),
        # pre-training step of the gated sum
        ("gated_train_8k", _case("gated", 4, wide16, 8192, 256, backward=True)),
        # training step of the single path with rotary positions, at a batch of the sequence-length sweep
        ("train_rope_4k", _case("train", 16, wide16, 4096, 256, backward=True, rope=True)),
        # training step of the whole dual-path layer
        ("layer_train_8k", _case("layer", 4, wide16, 8192, 256, backward=True)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


def _draw(rng):
    kind = rng.choice(["prefill", "prefill", "train", "train", "gated", "layer", "decode", "decode", "f32"])
    w = _log_int(rng, 32, 1024)
    if kind == "f32":
        kind = rng.choice(["prefill", "train"])
        return _case(kind, rng.randint(1, 4), rng.choice([(2, 2, 64), (8, 8, 64), (12, 12, 64), (8, 2, 128)]),
                     _log_int(rng, 200, 4096), min(w, 256), dtype="f32", per_head_perm=rng.random() < 0.5, backward=kind == "train")
    if kind == "decode":
        cap = _log_int(rng, 512, 131072)
        B = rng.randint(1, max(1, min(16, 131072 // cap)))
        return _case(kind, B, rng.choice(HEADS), cap, 1, varlen=B > 1, len=_log_int(rng, 64, cap))
    if kind == "prefill":
        return _case(kind, 1, rng.choice(HEADS), _log_int(rng, 200, 131072), w, rope=rng.random() < 0.5)
    n = _log_int(rng, 512, 16384)
    B = rng.randint(1, max(1, min(16, 65536 // n)))
    if kind == "layer":
        return _case(kind, B, rng.choice(HEADS[2:]), n, min(w, 512), backward=True)
    if kind == "gated":
        return _case(kind, B, rng.choice(HEADS[2:]), n, min(w, 512), backward=rng.random() < 0.7, per_head_perm=rng.random() < 0.3,
                     gate_per_dim=rng.random() < 0.3)
    grouped = rng.random() < 0.2  # fine-tuning the long-context shape
    return _case(kind, 1 if grouped else B, HEADS[0] if grouped else rng.choice(HEADS[2:]), n, min(w, 512), backward=True,
                 rope=rng.random() < 0.5)


def _desc(c, window, causal=1):
    dtype = sa.SA_BF16 if c["dtype"] == "bf16" else sa.SA_F32
    return sa.make_desc(c["B"], c["Hq"], c["Hkv"], c["n"], c["d"], c["w"], window, causal, dtype, 0.0, 1,
                        c["Hq"] if c["per_head_perm"] else 1, int(c["gate_per_dim"]), sa.SA_F32)


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    s.case = c
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def normal(*shape, dtype=dt):
        return torch.randn(shape, device=dev, dtype=torch.float32, generator=g).to(dtype)

    def empty(*shape, dtype=dt):
        return torch.empty(shape, device=dev, dtype=dtype)

    def workspace(desc, op):
        return empty(max(sa.sa_workspace_bytes(desc, op), 256), dtype=torch.uint8)

    B, Hq, Hkv, n, d = c["B"], c["Hq"], c["Hkv"], c["n"], c["d"]
    s.sa = _desc(c, sa.SA_WIN_SYM_CIRCULAR)
    if c["kind"] == "decode":
        s.q, s.K, s.V = normal(B, Hq, d), normal(B, Hkv, n, d), normal(B, Hkv, n, d)
        s.Y = torch.empty_like(s.q)
        s.ws = workspace(s.sa, sa.SA_OP_DECODE)
        s.lens = None
        if c["varlen"]:  # the longest sequence has `len` rows, the others from a quarter of that upwards
            lens = torch.randint(max(1, c["len"] // 4), c["len"] + 1, (B,), device=dev, generator=g, dtype=torch.int32)
            lens[seed % B] = c["len"]
            s.lens = lens
        return s

    s.seed = seed
    s.Q, s.K, s.V = normal(B, Hq, n, d), normal(B, Hkv, n, d), normal(B, Hkv, n, d)
    s.perm = empty(1, Hq if c["per_head_perm"] else 1, n, dtype=torch.int32)
    s.ws_perm = workspace(s.sa, sa.SA_OP_SAMPLE_PERM)
    s.Y = torch.empty_like(s.Q)
    if c["rope"]:
        s.table = empty(n, d // 2, 2, dtype=torch.float32)
        sa.sa_rope_table(n, d, 1e6, 0, s.table)
        s.Kr = torch.empty_like(s.K)
    if c["backward"]:
        s.dY = normal(B, Hq, n, d)
        s.dQ, s.dK, s.dV = torch.empty_like(s.Q), torch.empty_like(s.K), torch.empty_like(s.V)
    s.L_sa = empty(B, Hq, n, dtype=torch.float32) if c["backward"] else None
    if c["kind"] in ("gated", "layer"):
        s.swa = _desc(c, sa.SA_WIN_ONE_SIDED)
        s.L_swa = torch.empty_like(s.L_sa) if c["backward"] else None
        keep = c["backward"] or c["kind"] == "layer"
        s.Y_sa, s.Y_swa = (torch.empty_like(s.Q), torch.empty_like(s.Q)) if keep else (None, None)
    if c["kind"] == "gated":
        shape = (B, Hq, n, d) if c["gate_per_dim"] else (B, Hq, n)
        s.g_sa, s.g_swa = normal(*shape, dtype=torch.float32), normal(*shape, dtype=torch.float32)
        s.ws_fwd = workspace(s.sa, sa.SA_OP_GATED_FWD)
        if c["backward"]:
            s.dg_sa, s.dg_swa = torch.empty_like(s.g_sa), torch.empty_like(s.g_swa)
            s.ws = workspace(s.sa, sa.SA_OP_GATED_BWD)
    elif c["kind"] == "layer":
        dm = Hq * d
        s.W_sa, s.W_swa = ((normal(dm, dm, dtype=torch.float32) * dm ** -0.5).to(dt) for _ in range(2))
        s.G_sa, s.G_swa = torch.empty_like(s.Q), torch.empty_like(s.Q)
        s.dW_sa, s.dW_swa = torch.empty_like(s.W_sa), torch.empty_like(s.W_swa)
        s.ws = workspace(s.sa, sa.SA_OP_DUAL_PATH_BWD)
    elif c["backward"]:
        s.ws = workspace(s.sa, sa.SA_OP_BWD_ROPE if c["rope"] else sa.SA_OP_BWD)
    return s


def run(s):
    c = s.case
    if c["kind"] == "decode":
        if s.lens is not None:
            sa.sa_decode_fwd_varlen(s.sa, s.q, s.K, s.V, s.lens, c["len"], s.Y, None, s.ws)
        else:
            sa.sa_decode_fwd(s.sa, s.q, s.K, s.V, c["len"], s.Y, None, s.ws)
        return {"Y": s.Y}

    sa.sa_sample_perm(s.sa, s.seed, 0, s.perm, s.ws_perm)
    out = {"Y": s.Y, "perm": s.perm}
    if c["kind"] == "gated":
        sa.gated_sa_swa_fwd(s.sa, s.swa, s.Q, s.K, s.V, s.perm, s.g_sa, s.g_swa, s.Y, s.Y_sa, s.Y_swa, s.L_sa, s.L_swa, s.ws_fwd)
        if c["backward"]:
            sa.sa_bwd(s.sa, s.swa, s.Q, s.K, s.V, s.perm, s.g_sa, s.g_swa, s.Y_sa, s.Y_swa, s.L_sa, s.L_swa, s.dY,
                      s.dQ, s.dK, s.dV, s.dg_sa, s.dg_swa, s.ws)
            out.update(dg_sa=s.dg_sa, dg_swa=s.dg_swa)
    elif c["kind"] == "layer":
        sa.sa_dual_path_fwd(s.sa, s.swa, s.Q, s.K, s.V, s.perm, s.W_sa, s.W_swa, s.Y, s.Y_sa, s.Y_swa, s.G_sa, s.G_swa,
                            s.L_sa, s.L_swa)
        sa.sa_dual_path_bwd(s.sa, s.swa, s.Q, s.K, s.V, s.perm, s.W_sa, s.W_swa, s.Y_sa, s.Y_swa, s.G_sa, s.G_swa,
                            s.L_sa, s.L_swa, s.dY, s.dQ, s.dK, s.dV, s.dW_sa, s.dW_swa, s.ws)
        out.update(dW_sa=s.dW_sa, dW_swa=s.dW_swa)
    elif c["rope"]:
        sa.sa_rope(s.sa, None, s.K, s.table, None, s.Kr)
        sa.sa_fwd_rope(s.sa, s.Q, s.Kr, s.V, s.perm, s.table, s.Y, s.L_sa)
        if c["backward"]:
            sa.sa_bwd_rope(s.sa, s.Q, s.Kr, s.V, s.perm, s.table, s.Y, s.L_sa, s.dY, s.dQ, s.dK, s.dV, s.ws, dk_unrotated=1)
    else:
        sa.sa_fwd(s.sa, s.Q, s.K, s.V, s.perm, s.Y, s.L_sa)
        if c["backward"]:
            sa.sa_bwd(s.sa, None, s.Q, s.K, s.V, s.perm, None, None, s.Y, None, s.L_sa, None, s.dY, s.dQ, s.dK, s.dV, None, None, s.ws)
    if c["backward"]:
        out.update(dQ=s.dQ, dK=s.dK, dV=s.dV)
    return out


def _visible(n, w):
    """Visible pairs of one head: circular symmetric window on slots and causal on original positions (of every pair of
    tokens in reach exactly one direction is causal), and one-sided window in original order."""
    h = min((w - 1) // 2, (n - 1) // 2)
    m = min(w, n)
    return n * (h + 1), n * m - m * (m - 1) // 2


def work(case):
    """Visible pairs only (4 d flop each forward, 10 d backward), every input read once and every output written once."""
    c = case
    B, Hq, Hkv, n, d = c["B"], c["Hq"], c["Hkv"], c["n"], c["d"]
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "decode":
        rows = B * c["len"] if not c["varlen"] else c["len"] + (B - 1) * c["len"] * 5 // 8  # lengths spread over a quarter to all
        return {"bytes": 2 * rows * Hkv * d * e + 2 * B * Hq * d * e, "flops": 4 * rows * Hq * d}
    q, kv, rows = B * Hq * n * d * e, B * Hkv * n * d * e, B * Hq * n
    dm = Hq * d
    branches = 2 if c["kind"] in ("gated", "layer") else 1
    pairs = (_visible(n, c["w"])[0] + (_visible(n, c["w"])[1] if branches == 2 else 0)) * B * Hq
    nbytes = 2 * q + 2 * kv + 4 * n * (Hq if c["per_head_perm"] else 1)
    flops = 4 * d * pairs
    if c["rope"]:
        nbytes += 4 * n * d
    if c["kind"] == "gated":
        gates = 4 * rows * (d if c["gate_per_dim"] else 1)
        nbytes += 2 * gates * (2 if c["backward"] else 1)
    if c["kind"] == "layer":
        nbytes += 4 * dm * dm * e
        flops += 3 * 2 * 2 * B * n * dm * dm
    if c["backward"]:
        nbytes += 2 * q + 2 * kv
        flops += 10 * d * pairs
    return {"bytes": nbytes, "flops": flops}


def _cost(case):
    """What bounds the draw: seconds at 8 TB/s and 2.5 PFLOP/s (fp32: 0.15)."""
    w = work(case)
    return w["bytes"] / 8e12 + w["flops"] / (2.5e15 if case["dtype"] == "bf16" else 1.5e14)


def tolerance(case):
    """About four times what the paths show against 64-bit softmax attention and its autograd.  bf16: 2.0e-3 (outputs) to
    2.7e-3 (gradients), largest difference 0.064 of the root mean square.  fp32: 1.8e-7 to 5.0e-7, largest 1.1e-5.
    Permutations are whole numbers and stay the same."""
    return {"rel": 1e-2, "max": 0.25} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 5e-5}
