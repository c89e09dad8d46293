"""GPU parity of sa_gate_proj_fwd (Eq. 6 + Eq. 5: gate projections over the model dimension and the
gated sum) against the fp64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def run_case(B, H, n, d, seed, dual=True, w_scale=None, want_gates=True):
    from oracle import binding as orc
    from paper_2604_00754_amd import binding as sa
    from paper_2604_00754_amd import synth
    dm = H * d
    print(f"case gate_proj B{B} H{H} n{n} d{d} dm{dm} dual={dual}", flush=True)
    rng = np.random.default_rng(synth.BASE_SEED + seed)
    r16 = lambda a: synth.round_to_bf16(a.astype(np.float32))
    Ysa = r16(rng.standard_normal((B, H, n, d)))
    Yswa = r16(rng.standard_normal((B, H, n, d)))
    s = w_scale if w_scale is not None else 1.0 / np.sqrt(dm)   # logits ~ N(0, 1)
    Wsa, Wswa = r16(rng.standard_normal((dm, dm)) * s), r16(rng.standard_normal((dm, dm)) * s)
    c = orc.desc(B, H, H, n, d, 4)
    if dual:
        Yr, La, Lb = orc.gate_proj_fwd(c, Ysa, Yswa, Wsa, Wswa, want_logits=True)
    else:
        Yr, La, Lb = orc.gate_proj_fwd(c, Ysa, None, Wsa, None, want_logits=True)
    dev = lambda a: U.to_dev(a, "bf16")
    tYsa, tWsa = dev(Ysa), dev(Wsa)
    tYswa, tWswa = (dev(Yswa), dev(Wswa)) if dual else (None, None)
    Y = torch.full_like(tYsa, float("nan"))
    Ga = torch.full_like(tYsa, float("nan")) if want_gates else None
    Gb = torch.full_like(tYsa, float("nan")) if want_gates and dual else None
    desc = sa.make_desc(B, H, H, n, d, 4)
    sa.sa_gate_proj_fwd(desc, tYsa, tYswa, tWsa, tWswa, Y, Ga, Gb)
    torch.cuda.synchronize()
    U.assert_close(U.to_np64(Y), Yr, "bf16", "Y")
    if want_gates:
        sig = lambda x: 1 / (1 + np.exp(-x))
        U.assert_close(U.to_np64(Ga), sig(La), "bf16", "G_sa")
        if dual:
            U.assert_close(U.to_np64(Gb), sig(Lb), "bf16", "G_swa")


@pytest.mark.parametrize("d,H", [(64, 2), (64, 6), (128, 1), (128, 3)])
def test_gate_proj_dual_path(d, H):
    run_case(2, H, 300, d, seed=d + H)          # ragged token tiles (300 = 2 * 128 + 44)


def test_gate_proj_single_path_and_no_gate_outputs():
    run_case(1, 4, 129, 64, seed=7, dual=False)
    run_case(1, 2, 64, 128, seed=8, dual=True, want_gates=False)


def test_gate_proj_saturating_and_zero_weights():
    run_case(1, 2, 200, 64, seed=9, w_scale=2.0)    # |logits| ~ 20: gates saturate at 0 / 1
    run_case(1, 2, 200, 64, seed=10, w_scale=0.0)   # both gates exactly 1/2


def test_gate_proj_pretraining_width():
    """d_model = 1024 (16 heads of 64) as in the paper's pre-training setup (App. B, App. C), a few token tiles."""
    run_case(1, 16, 1000, 64, seed=11)


def test_gate_proj_rejects_unsupported():
    from paper_2604_00754_amd import binding as sa
    t = torch.zeros((1, 1, 8, 64), device=U.DEV, dtype=torch.bfloat16)
    w = torch.zeros((64, 64), device=U.DEV, dtype=torch.bfloat16)
    with pytest.raises(sa.SaError) as e:  # dm = 64 is not a multiple of 128
        sa.sa_gate_proj_fwd(sa.make_desc(1, 1, 1, 8, 64, 4), t, t, w, w, torch.empty_like(t))
    assert e.value.status == sa.SA_ERR_UNSUPPORTED
    with pytest.raises(sa.SaError) as e:  # second branch given without its weight
        t2 = torch.zeros((1, 2, 8, 64), device=U.DEV, dtype=torch.bfloat16)
        w2 = torch.zeros((128, 128), device=U.DEV, dtype=torch.bfloat16)
        sa.sa_gate_proj_fwd(sa.make_desc(1, 2, 2, 8, 64, 4), t2, t2, w2, None, torch.empty_like(t2))
    assert e.value.status == sa.SA_ERR_NULL


def run_bwd_case(B, H, n, d, seed, dual=True):
    """Forward on the GPU (to get the gate values it saves), then the backward, against the fp64
    gradient of the oracle.  The oracle recomputes g_x in fp64; the GPU uses its bf16-rounded copy."""
    from oracle import binding as orc
    from paper_2604_00754_amd import binding as sa
    from paper_2604_00754_amd import synth
    dm = H * d
    print(f"case gate_proj_bwd B{B} H{H} n{n} d{d} dm{dm} dual={dual}", flush=True)
    rng = np.random.default_rng(synth.BASE_SEED + 100 + seed)
    r16 = lambda a: synth.round_to_bf16(a.astype(np.float32))
    Ysa, Yswa, dY = (r16(rng.standard_normal((B, H, n, d))) for _ in range(3))
    Wsa, Wswa = (r16(rng.standard_normal((dm, dm)) / np.sqrt(dm)) for _ in range(2))
    c = orc.desc(B, H, H, n, d, 4)
    ref = orc.gate_proj_bwd(c, Ysa, Yswa if dual else None, Wsa, Wswa if dual else None, dY)
    dev = lambda a: U.to_dev(a, "bf16")
    tYsa, tWsa, tdY = dev(Ysa), dev(Wsa), dev(dY)
    tYswa, tWswa = (dev(Yswa), dev(Wswa)) if dual else (None, None)
    Y, Ga = torch.empty_like(tYsa), torch.empty_like(tYsa)
    Gb = torch.empty_like(tYsa) if dual else None
    desc = sa.make_desc(B, H, H, n, d, 4)
    sa.sa_gate_proj_fwd(desc, tYsa, tYswa, tWsa, tWswa, Y, Ga, Gb)
    nan = lambda t: torch.full_like(t, float("nan"))
    dYsa, dWsa = nan(tYsa), nan(tWsa)
    dYswa, dWswa = (nan(tYsa), nan(tWsa)) if dual else (None, None)
    op = sa.SA_OP_GATE_PROJ_BWD if dual else sa.SA_OP_GATE_PROJ_BWD_SINGLE
    ws = torch.full((sa.sa_workspace_bytes(desc, op),), 255, device=U.DEV, dtype=torch.uint8)
    sa.sa_gate_proj_bwd(desc, tYsa, tYswa, tWsa, tWswa, Ga, Gb, tdY, dYsa, dYswa, dWsa, dWswa, ws)
    torch.cuda.synchronize()
    # gradients are sums of bf16-rounded products: max-abs bar scaled by the tensor's own magnitude
    for name, got in (("dYsa", dYsa), ("dWsa", dWsa)) + ((("dYswa", dYswa), ("dWswa", dWswa)) if dual else ()):
        r = ref[name]
        U.assert_close(U.to_np64(got), r, "bf16", name, scale_abs=max(1.0, float(np.abs(r).max())))
    if not dual:  # too small a workspace is refused on the host
        with pytest.raises(sa.SaError) as e:
            sa.sa_gate_proj_bwd(desc, tYsa, None, tWsa, None, Ga, None, tdY, dYsa, None, dWsa, None, ws[:-256])
        assert e.value.status == sa.SA_ERR_WORKSPACE


@pytest.mark.parametrize("d,H", [(64, 2), (64, 4), (128, 1), (128, 2)])
def test_gate_proj_bwd_dual_path(d, H):
    run_bwd_case(2, H, 300, d, seed=d + H)


def test_gate_proj_bwd_single_path_and_several_token_chunks():
    run_bwd_case(1, 2, 9000, 64, seed=5, dual=False)   # 3 token chunks of the dW kernel, ragged tail
    run_bwd_case(2, 2, 1100, 64, seed=6, dual=True)


@pytest.mark.parametrize("B,n", [(1, 255), (1, 256), (2, 257), (1, 1100), (3, 2049)])
def test_backward_branches_together_and_one_after_the_other(B, n):
    """The launches of the backward serve both branches, with token chunks of dW cut down for short calls; a second-branch
    gradient in the place of dY sends the branches through one after the other.  Both must agree: dY_x to the bit, dW up to
    the order of its fp32 sums (one bf16 rounding: 2^-8 of the largest entry)."""
    from paper_2604_00754_amd import binding as sa
    H, d = 4, 64
    print(f"case gate_proj_bwd together B{B} H{H} n{n} d{d}", flush=True)
    gen = torch.Generator(device=U.DEV)
    gen.manual_seed(n)
    rnd = lambda *s: torch.randn(s, device=U.DEV, generator=gen).to(torch.bfloat16)
    Ya, Yb, dY, Wa, Wb = rnd(B, H, n, d), rnd(B, H, n, d), rnd(B, H, n, d), rnd(H * d, H * d) * 0.06, rnd(H * d, H * d) * 0.06
    Ga, Gb = torch.sigmoid(rnd(B, H, n, d)), torch.sigmoid(rnd(B, H, n, d))
    desc = sa.make_desc(B, H, H, n, d, 4)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_GATE_PROJ_BWD), device=U.DEV, dtype=torch.uint8)
    got = []
    for in_place in (False, True):
        g = dY.clone()
        dYa, dYb = torch.full_like(dY, float("nan")), g if in_place else torch.full_like(dY, float("nan"))
        dWa, dWb = torch.full_like(Wa, float("nan")), torch.full_like(Wb, float("nan"))
        ws.fill_(255)
        sa.sa_gate_proj_bwd(desc, Ya, Yb, Wa, Wb, Ga, Gb, g, dYa, dYb, dWa, dWb, ws)
        torch.cuda.synchronize()
        got.append((dYa, dYb, dWa, dWb))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    for x in (2, 3):
        a, b = got[0][x].float(), got[1][x].float()
        assert torch.isfinite(a).all() and (a - b).abs().max() <= 2 ** -8 * b.abs().max()
    # against fp64: dW_x = dz^T y with dz rounded to bf16 (2^-9 a term, averaged out over the sum; stored with 2^-9 more)
    tok = lambda t: t.double().permute(0, 2, 1, 3).reshape(B * n, H * d)
    dz = tok(dY) * tok(Ya) * tok(Ga) * (1 - tok(Ga))
    ref = dz.T @ tok(Ya)
    assert (got[0][2].double() - ref).norm() <= 5e-3 * ref.norm()


@pytest.mark.parametrize("B,H,d,n,dual", [(1, 12, 64, 257, True), (1, 12, 64, 2048, True), (1, 12, 64, 4097, True), (2, 2, 64, 1100, False),
                                          (1, 16, 128, 300, True), (1, 2, 64, 8192, False)])
def test_weight_gradients_of_short_calls_repeat_themselves(B, H, d, n, dual):
    """At most two pieces of 4096 tokens: dW has the same bits on every call, whatever the workspace holds before, and is dz^T y in
    fp64 within 5e-3 (dz rounded to bf16, 2^-9 a term, averaged out over the sum; stored with 2^-9 more)."""
    from paper_2604_00754_amd import binding as sa
    print(f"case gate_proj_bwd repeats B{B} H{H} d{d} n{n} dual={dual}", flush=True)
    gen = torch.Generator(device=U.DEV)
    gen.manual_seed(n)
    rnd = lambda *s: torch.randn(s, device=U.DEV, generator=gen).to(torch.bfloat16)
    k = 2 if dual else 1
    Y, W, G = [rnd(B, H, n, d) for _ in range(k)], [rnd(H * d, H * d) * 0.06 for _ in range(k)], [torch.sigmoid(rnd(B, H, n, d)) for _ in range(k)]
    dY = rnd(B, H, n, d)
    pad = [None] * (2 - k)
    desc = sa.make_desc(B, H, H, n, d, 4)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_GATE_PROJ_BWD if dual else sa.SA_OP_GATE_PROJ_BWD_SINGLE), device=U.DEV, dtype=torch.uint8)
    first = None
    for rep in range(8):
        ws.fill_(255 if rep % 2 == 0 else 0)
        dYx, dW = [torch.empty_like(dY) for _ in range(k)], [torch.full_like(w, float("nan")) for w in W]
        sa.sa_gate_proj_bwd(desc, *Y, *pad, *W, *pad, *G, *pad, dY, *dYx, *pad, *dW, *pad, ws)
        torch.cuda.synchronize()
        first = first or dW
        assert all(torch.equal(a, b) for a, b in zip(dW, first))
    tok = lambda t: t.double().permute(0, 2, 1, 3).reshape(B * n, H * d)
    for x in range(k):
        ref = (tok(dY) * tok(Y[x]) * tok(G[x]) * (1 - tok(G[x]))).T @ tok(Y[x])
        assert (first[x].double() - ref).norm() <= 5e-3 * ref.norm()


def products_on(B, H, n, d, dual, backward):
    from paper_2604_00754_amd import binding as sa
    return sa.gate_kernel(sa.make_desc(B, H, H, n, d, 4), backward, dual)


@pytest.mark.parametrize("B,H,n,d,dual,wide", [(11, 16, 257, 64, True, True), (7, 8, 600, 128, True, True), (22, 8, 257, 64, True, False),
                                               (43, 8, 300, 64, False, True),
                                               (65, 4, 129, 128, False, True), (86, 4, 300, 64, False, True), (129, 2, 129, 128, False, True),
                                               (130, 4, 60, 64, False, False)])
def test_wide_tiles_forward(B, H, n, d, dual, wide):
    """Batches that fill a round of 256 CUs with tiles of 256 tokens x 128 (both branches) or 256 (single path) features better than
    with tiles of 128 x 128 (too few features, or too few tiles: narrow ones); ragged token tiles, with and without gate outputs."""
    assert products_on(B, H, n, d, dual, False) == f"gate_proj_{'wide' if wide else 'fwd'}_bf16_kernel"
    run_case(B, H, n, d, seed=B + n, dual=dual, want_gates=n != 600)


@pytest.mark.parametrize("B,H,n,d,dual,wide", [(22, 8, 257, 64, True, True), (33, 4, 129, 128, True, True), (43, 8, 300, 64, False, True),
                                               (65, 4, 129, 128, False, True), (65, 4, 129, 64, True, False), (43, 2, 300, 128, True, False),
                                               (52, 4, 600, 64, False, False)])
def test_wide_tiles_backward(B, H, n, d, dual, wide):
    assert products_on(B, H, n, d, dual, True) == f"gate_proj_{'wide' if wide else 'fwd'}_bf16_kernel"
    run_bwd_case(B, H, n, d, seed=B + n, dual=dual)


@pytest.mark.parametrize("B,H,n,d,dual", [(7, 2, 333, 64, True), (9, 1, 97, 128, False), (40, 2, 31, 64, True)])
def test_weight_gradient_pieces_across_batches(B, H, n, d, dual):
    """Pieces of dW that end inside one batch and begin inside another, ragged last steps within a piece."""
    run_bwd_case(B, H, n, d, seed=B + n, dual=dual)
