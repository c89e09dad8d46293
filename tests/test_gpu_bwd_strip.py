"""GPU parity of the one-pass bf16 backward (d = 64, one query head per KV head) against the fp64 oracle, at the sizes where
its strips, key blocks and roles meet: strip lengths around multiples of the 32-slot blocks, windows around the five and nine key
blocks its waves hold, windows that wrap onto the strip itself, and more strips than one round of workgroups."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U
from tests.test_gpu_bwd import grad_close, run_bwd, run_gated_bwd
from tests.test_gpu_rope import run_bwd_rope

pytestmark = pytest.mark.gpu

CIRC, LIN, ONE = 0, 1, 2


def on_strips(B, H, n, w, window, identity=False, rotated=False):
    from paper_2604_00754_amd import binding as sa
    return sa.bwd_kernel(sa.make_desc(B, H, H, n, 64, w, window), permuted=not identity, rotated=rotated) == "bwd_strip_bf16_kernel"


@pytest.mark.parametrize("w", [1, 3, 33, 65, 129, 131, 200, 257, 259])
@pytest.mark.parametrize("window,identity", [(CIRC, False), (LIN, False), (ONE, True)])
def test_windows_around_the_key_blocks_of_a_workgroup(w, window, identity):
    assert on_strips(1, 3, 415, w, window, identity) == (w <= 257)
    run_bwd(1, 3, 3, 415, 64, w, window, 1, "bf16", seed=300 + w, identity=identity)


@pytest.mark.parametrize("B,H,n,w,served", [(1, 64, 511, 100, "both"), (2, 70, 97, 40, "both"), (1, 130, 256, 256, "circular"), (1, 5, 32, 31, "both"),
                                            (1, 1, 40, 8, "both"), (3, 100, 300, 64, "both"), (1, 257, 256, 33, ""), (1, 200, 512, 100, "both"), (1, 250, 700, 256, "both"),
                                            (2, 240, 300, 64, "both")])
def test_strip_lengths(B, H, n, w, served):
    """64 heads: four strips each; 140 and 200: one each, of four and of sixteen blocks (more key blocks than a workgroup's waves); 250: of 22,
    nine key blocks in reach; 300 and 480: two rounds of workgroups (257 over 256 slots: two kernels); 32 slots: one block."""
    assert on_strips(B, H, n, w, CIRC) == (served != "") and on_strips(B, H, n, w, ONE) == (served == "both")
    run_bwd(B, H, H, n, 64, w, CIRC, 1, "bf16", seed=400 + n)
    run_bwd(B, H, H, n, 64, w, ONE, 0, "bf16", seed=401 + n)


def test_permutation_per_head_and_batch():
    assert on_strips(2, 6, 333, 90, CIRC)
    run_bwd(2, 6, 6, 333, 64, 90, CIRC, 1, "bf16", perm_B=2, perm_H=6, seed=500)


@pytest.mark.parametrize("B,H,n,w,per_dim,gate_dtype", [(2, 3, 130, 33, 0, "f32"), (2, 3, 300, 256, 0, "f32"), (1, 200, 512, 100, 0, "f32"),
                                                        (1, 250, 700, 256, 0, "f32"), (1, 3, 300, 90, 1, "f32"), (1, 7, 200, 200, 1, "bf16")])
def test_second_branch_adds(B, H, n, w, per_dim, gate_dtype):
    """One block per strip and many, both reaches; gates folded into LSE and D, gates per dimension (dO of either branch in memory)."""
    assert on_strips(B, H, n, w, CIRC)
    run_gated_bwd(B, H, H, n, 64, w, "bf16", per_dim=per_dim, gate_dtype=gate_dtype, seed=510 + n)


@pytest.mark.parametrize("n,w,gate_dtype", [(300, 80, "f32"), (415, 200, "bf16")])
def test_rows_of_closed_gates(n, w, gate_dtype):
    """Rows whose gate is closed enter with an LSE of infinity, rows all but closed with one far above their scores."""
    assert on_strips(1, 4, n, w, CIRC)
    run_gated_bwd(1, 4, 4, n, 64, w, "bf16", gate_dtype=gate_dtype, seed=530 + n, close_gates=True)


# B, H, n, w, window, causal, perm_H, identity
ROTATED = [
    (2, 4, 700, 128, CIRC, 1, 1, False), (1, 6, 333, 200, CIRC, 1, 6, False), (2, 3, 415, 129, ONE, 1, 1, True), (1, 5, 415, 257, ONE, 0, 1, False),
    (1, 3, 301, 33, LIN, 0, 1, False), (1, 5, 40, 17, CIRC, 1, 1, False),
    (1, 256, 512, 100, CIRC, 1, 1, False), (1, 250, 700, 256, CIRC, 1, 1, False),  # more key blocks to a strip than waves
]


@pytest.mark.parametrize("interleaved", [0, 1])
@pytest.mark.parametrize("dk_unrotated", [0, 1])
@pytest.mark.parametrize("case", ROTATED, ids=lambda c: f"B{c[0]}H{c[1]}n{c[2]}w{c[3]}win{c[4]}c{c[5]}")
def test_rotations(case, interleaved, dk_unrotated):
    """Q turned in its tile, dQ and (on request) dK turned back as rows: both pair layouts, both reaches, with and without the causal test."""
    B, H, n, w, window, causal, perm_H, identity = case
    assert on_strips(B, H, n, w, window, identity, rotated=True)
    run_bwd_rope(B, H, H, n, 64, w, window, causal, perm_H, interleaved, dk_unrotated, 700 + n + w, identity)


def test_results_repeat_and_outputs_over_inputs_keep_their_path():
    """Two calls give the same bits.  dK over K and dV over V, which only the two-kernel form can serve, give its gradients."""
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(1, 8, 8, 700, 64, 128, "bf16", 1, 1, 7, grads=True)
    Q, K, V, dY = (U.to_dev(x[k], "bf16") for k in ("Q", "K", "V", "dY"))
    perm = torch.from_numpy(x["perm"]).to(U.DEV)
    desc = U.sa_desc(wl, CIRC, 1)
    Y, L = torch.empty_like(Q), torch.empty((1, 8, 700), device=U.DEV)
    sa.sa_fwd(desc, Q, K, V, perm, Y, L)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_BWD), device=U.DEV, dtype=torch.uint8)
    grads = []
    for _ in range(2):
        g = [torch.empty_like(Q) for _ in range(3)]
        sa.sa_bwd(desc, None, Q, K, V, perm, None, None, Y, None, L, None, dY, *g, None, None, ws)
        grads.append(g)
    Kc, Vc, dQ = K.clone(), V.clone(), torch.empty_like(Q)
    sa.sa_bwd(desc, None, Q, Kc, Vc, perm, None, None, Y, None, L, None, dY, dQ, Kc, Vc, None, None, ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*grads))
    for got, ref, what in ((dQ, grads[0][0], "dQ"), (Kc, grads[0][1], "dK"), (Vc, grads[0][2], "dV")):
        grad_close(U.to_np64(got), U.to_np64(ref), "bf16", what)


@pytest.mark.parametrize("window,causal", [(CIRC, 1), (ONE, 0)])
def test_large_scores(window, causal):
    """LSE enters through three bf16 values: scores far from zero (|logit| up to about 30)."""
    from oracle import binding as orc
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(1, 2, 2, 300, 64, 80, "bf16", 1, 1, 11, grads=True)
    x["Q"] = (x["Q"] * 4).astype(np.float32)  # still exact in bf16
    assert on_strips(1, 2, 300, 80, window)
    oc = U.orc_desc(wl, window, causal)
    ref = orc.sa_bwd(oc, x["Q"], x["K"], x["V"], x["perm"], x["dY"])
    Q, K, V, dY = (U.to_dev(x[k], "bf16") for k in ("Q", "K", "V", "dY"))
    perm = torch.from_numpy(x["perm"]).to(U.DEV)
    desc = U.sa_desc(wl, window, causal)
    Y, L = torch.empty_like(Q), torch.empty((1, 2, 300), device=U.DEV)
    sa.sa_fwd(desc, Q, K, V, perm, Y, L)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_BWD), device=U.DEV, dtype=torch.uint8)
    g = [torch.empty_like(Q) for _ in range(3)]
    sa.sa_bwd(desc, None, Q, K, V, perm, None, None, Y, None, L, None, dY, *g, None, None, ws)
    torch.cuda.synchronize()
    for got, r, what in zip(g, ref, ("dQ", "dK", "dV")):
        grad_close(U.to_np64(got), r, "bf16", what)


@pytest.mark.parametrize("scale", [0.02, 0.25, 0.5])
def test_given_scale(scale):
    """-LSE / scale is where S starts: scales on either side of 1 / sqrt(d).  (0.5: |logit| up to about 20)"""
    assert on_strips(1, 3, 300, 80, CIRC) and on_strips(1, 3, 300, 200, CIRC)
    run_bwd(1, 3, 3, 300, 64, 80, CIRC, 1, "bf16", seed=540, scale=scale)
    run_bwd(1, 3, 3, 300, 64, 200, CIRC, 0, "bf16", seed=541, scale=scale)


@pytest.mark.parametrize("d", [64, 128])
def test_infinite_row_sums_stay_out_of_the_probabilities(d):
    """An infinity in dO, or an output row that is not finite (D = rowsum(dO o O) then is neither), spoils dQ and dK; the probabilities,
    and with them what dV gets from finite columns of dO, are those of a finite call.  (d = 128: the two kernels)"""
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(1, 2, 2, 300, d, 80, "bf16", 1, 1, 21, grads=True)
    Q, K, V, dY = (U.to_dev(x[k], "bf16") for k in ("Q", "K", "V", "dY"))
    perm = torch.from_numpy(x["perm"]).to(U.DEV)
    desc = U.sa_desc(wl, CIRC, 1)
    assert sa.bwd_kernel(desc) == ("bwd_strip_bf16_kernel" if d == 64 else "bwd_mfma_bf16_kernel")
    Y, L = torch.empty_like(Q), torch.empty((1, 2, 300), device=U.DEV)
    sa.sa_fwd(desc, Q, K, V, perm, Y, L)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_BWD), device=U.DEV, dtype=torch.uint8)

    def dv(Y, dY):
        g = [torch.empty_like(Q) for _ in range(3)]
        sa.sa_bwd(desc, None, Q, K, V, perm, None, None, Y, None, L, None, dY, *g, None, None, ws)
        torch.cuda.synchronize()
        assert not torch.isfinite(g[0]).all() or torch.isfinite(dY).all() and torch.isfinite(Y).all()
        return g[2]

    want = dv(Y, dY)
    assert torch.isfinite(want).all()
    bad = dY.clone()
    bad[0, 1, 77, 5] = float("inf")
    got, rest = dv(Y, bad), [c for c in range(d) if c != 5]
    assert torch.equal(got[..., rest], want[..., rest])
    bad = Y.clone()
    bad[0, 0, 123, 9] = float("-inf")
    assert torch.equal(dv(bad, dY), want)
