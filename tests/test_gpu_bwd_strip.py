"""GPU parity of the one-pass bf16 backward (d = 64, one query head per KV head) against the fp64 oracle, at the sizes where
its strips, key blocks and roles meet: strip lengths around multiples of the 32-slot blocks, windows around the five and nine key
blocks its waves hold, windows that wrap onto the strip itself, and more strips than one round of workgroups."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U
from tests.test_gpu_bwd import grad_close, run_bwd, run_gated_bwd

pytestmark = pytest.mark.gpu

CIRC, LIN, ONE = 0, 1, 2


@pytest.mark.parametrize("w", [1, 3, 33, 65, 129, 131, 200, 257, 259])
@pytest.mark.parametrize("window,identity", [(CIRC, False), (LIN, False), (ONE, True)])
def test_windows_around_the_key_blocks_of_a_workgroup(w, window, identity):
    run_bwd(1, 3, 3, 415, 64, w, window, 1, "bf16", seed=300 + w, identity=identity)


@pytest.mark.parametrize("B,H,n,w", [(1, 64, 511, 100), (2, 70, 97, 40), (1, 130, 256, 256), (1, 5, 32, 31), (1, 1, 40, 8), (3, 100, 300, 64)])
def test_strip_lengths(B, H, n, w):
    """64 heads: four strips each; 140: one of four blocks; 300: two rounds of workgroups; 32 slots: one block."""
    run_bwd(B, H, H, n, 64, w, CIRC, 1, "bf16", seed=400 + n)
    run_bwd(B, H, H, n, 64, w, ONE, 0, "bf16", seed=401 + n)


def test_permutation_per_head_and_batch():
    run_bwd(2, 6, 6, 333, 64, 90, CIRC, 1, "bf16", perm_B=2, perm_H=6, seed=500)


@pytest.mark.parametrize("n,w", [(130, 33), (300, 256)])
def test_second_branch_adds(n, w):
    run_gated_bwd(2, 3, 3, n, 64, w, "bf16", seed=510 + n)


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
def test_rows_of_a_closed_gate_and_large_scores(window, causal):
    """LSE enters through three bf16 values: scores far from zero (|logit| up to about 30) and a given scale."""
    from oracle import binding as orc
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(1, 2, 2, 300, 64, 80, "bf16", 1, 1, 11, grads=True)
    x["Q"] = (x["Q"] * 4).astype(np.float32)  # still exact in bf16
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
