"""sa_fwd where the sorted-list kernel serves (d = 128, causal, four query heads of a KV group on one permutation, long windows or
long calls; every case says which kernel it expects): groups of 128 slots cut into quarters, lists of the band, their sections and the fallbacks, against the
fp64 oracle.  Bars: the 2e-2 / 5e-3 of the bf16 configuration (the arithmetic of a score and of a sum is the same as in the
kernel for short calls)."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U
from tests.test_gpu_fwd import run_fwd

pytestmark = pytest.mark.gpu

CIRC, LIN, ONE = 0, 1, 2

CASES = [
    # B, Hq, Hkv, n, w, window, perm_B, runs on the sorted kernel
    (4, 8, 2, 1024, 768, CIRC, 1, True),    # 256 workgroups: the fewest it is taken for
    (4, 8, 2, 1025, 769, CIRC, 4, True),    # a group of one slot
    (4, 8, 2, 1055, 800, ONE, 1, True),     # of 31
    (4, 8, 2, 1057, 780, LIN, 1, True),     # of 33: a quarter of one query
    (4, 8, 1, 1151, 769, CIRC, 4, True),    # of 127; two head sets of one KV head
    (5, 4, 1, 1700, 1023, CIRC, 1, True),   # five band slots per thread
    (5, 4, 1, 1700, 1800, CIRC, 1, True),   # the band wraps around the ring: every slot twice in a group's band
    (4, 8, 2, 2100, 1920, LIN, 1, True),    # 2035 slots of band at most, clipped at either end
    (4, 8, 2, 2100, 1921, ONE, 1, True),    # the longest band: 2048 slots, a full list
    (4, 8, 2, 2100, 1922, ONE, 1, False),   # one slot over what a list holds
    (4, 8, 2, 1024, 766, CIRC, 1, False),   # a window below the line for 256 workgroups
]


def kernel_of(B, Hq, Hkv, n, w, window, perm_B, rotated=False):
    from paper_2604_00754_amd import binding as sa
    return sa.fwd_kernel(sa.make_desc(B, Hq, Hkv, n, 128, w, window, perm_B=perm_B), rotated=rotated)


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"B{c[0]}H{c[1]}-{c[2]}n{c[3]}w{c[4]}win{c[5]}pb{c[6]}")
def test_sorted_forward(case):
    *shape, served = case
    assert (kernel_of(*shape) == "fwd_sorted_bf16_kernel") == served
    B, Hq, Hkv, n, w, window, perm_B = shape
    run_fwd(B, Hq, Hkv, n, 128, w, window, 1, "bf16", perm_B=perm_B, seed=n + w)


LARGE = [
    # B, Hq, Hkv, n, w, window, perm_B, rotated.  One workgroup takes two head sets, the last one of three by itself
    (171, 12, 3, 320, 400, CIRC, 171, False),   # a window longer than the sequence; a group of 64
    (256, 12, 3, 257, 257, CIRC, 256, True),    # a group of one slot
    (342, 12, 3, 255, 193, ONE, 342, True),     # narrow windows; a group of 127
    (781, 12, 3, 200, 193, LIN, 1, False),      # the narrowest; one permutation for the batch
    # ... and one set, window longer than the sequence
    (9, 12, 3, 460, 900, CIRC, 1, True),
]


@pytest.mark.parametrize("case", LARGE, ids=lambda c: f"B{c[0]}H{c[1]}-{c[2]}n{c[3]}w{c[4]}win{c[5]}pb{c[6]}rope{int(c[7])}")
def test_sorted_forward_batches(case):
    """Head sets that share a workgroup's list, batches with a permutation each and the narrower windows, against softmax
    attention over the visible slots in fp32 on the same bf16 rows (rotated: on rows turned in fp64 and rounded to bf16)."""
    from oracle import rope as R
    from paper_2604_00754_amd import binding as sa
    B, Hq, Hkv, n, w, window, perm_B, rotated = case
    assert kernel_of(*case) == "fwd_sorted_bf16_kernel"
    print(f"case sorted batch {case}", flush=True)
    gen = torch.Generator(device=U.DEV)
    gen.manual_seed(n + w)
    Q, K, V = (torch.randn(s, device=U.DEV, generator=gen).to(torch.bfloat16) for s in ((B, Hq, n, 128), (B, Hkv, n, 128), (B, Hkv, n, 128)))
    perm = torch.stack([torch.randperm(n, device=U.DEV, generator=gen) for _ in range(perm_B)])
    desc = sa.make_desc(B, Hq, Hkv, n, 128, w, window, perm_B=perm_B)
    Y, L = torch.full_like(Q, float("nan")), torch.full((B, Hq, n), float("nan"), device=U.DEV)
    perm32 = perm.to(torch.int32).view(perm_B, 1, n).contiguous()
    turned = Q
    if rotated:
        ang = torch.from_numpy(R.angles(n, 128)).to(U.DEV)
        a, b, c, s = Q[..., :64].double(), Q[..., 64:].double(), torch.cos(ang), torch.sin(ang)
        turned = torch.cat((a * c - b * s, a * s + b * c), -1).to(torch.bfloat16)
        sa.sa_fwd_rope(desc, Q, K, V, perm32, torch.stack((c, s), -1).float().contiguous(), Y, L)
    else:
        sa.sa_fwd(desc, Q, K, V, perm32, Y, L)
    torch.cuda.synchronize()
    t = torch.arange(n, device=U.DEV)
    off = t[:, None] - t[None, :]
    near = {CIRC: 2 * torch.minimum(off.abs(), n - off.abs()) < w, LIN: 2 * off.abs() < w, ONE: (off >= 0) & (off < w)}[window]
    err = mass = torch.zeros((), device=U.DEV, dtype=torch.float64)
    worst = worst_l = 0.0
    for i in range(B):
        p = perm[i if perm_B > 1 else 0]
        q, k, v = turned[i].float()[:, p].view(Hkv, -1, n, 128), K[i].float()[:, p], V[i].float()[:, p]
        z = (q @ k[:, None].transpose(-1, -2).contiguous()) * 128 ** -0.5
        z = z.masked_fill(~(near & (p[None, :] <= p[:, None])), -float("inf"))
        ref, lse = (torch.softmax(z, -1) @ v[:, None]).view(Hq, n, 128), torch.logsumexp(z, -1).view(Hq, n)
        d = (Y[i].float()[:, p] - ref).double()
        err, mass = err + (d * d).sum(), mass + (ref.double() ** 2).sum()
        worst, worst_l = max(worst, d.abs().max().item()), max(worst_l, (L[i][:, p] - lse).abs().max().item())
    assert worst <= 2e-2 and (err / mass).sqrt().item() <= 5e-3 and worst_l <= 4e-3, (worst, (err / mass).sqrt().item(), worst_l)


def test_sorted_forward_scores_outside_fp32_exponentials():
    """Logits of about +-150 in some rows send their workgroup through its list again in the online form; later keys that
    outscore the visible ones (K grows with the position) must not show in either form."""
    assert kernel_of(4, 8, 2, 1100, 800, CIRC, 1) == kernel_of(4, 8, 2, 1030, 780, CIRC, 1) == "fwd_sorted_bf16_kernel"
    run_fwd(4, 8, 2, 1100, 128, 800, CIRC, 1, "bf16", seed=3, k_growth=10.0)
    from oracle import binding as orc
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(4, 8, 2, 1030, 128, 780, seed=8)
    from paper_2604_00754_amd import synth
    scale = np.ones((1, 1, 1030, 1), np.float32)
    scale[:, :, 100:400] = 40.0
    x["Q"] = synth.round_to_bf16(x["Q"] * scale)
    Yr, Lr = orc.sa_fwd(U.orc_desc(wl, CIRC, 1), x["Q"], x["K"], x["V"], x["perm"])
    Q, K, V = (U.to_dev(x[k], "bf16") for k in "QKV")
    Y, L = torch.empty_like(Q), torch.empty(Q.shape[:3], device=U.DEV, dtype=torch.float32)
    sa.sa_fwd(U.sa_desc(wl, CIRC, 1), Q, K, V, torch.from_numpy(x["perm"]).to(U.DEV), Y, L)
    torch.cuda.synchronize()
    U.assert_close(U.to_np64(Y), Yr, "bf16", "Y")
    # |LSE| reaches 150: fp32 keeps 1e-5 of it beside the 4e-3 of the bf16 row sums
    assert np.abs(U.to_np64(L) - Lr).max() <= 4e-3 + 1e-5 * np.abs(Lr).max()


@pytest.mark.parametrize("interleaved", [0, 1])
def test_sorted_forward_with_rotation(interleaved):
    """The rotation of Q inside the kernel (table rows through LDS) against the pass over Q in memory.  The two may contract
    a c - b s into a multiply-add on either side, which moves a product by half an ulp of fp32; where the sum lies that close to the
    middle of two bf16 values (about one value in 2^15) it rounds to the other one.  A score is a sum of 128 products of such
    values, so the outputs agree far inside the bars of the bf16 configuration: a tenth of them is asked for."""
    from paper_2604_00754_amd import binding as sa
    wl, x = U.make_case(4, 8, 2, 1100, 128, 800, seed=5)
    assert all(kernel_of(4, 8, 2, 1100, 800, CIRC, 1, rotated=r) == "fwd_sorted_bf16_kernel" for r in (False, True))
    Q, K, V = (U.to_dev(x[k], "bf16") for k in "QKV")
    perm = torch.from_numpy(x["perm"]).to(U.DEV)
    d = U.sa_desc(wl, CIRC, 1)
    table = torch.empty(wl.n, 64, 2, device=U.DEV)
    sa.sa_rope_table(wl.n, 128, 1e4, 7, table)
    Y0, Y1, Qr = torch.empty_like(Q), torch.empty_like(Q), torch.empty_like(Q)
    sa.sa_rope(d, Q, None, table, Qr, None, interleaved=interleaved)
    sa.sa_fwd(d, Qr, K, V, perm, Y0)
    sa.sa_fwd_rope(d, Q, K, V, perm, table, Y1, interleaved=interleaved)
    torch.cuda.synchronize()
    max_abs, rel = U.errors(U.to_np64(Y1), U.to_np64(Y0))
    assert max_abs <= 2e-2 and rel <= 5e-4, (max_abs, rel)


def test_index_tensor_that_names_positions_twice_stays_inside_the_tensors():
    """Entries of perm that are in range but no bijection: the rows of the positions named more than once are undefined, every
    other row is attention over the slots as they are named, and nothing is read or written outside the tensors (Y lies
    between guard rows).  Twins in one quarter, in two quarters of a group, in two groups, and a group of one position."""
    from paper_2604_00754_amd import binding as sa
    B, Hq, Hkv, n, d, w = 4, 8, 2, 1100, 128, 800
    assert kernel_of(B, Hq, Hkv, n, w, CIRC, 1) == "fwd_sorted_bf16_kernel"
    gen = torch.Generator(device=U.DEV)
    gen.manual_seed(11)
    perm = torch.randperm(n, device=U.DEV, generator=gen)
    perm[1], perm[70], perm[900] = perm[0], perm[2], perm[3]
    perm[256:384] = 5
    Q, K, V = (torch.randn(s, device=U.DEV, generator=gen).to(torch.bfloat16) for s in ((B, Hq, n, d), (B, Hkv, n, d), (B, Hkv, n, d)))
    guard = 64 * d
    store = torch.full((Q.numel() + 2 * guard,), 7.0, device=U.DEV, dtype=torch.bfloat16)
    Y = store[guard:guard + Q.numel()].view_as(Q)
    sa.sa_fwd(sa.make_desc(B, Hq, Hkv, n, d, w), Q, K, V, perm.to(torch.int32).view(1, 1, n).contiguous(), Y)
    torch.cuda.synchronize()
    assert (store[:guard] == 7).all() and (store[-guard:] == 7).all()
    s = torch.arange(n, device=U.DEV)
    dist = (s[:, None] - s[None, :]).abs()
    seen = (2 * torch.minimum(dist, n - dist) < w) & (perm[None, :] <= perm[:, None])
    once = torch.bincount(perm, minlength=n)[perm] == 1
    for b in range(B):
        for h in range(Hq):
            k, v = K[b, h // (Hq // Hkv)].float()[perm], V[b, h // (Hq // Hkv)].float()[perm]
            z = (Q[b, h].float()[perm] @ k.T.contiguous()) * d ** -0.5
            ref = torch.softmax(z.masked_fill(~seen, -float("inf")), -1) @ v
            U.assert_close(U.to_np64(Y[b, h][perm][once]), U.to_np64(ref[once]), "bf16", f"Y[{b},{h}]")
