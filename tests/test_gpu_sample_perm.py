"""GPU parity of sa_sample_perm (on-device permutation sampling, Sec. 3.3) against the numpy oracle:
bit-exact, since both sides sort the same SplitMix64 keys."""
import numpy as np
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def sample(B, H, perm_B, perm_H, n, seed, layer, workspace=False):
    """workspace=False: every bucket of keys gathered by a pass over all of them; True: with the workspace, where longer calls leave
    every key once."""
    from paper_2604_00754_amd import binding as sa
    desc = sa.make_desc(B, H, H, n, 64, 8, perm_B=perm_B, perm_H=perm_H)
    perm = torch.full((perm_B, perm_H, n), -1, device=U.DEV, dtype=torch.int32)
    ws = None
    if workspace:  # filled with ones: nothing may be read from it that the call did not write
        ws = torch.full((sa.sa_workspace_bytes(desc, sa.SA_OP_SAMPLE_PERM),), 0xFF, device=U.DEV, dtype=torch.uint8)
    sa.sa_sample_perm(desc, seed, layer, perm, ws)
    torch.cuda.synchronize()
    return desc, perm


@pytest.mark.parametrize("n", [1, 5, 256, 1000, 1024, 4097, 16384, 20011, 32768])
def test_sample_perm_matches_oracle_bit_for_bit(n):
    from oracle import perm_sampler as ps
    print(f"case sample_perm n{n}", flush=True)
    for perm_B, perm_H, seed, layer in ((1, 1, 0, 0), (2, 3, 20260400754, 5)):
        ref = ps.sample_perm(seed, layer, perm_B, perm_H, n)
        for workspace in (False, True):
            _, perm = sample(2, 3, perm_B, perm_H, n, seed, layer, workspace)
            assert np.array_equal(perm.cpu().numpy(), ref), f"workspace={workspace}"


def test_sample_perm_long_sequence_and_full_64_bit_seed():
    from oracle import perm_sampler as ps
    from paper_2604_00754_amd import binding as sa
    n, seed = 131072, 2 ** 64 - 3
    ref = ps.sample_perm(seed, 1, 1, 1, n)
    desc, perm = sample(1, 1, 1, 1, n, seed, 1)
    assert np.array_equal(perm.cpu().numpy(), ref)
    desc, perm = sample(1, 1, 1, 1, n, seed, 1, workspace=True)
    assert np.array_equal(perm.cpu().numpy(), ref)
    ws = torch.empty(sa.sa_workspace_bytes(desc, sa.SA_OP_CHECK_PERM), device=U.DEV, dtype=torch.uint8)
    sa.sa_check_perm(desc, perm, ws)  # raises unless every slice is a bijection


def test_sampled_permutation_feeds_the_attention_kernel():
    """The sampler's output is used as it is: sa_fwd with the device-sampled permutation against the
    oracle run with the oracle-sampled one."""
    from oracle import binding as orc
    from oracle import perm_sampler as ps
    from paper_2604_00754_amd import binding as sa
    B, H, n, d, w = 1, 2, 700, 64, 64
    wl, x = U.make_case(B, H, H, n, d, w, "bf16", 1, 2, seed=70)
    desc = sa.make_desc(B, H, H, n, d, w, perm_B=1, perm_H=2)
    perm = torch.empty((1, 2, n), device=U.DEV, dtype=torch.int32)
    sa.sa_sample_perm(desc, 99, 2, perm)
    Q, K, V = (U.to_dev(x[k], "bf16") for k in "QKV")
    Y = torch.empty_like(Q)
    sa.sa_fwd(desc, Q, K, V, perm, Y, None)
    torch.cuda.synchronize()
    Yr, _ = orc.sa_fwd(orc.desc(B, H, H, n, d, w, orc.WIN_SYM_CIRCULAR, 1, 1, 2), x["Q"], x["K"], x["V"],
                       ps.sample_perm(99, 2, 1, 2, n))
    U.assert_close(U.to_np64(Y), Yr, "bf16", "Y")


def test_sample_perm_rejects_bad_arguments():
    from paper_2604_00754_amd import binding as sa
    desc = sa.make_desc(1, 1, 1, 16, 64, 4)
    with pytest.raises(sa.SaError) as e:
        sa.sa_sample_perm(desc, 1, 0, None)
    assert e.value.status == sa.SA_ERR_NULL
    perm = torch.empty((1, 1, 16), device=U.DEV, dtype=torch.int32)
    with pytest.raises(sa.SaError) as e:
        sa.sa_sample_perm(desc, 1, -1, perm)
    assert e.value.status == sa.SA_ERR_SHAPE
    big = sa.make_desc(1, 1, 1, 4096, 64, 4)
    perm = torch.empty((1, 1, 4096), device=U.DEV, dtype=torch.int32)
    ws = torch.empty(sa.sa_workspace_bytes(big, sa.SA_OP_SAMPLE_PERM) - 1, device=U.DEV, dtype=torch.uint8)
    with pytest.raises(sa.SaError) as e:
        sa.sa_sample_perm(big, 1, 0, perm, ws)
    assert e.value.status == sa.SA_ERR_WORKSPACE


@pytest.mark.parametrize("slices,n", [(1, 2), (1, 65), (3, 257), (1, 19999), (1, 23439), (12, 5700), (12, 6500), (2, 32769),
                                      (1, 65537), (1, (1 << 17) + 1), (1, 1 << 20)])
def test_sample_perm_gathering_forms(slices, n):
    """Both ways of gathering a bucket, on both sides of the line between them (6 million keys formed by the scan) and at
    odd piece, bucket and slice counts: bit for bit the oracle's argsort."""
    from oracle import perm_sampler as ps
    print(f"case sample_perm {slices} x {n}", flush=True)
    ref = ps.sample_perm(31, 4, 1, slices, n)
    for workspace in (False, True):
        _, perm = sample(1, slices, 1, slices, n, 31, 4, workspace)
        assert np.array_equal(perm.cpu().numpy(), ref), f"workspace={workspace}"


@pytest.mark.parametrize("workspace", [False, True])
@pytest.mark.parametrize("cap", [1, 40, 64, 140])
@pytest.mark.parametrize("slices,n", [(2, 300), (3, 20000)])
def test_sample_perm_buckets_that_do_not_fit(slices, n, cap, workspace):
    """With room for fewer keys than a bucket holds (64 to 128 on average) some or all buckets are ranked by a pass over every key:
    the same permutation, bit for bit."""
    import ctypes as C
    from oracle import perm_sampler as ps
    from paper_2604_00754_amd import binding as sa
    print(f"case sample_perm {slices} x {n} cap {cap} workspace={workspace}", flush=True)
    desc = sa.make_desc(1, slices, slices, n, 64, 8, perm_H=slices)
    perm = torch.full((1, slices, n), -1, device=U.DEV, dtype=torch.int32)
    ws = torch.full((sa.sa_workspace_bytes(desc, sa.SA_OP_SAMPLE_PERM),), 0xFF, device=U.DEV, dtype=torch.uint8) if workspace else None
    assert sa.raw().sa_internal_sample_perm(C.byref(desc), 7, 2, perm.data_ptr(), ws.data_ptr() if workspace else None,
                                            ws.numel() if workspace else 0, cap, torch.cuda.current_stream().cuda_stream) == sa.SA_OK
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy(), ps.sample_perm(7, 2, 1, slices, n))
