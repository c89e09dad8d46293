"""Host-only checks of the C ABI: the library loads, exports every symbol include/sa.h declares, and
reports argument errors before anything is launched (no GPU needed, no kernel is run)."""
import ctypes as C
import os
import re

import pytest

from paper_2604_00754_amd import binding as sa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = C.c_void_p(4096)  # never dereferenced: every call below must fail validation first


def declared_functions():
    text = open(os.path.join(ROOT, "include", "sa.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b((?:sa|swa|gated)_\w+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert set(names) == set(sa.EXPORTS), names
    lib = sa.raw()
    for name in names:
        assert getattr(lib, name) is not None


def test_status_strings():
    for code in range(8):
        assert sa.status_string(code) and sa.status_string(code) != "unknown status"
    assert sa.status_string(99) == "unknown status"


def good():
    return sa.make_desc(2, 8, 2, 1000, 128, 256, sa.SA_WIN_SYM_CIRCULAR, 1, sa.SA_BF16, 0.0, 1, 1)


def fwd(desc, q=FAKE, k=FAKE, v=FAKE, y=FAKE):
    d = C.byref(desc) if desc is not None else None
    return sa.raw().sa_fwd(d, q, k, v, None, y, None, None, 0, None)


def test_null_arguments():
    assert fwd(None) == sa.SA_ERR_NULL
    for kw in ("q", "k", "v", "y"):
        assert fwd(good(), **{kw: None}) == sa.SA_ERR_NULL
    d = good()
    assert sa.raw().sa_check_perm(C.byref(d), None, FAKE, 1 << 30, None) == sa.SA_ERR_NULL


@pytest.mark.parametrize("field,value,status", [
    ("B", 0, sa.SA_ERR_SHAPE), ("n", 0, sa.SA_ERR_SHAPE), ("w", 0, sa.SA_ERR_SHAPE),
    ("Hkv", 3, sa.SA_ERR_SHAPE), ("window", 3, sa.SA_ERR_SHAPE), ("window", -1, sa.SA_ERR_SHAPE),
    ("perm_B", 3, sa.SA_ERR_SHAPE), ("perm_H", 2, sa.SA_ERR_SHAPE), ("causal_orig", 2, sa.SA_ERR_SHAPE),
    ("gate_per_dim", 2, sa.SA_ERR_SHAPE), ("scale", float("nan"), sa.SA_ERR_SHAPE),
    ("d", 96, sa.SA_ERR_UNSUPPORTED), ("d", 256, sa.SA_ERR_UNSUPPORTED), ("dtype", 2, sa.SA_ERR_UNSUPPORTED),
    ("gate_dtype", 5, sa.SA_ERR_UNSUPPORTED),
])
def test_bad_descriptors(field, value, status):
    d = good()
    setattr(d, field, value)
    assert fwd(d) == status
    assert sa.sa_workspace_bytes(d, sa.SA_OP_BWD) == 0


def test_workspace_sizes_and_checks():
    d = good()
    rows = d.B * d.Hq * d.n
    assert sa.sa_workspace_bytes(d, sa.SA_OP_FWD) == 0
    assert sa.sa_workspace_bytes(d, sa.SA_OP_GATED_FWD) >= rows * d.d * 2   # the first branch as a bf16 tensor
    f32 = good()
    f32.dtype = sa.SA_F32
    assert sa.sa_workspace_bytes(f32, sa.SA_OP_GATED_FWD) == 0
    ws_bwd = sa.sa_workspace_bytes(d, sa.SA_OP_BWD)
    ws_gated = sa.sa_workspace_bytes(d, sa.SA_OP_GATED_BWD)
    assert ws_bwd >= rows * 4 and ws_bwd % 256 == 0
    assert ws_gated >= 2 * rows * 4 + 2 * rows * d.d * 2
    assert sa.sa_workspace_bytes(d, sa.SA_OP_CHECK_PERM) >= d.n * 4 + 4
    lib = sa.raw()
    args = [C.byref(d), None] + [FAKE] * 17
    # ungated backward: workspace too small / missing
    assert lib.sa_bwd(*args, ws_bwd - 1, None) == sa.SA_ERR_WORKSPACE
    args_nows = list(args)
    args_nows[18] = None
    assert lib.sa_bwd(*args_nows, ws_bwd, None) == sa.SA_ERR_WORKSPACE
    # gated backward needs the larger workspace and all gate pointers
    swa = good()
    swa.window = sa.SA_WIN_ONE_SIDED
    gargs = [C.byref(d), C.byref(swa)] + [FAKE] * 17
    assert lib.sa_bwd(*gargs, ws_bwd, None) == sa.SA_ERR_WORKSPACE
    gargs_null = list(gargs)
    gargs_null[6] = None  # gate_sa
    assert lib.sa_bwd(*gargs_null, ws_gated, None) == sa.SA_ERR_NULL
    assert lib.sa_check_perm(C.byref(d), FAKE, FAKE, 16, None) == sa.SA_ERR_WORKSPACE


def test_gated_descriptors_must_agree():
    a, b = good(), good()
    b.window = sa.SA_WIN_ONE_SIDED
    lib = sa.raw()
    call = lambda x, y: lib.gated_sa_swa_fwd(C.byref(x), C.byref(y), FAKE, FAKE, FAKE, None, FAKE, FAKE,
                                             FAKE, None, None, None, None, None, 0, None)
    b.n = 999
    assert call(a, b) == sa.SA_ERR_SHAPE
    b.n = a.n
    b.dtype = sa.SA_F32
    assert call(a, b) == sa.SA_ERR_SHAPE
    b.dtype = a.dtype
    assert call(a, b) == sa.SA_ERR_WORKSPACE
    assert lib.gated_sa_swa_fwd(C.byref(a), C.byref(b), FAKE, FAKE, FAKE, None, None, FAKE, FAKE, None,
                                None, None, None, None, 0, None) == sa.SA_ERR_NULL


def test_binding_raises_with_status():
    d = good()
    d.d = 96
    with pytest.raises(sa.SaError) as e:
        sa._check(fwd(d), "sa_fwd")
    assert e.value.status == sa.SA_ERR_UNSUPPORTED


def test_decode_step_arguments():
    """sa_decode_fwd reports bad lengths, missing pointers and a short workspace before any launch."""
    d = good()
    lib = sa.raw()
    need = sa.sa_workspace_bytes(d, sa.SA_OP_DECODE)
    # one partial result of d + 2 floats per (b, hq) and chunk of the cache; chunks hold at most 1024 rows
    assert need >= 2 * 8 * (128 + 2) * 4 and need % 256 == 0

    def call(length=1000, q=FAKE, k=FAKE, v=FAKE, y=FAKE, ws=FAKE, ws_bytes=need):
        return lib.sa_decode_fwd(C.byref(d), q, k, v, length, y, None, ws, ws_bytes, None)

    for bad in (0, -1, 1001):
        assert call(length=bad) == sa.SA_ERR_SHAPE
    for kw in ("q", "k", "v", "y"):
        assert call(**{kw: None}) == sa.SA_ERR_NULL
    assert call(ws=None) == sa.SA_ERR_WORKSPACE
    assert call(ws_bytes=need - 1) == sa.SA_ERR_WORKSPACE
    assert lib.sa_decode_fwd(None, FAKE, FAKE, FAKE, 1, FAKE, None, FAKE, need, None) == sa.SA_ERR_NULL
    # the per-sequence form takes the same checks, and needs its length array
    assert lib.sa_decode_fwd_varlen(C.byref(d), FAKE, FAKE, FAKE, None, 1000, FAKE, None, FAKE, need, None) == sa.SA_ERR_NULL
    assert lib.sa_decode_fwd_varlen(C.byref(d), FAKE, FAKE, FAKE, FAKE, 1001, FAKE, None, FAKE, need, None) == sa.SA_ERR_SHAPE
    assert lib.sa_decode_fwd_varlen(C.byref(d), FAKE, FAKE, FAKE, FAKE, 1000, FAKE, None, FAKE, need - 1, None) == sa.SA_ERR_WORKSPACE
    # more (b, hq) pairs than one launch dimension holds
    wide = sa.make_desc(2048, 64, 64, 16, 64, 2)
    assert lib.sa_decode_fwd(C.byref(wide), FAKE, FAKE, FAKE, 16, FAKE, None, FAKE, 1 << 40, None) == sa.SA_ERR_UNSUPPORTED
    # the workspace is sized by the capacity: it never grows when the descriptor's n shrinks
    small = sa.make_desc(2, 8, 2, 500, 128, 256)
    assert sa.sa_workspace_bytes(small, sa.SA_OP_DECODE) <= need


def test_misaligned_pointers_are_refused_before_any_launch():
    """Tensors are accessed 16 bytes at a time: an address off that grid is reported, not launched."""
    d = good()
    lib = sa.raw()
    odd = C.c_void_p(4096 + 8)     # 8-byte aligned only
    for kw in ("q", "k", "v", "y"):
        assert fwd(d, **{kw: odd}) == sa.SA_ERR_UNSUPPORTED
    # perm and LSE need their element's alignment
    assert lib.sa_fwd(C.byref(d), FAKE, FAKE, FAKE, C.c_void_p(4098), FAKE, None, None, 0, None) == sa.SA_ERR_UNSUPPORTED
    assert lib.sa_fwd(C.byref(d), FAKE, FAKE, FAKE, None, FAKE, C.c_void_p(4098), None, 0, None) == sa.SA_ERR_UNSUPPORTED
    need = sa.sa_workspace_bytes(d, sa.SA_OP_DECODE)
    assert lib.sa_decode_fwd(C.byref(d), FAKE, odd, FAKE, 10, FAKE, None, FAKE, need, None) == sa.SA_ERR_UNSUPPORTED
    assert lib.sa_decode_fwd(C.byref(d), FAKE, FAKE, FAKE, 10, FAKE, None, odd, need, None) == sa.SA_ERR_UNSUPPORTED
    nb = sa.sa_workspace_bytes(d, sa.SA_OP_BWD)
    args = [FAKE] * 17
    args[13] = odd                 # dV
    assert lib.sa_bwd(C.byref(d), None, *args, nb, None) == sa.SA_ERR_UNSUPPORTED


def test_row_count_must_fit_32_bits():
    """B * Hq * n rows are counted in 32-bit integers inside the library: more is a shape error, not a launch."""
    ok = sa.make_desc(16, 64, 8, 1 << 20, 128, 512)          # 2^30 rows
    assert sa.sa_workspace_bytes(ok, sa.SA_OP_BWD) > 0
    big = sa.make_desc(64, 64, 8, 1 << 20, 128, 512)         # 2^32 rows
    assert fwd(big) == sa.SA_ERR_SHAPE
    assert sa.sa_workspace_bytes(big, sa.SA_OP_BWD) == 0


def test_one_head_must_span_less_than_2_gib_in_bf16():
    """The bf16 kernels form 32-bit byte offsets inside a head: n * d * 2 >= 2^31 is refused on the host, by the
    forward and by the backward alike (the fp32 path has no such limit)."""
    lib = sa.raw()
    big = sa.make_desc(1, 1, 1, 1 << 23, 128, 512)           # 2^23 rows of 256 bytes = 2 GiB
    assert fwd(big) == sa.SA_ERR_UNSUPPORTED
    nb = sa.sa_workspace_bytes(big, sa.SA_OP_BWD)
    assert nb > 0
    assert lib.sa_bwd(C.byref(big), None, *([FAKE] * 17), nb, None) == sa.SA_ERR_UNSUPPORTED
    ok = sa.make_desc(1, 1, 1, (1 << 23) - 1, 128, 512)
    assert lib.sa_bwd(C.byref(ok), None, *([FAKE] * 17), nb - 1024, None) == sa.SA_ERR_WORKSPACE   # passes the size check


def test_static_decode_refuses_what_its_buffer_cannot_hold():
    """sa_decode_fwd_static judges the size on the host, before it touches the device."""
    lib = sa.raw()
    fits = sa.make_desc(1, 32, 4, 131072, 128, 1024)
    assert 0 < sa.sa_workspace_bytes(fits, sa.SA_OP_DECODE) <= sa.SA_STATIC_SCRATCH_BYTES
    big = sa.make_desc(16, 32, 8, 131072, 128, 1024)
    assert sa.sa_workspace_bytes(big, sa.SA_OP_DECODE) > sa.SA_STATIC_SCRATCH_BYTES
    assert lib.sa_decode_fwd_static(C.byref(big), FAKE, FAKE, FAKE, 16, FAKE, None, None) == sa.SA_ERR_STATIC_LIMIT
    assert sa.status_string(sa.SA_ERR_STATIC_LIMIT).startswith("request needs more scratch")
    assert lib.sa_decode_fwd_static(C.byref(fits), None, FAKE, FAKE, 16, FAKE, None, None) == sa.SA_ERR_NULL
    assert lib.sa_decode_fwd_static(C.byref(fits), FAKE, FAKE, FAKE, 0, FAKE, None, None) == sa.SA_ERR_SHAPE
    assert lib.sa_decode_fwd_static(None, FAKE, FAKE, FAKE, 1, FAKE, None, None) == sa.SA_ERR_NULL


def test_bwd_rope_arguments():
    """sa_bwd_rope validates on the host: nulls, flags, dtype, alignment, the 2 GiB head limit, the workspace
    (the plain backward's plus the rotated query rows)."""
    lib = sa.raw()
    d = good()
    need = sa.sa_workspace_bytes(d, sa.SA_OP_BWD_ROPE)
    assert need >= sa.sa_workspace_bytes(d, sa.SA_OP_BWD) + d.B * d.Hq * d.n * d.d * 2

    def call(desc=d, table=FAKE, inter=0, dku=0, dv=FAKE, ws=FAKE, nb=need):
        return lib.sa_bwd_rope(C.byref(desc), FAKE, FAKE, FAKE, None, table, inter, dku, FAKE, FAKE, FAKE, FAKE, FAKE,
                               dv, ws, nb, None)

    assert call(table=None) == sa.SA_ERR_NULL
    assert call(dv=None) == sa.SA_ERR_NULL
    assert call(inter=2) == sa.SA_ERR_SHAPE
    assert call(dku=-1) == sa.SA_ERR_SHAPE
    assert call(dv=C.c_void_p(4096 + 8)) == sa.SA_ERR_UNSUPPORTED
    assert call(table=C.c_void_p(4096 + 4)) == sa.SA_ERR_UNSUPPORTED
    assert call(ws=None) == sa.SA_ERR_WORKSPACE
    assert call(nb=need - 1) == sa.SA_ERR_WORKSPACE
    f32 = sa.make_desc(2, 8, 2, 1000, 128, 256, dtype=sa.SA_F32)
    assert call(desc=f32) == sa.SA_ERR_UNSUPPORTED
    big = sa.make_desc(1, 1, 1, 1 << 23, 128, 512)
    assert call(desc=big, nb=1 << 40) == sa.SA_ERR_UNSUPPORTED


def test_forward_kernel_that_each_case_of_its_gpu_test_expects():
    """The dispatch rule of the forward, asked of the library without a GPU: the cases that test the sorted kernel reach it."""
    from tests import test_gpu_fwd_sorted as S
    for *shape, served in S.CASES:
        assert S.kernel_of(*shape) == ("fwd_sorted_bf16_kernel" if served else "fwd_mfma_bf16_kernel"), shape
    for case in S.LARGE:
        assert S.kernel_of(*case) == "fwd_sorted_bf16_kernel", case
    mk = sa.make_desc
    assert sa.fwd_kernel(mk(1, 32, 8, 32768, 128, 512)) == "fwd_sorted_bf16_kernel"
    # no index tensor, another one per head, another head size, groups of two, no causal test, fp32: the general kernels
    assert sa.fwd_kernel(mk(1, 32, 8, 32768, 128, 512), permuted=False) == "fwd_mfma_bf16_kernel"
    for d in (mk(1, 32, 8, 32768, 128, 512, perm_H=32), mk(1, 32, 8, 32768, 64, 512), mk(1, 16, 8, 32768, 128, 512),
              mk(1, 32, 8, 32768, 128, 512, causal_orig=0)):
        assert sa.fwd_kernel(d) == "fwd_mfma_bf16_kernel"
    # a window that reaches past both ends of a short sequence counts as the sequence, quarters without queries not at all
    for n in (148, 191):
        assert sa.fwd_kernel(mk(22, 48, 12, n, 128, 562, window=sa.SA_WIN_SYM_LINEAR, perm_B=22), rotated=True) == "fwd_mfma_bf16_kernel"
    assert sa.fwd_kernel(mk(1, 32, 8, 32768, 128, 512, dtype=sa.SA_F32)) == "fwd_f32_kernel"
    assert sa.fwd_kernel(mk(1, 32, 8, 0, 128, 512)) == ""


# heads, n, w, window, rotated, kernel; microseconds of a call with (two kernels, strips) on one MI355X
BWD_ROUTES = [
    (257, 256, 257, sa.SA_WIN_ONE_SIDED, 0, "mfma"),     # 33.6, 53.7: a second round of workgroups for one head
    (257, 256, 33, sa.SA_WIN_SYM_CIRCULAR, 0, "mfma"),   # 29.1, 34.5
    (300, 256, 200, sa.SA_WIN_SYM_CIRCULAR, 1, "mfma"),  # 56.8, 73.5
    (260, 300, 130, sa.SA_WIN_ONE_SIDED, 0, "mfma"),     # 38.9, 48.7
    (256, 256, 257, sa.SA_WIN_ONE_SIDED, 0, "mfma"),     # 24.8, 28.6: one round, windows as long as the sequence
    (2048, 256, 257, sa.SA_WIN_SYM_CIRCULAR, 0, "mfma"),  # 236, 256
    (480, 128, 64, sa.SA_WIN_SYM_CIRCULAR, 0, "mfma"),   # 25, 28
    (256, 256, 129, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 26.9, 23.0
    (480, 300, 257, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 85, 69
    (512, 256, 65, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 48.0, 35.6
    (1, 300, 17, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),    # 14.5, 9.1
    (192, 512, 257, sa.SA_WIN_ONE_SIDED, 0, "strip"),    # 48.5, 40.8
    (64, 8192, 256, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 238, 146
    (256, 4096, 256, sa.SA_WIN_SYM_CIRCULAR, 1, "strip"),  # 590, 345
    (108, 566, 225, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 44.2, 30.5: a third workgroup of the two kernels to a CU
    (48, 1291, 229, sa.SA_WIN_SYM_CIRCULAR, 1, "strip"),  # 54.3, 41.5
    (132, 992, 35, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 58.5, 45.0
    (144, 903, 142, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 70.4, 56.3
    (176, 1093, 148, sa.SA_WIN_SYM_CIRCULAR, 1, "strip"),  # 102.5, 86.0
    (133, 921, 131, sa.SA_WIN_ONE_SIDED, 0, "strip"),    # 64.9, 50.0
    (320, 512, 65, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 62.5, 52.2
    (153, 1797, 1, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),  # 71.9, 54.6
    (96, 575, 205, sa.SA_WIN_ONE_SIDED, 1, "mfma"),      # 34.3, 39.4
    (64, 65535, 257, sa.SA_WIN_SYM_CIRCULAR, 0, "strip"),
    (64, 65536, 257, sa.SA_WIN_SYM_CIRCULAR, 0, "mfma"),  # positions no longer fit 16 bits
    (64, 8192, 258, sa.SA_WIN_ONE_SIDED, 0, "mfma"),     # a window past what the waves of a workgroup hold
]


@pytest.mark.parametrize("case", BWD_ROUTES, ids=lambda c: "-".join(map(str, c)))
def test_backward_takes_the_faster_kernel(case):
    heads, n, w, window, rotated, kernel = case
    desc = sa.make_desc(1, heads, heads, n, 64, w, window)
    assert sa.bwd_kernel(desc, permuted=window != sa.SA_WIN_ONE_SIDED, rotated=rotated) == f"bwd_{kernel}_bf16_kernel"
    # grouped heads and d = 128 have the two kernels only
    for other in (sa.make_desc(1, 2 * heads, heads, n, 64, w, window), sa.make_desc(1, heads, heads, n, 128, w, window)):
        assert sa.bwd_kernel(other) == "bwd_mfma_bf16_kernel"


@pytest.mark.parametrize("heads", [2, 8, 12, 16, 20, 24, 26, 28, 30, 32, 36, 48, 64])
@pytest.mark.parametrize("B,n", [(1, 200), (1, 8192), (2, 4096), (3, 2048), (4, 8192), (16, 4096), (13, 613)])
@pytest.mark.parametrize("dual", [0, 1])
def test_weight_gradient_pieces(heads, B, n, dual):
    """Two pieces at most where the additions to dW keep their order; long calls leave few of the places of their rounds of workgroups
    (two to a CU) empty, in pieces that stay long."""
    tiles, pieces = (heads * 64 // 128) ** 2 * (1 + dual), sa.gate_dw_pieces(sa.make_desc(B, heads, heads, n, 64, 4), dual)
    if (n + 4095) // 4096 * B <= 2:
        assert pieces <= 2
    else:
        assert 1 <= pieces <= max(1, B * n // 256, min(16, 32 // tiles, B * n // 64))
        if B * n >= 32768 and B * n * tiles >= 2048 * 512 and tiles <= 512:
            assert B * n // pieces >= 2048
            assert tiles * pieces >= 0.87 * 512 * -(-tiles * pieces // 512)


# B, heads of 64, n, backward, dual, wide; microseconds of a call (the whole one, backward) with (narrow, wide) tiles on one MI355X
GATE_ROUTES = [
    (4, 8, 8192, 0, 1, False),   # 55.5, 60.1
    (16, 8, 4096, 0, 1, False),  # 106, 115
    (8, 10, 8192, 0, 1, False),  # 155, 165
    (6, 8, 8192, 0, 0, False),   # 48.0, 52.4: one round and a half
    (4, 4, 8192, 1, 1, False),   # 71.9, 74.8
    (2, 12, 8474, 0, 1, False),  # 70.7, 76.7
    (13, 12, 2774, 0, 1, False),  # 142, 152
    (11, 12, 4039, 1, 1, True),  # 390, 370
    (3, 12, 14481, 1, 1, True),  # 382, 363
    (16, 12, 3338, 1, 0, True),  # 251, 240
    (6, 12, 5316, 0, 0, True),   # 60.8, 56.4
    (3, 4, 16789, 0, 0, True),   # 21.0, 17.7
    (13, 4, 4096, 0, 0, True),   # 23.6, 20.5
    (3, 8, 4096, 0, 1, False),   # 27.7, 28.8
    (4, 8, 8192, 0, 0, True),    # 29.9, 28.1
    (8, 12, 8192, 0, 0, True),   # 115, 95.7
    (4, 16, 8192, 0, 1, True),   # 180, 171
    (4, 16, 8192, 1, 1, True),   # 436, 403
    (6, 16, 8192, 0, 0, True),   # 141, 113
    (1, 32, 4096, 1, 1, True),   # 207, 186
    (16, 12, 513, 0, 1, False),  # 34.5, 54.1: a wide tile pads further
]


@pytest.mark.parametrize("case", GATE_ROUTES, ids=lambda c: "-".join(map(str, c)))
def test_gate_products_take_the_faster_tiles(case):
    B, heads, n, backward, dual, wide = case
    for H, d in ((heads, 64), (heads // 2, 128)):
        assert sa.gate_kernel(sa.make_desc(B, H, H, n, d, 4), backward, dual) == f"gate_proj_{'wide' if wide else 'fwd'}_bf16_kernel"
