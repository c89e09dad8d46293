"""Host-only checks of bench.py's bookkeeping (no GPU): the HBM-traffic figures it reports come from the counter
records under profiles/, and are withheld when the kernel sources differ from the ones the counters were read with."""
import importlib.util
import os
import shutil

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load_bench():
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_traffic_records_parse_and_are_plausible():
    b = load_bench()
    for op, wl, algorithmic in (("sa_fwd", "qwen3_8b_prefill_32k", 675.4e6), ("sa_bwd", "pretrain_fwdbwd_8k", 539e6)):
        nbytes, source = b.measured_traffic(op, wl)
        # either the record matches the sources in this tree (a figure at or above the algorithmic bytes), or it is
        # withheld with the reason
        assert nbytes is None or algorithmic <= nbytes <= 3 * algorithmic, (op, nbytes)
        assert source


def test_traffic_is_withheld_when_a_kernel_source_changes(tmp_path):
    b = load_bench()
    shutil.copytree(b.CSRC, tmp_path / "csrc", ignore=shutil.ignore_patterns("*.o", "*.tmp"))
    b.CSRC = str(tmp_path / "csrc")
    before, _ = b.measured_traffic("sa_fwd", "qwen3_8b_prefill_32k")
    with open(tmp_path / "csrc" / "sa_fwd_mfma.hip", "a") as f:
        f.write("// edited\n")
    after, why = b.measured_traffic("sa_fwd", "qwen3_8b_prefill_32k")
    assert after is None and "changed" in why
    assert b.measured_traffic("no_such_op", "nowhere")[0] is None
    # (before is a number in a tree whose sources match the record, None otherwise: both are legitimate states)
    assert before is None or before > 0


def test_multi_gpu_request_is_refused():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode == 2 and "ONE GPU" in r.stderr


def test_flop_counts_of_the_forward():
    """Pairs that are seen, and what the sorted kernel walks for them, counted one by one on a small ring."""
    import numpy as np
    b = load_bench()
    n, w, d = 300, 101, 128
    perm = np.random.default_rng(0).permutation(n)
    slot = np.arange(n)
    dist = abs(slot[:, None] - slot[None, :])
    near = 2 * np.minimum(dist, n - dist) < w
    assert b.visible_flop(n, w, d, 1, 4) == 4 * d * 4 * int((near & (perm[None, :] <= perm[:, None])).sum())
    tiles = 0
    for p0 in range(0, n, 128):
        group = sorted(range(p0, min(p0 + 128, n)), key=lambda s: perm[s])
        band = [t % n for t in range(p0 - 50, min(p0 + 128, n) + 50)]
        for q in range(0, len(group), 32):
            keys = sum(any(perm[t] <= perm[s] for s in group[q:q + 32]) for t in band)
            tiles += -(-keys // 32)
    assert b.executed_flop_sorted(perm, w, d, 1, 4) == tiles * 4 * 32 * 32 * d * 4
