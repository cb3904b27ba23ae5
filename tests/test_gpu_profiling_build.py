"""The profiling build (python -m paper_2505_20776_amd.build --stamps) gives the results of the ordinary one: its stamps lie in
workspace that the kernels do not use.  Skipped where that library is not built."""
import os
import subprocess
import sys

import numpy as np
import pytest

from workloads import make_workload, random_parent_tree

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STAMPS = os.path.join(ROOT, "paper_2505_20776_amd", "libspecext_stamps.so")

# fp32 partials: the stamps would start in the partials of rows that workgroups 2048 and 1024 merge, when the first are done
CASES = [
    # dtype, d, query heads, KV heads, nodes, keys, splits
    ("bf16", 64, 128, 16, 128, 128, 2),
    ("f32", 128, 64, 8, 128, 128, 2),
    ("bf16", 128, 32, 8, 60, 2048, 8),          # fp16 partials
]


def _results():
    from paper_2505_20776_amd import harness as hx
    out = {}
    for dtype, d, hq, hkv, T, L, splits in CASES:
        wl = make_workload("stamps", seed=d, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=L,
                           parent=random_parent_tree(T, 9, np.random.default_rng(d)), chunk_size=32, top_k=4, n_needles=0,
                           value_std=1.0)
        print(f"[case] {dtype} d={d} Hq={hq} Hkv={hkv} T={T} L={L} splits={splits}", flush=True)
        res = hx.run_verify(wl, num_splits=splits, out_dtype="f32", want_scores=False)
        out[f"{dtype}{d}"] = res["out"]
    return out


def test_same_results(tmp_path):
    if not os.path.exists(STAMPS):
        pytest.skip("the profiling build is not there")
    path = str(tmp_path / "stamped.npz")
    child = subprocess.run([sys.executable, "-u", os.path.abspath(__file__), path], cwd=ROOT, timeout=110,
                           env=dict(os.environ, SPECEXT_LIBRARY=STAMPS, PYTHONPATH=ROOT))
    assert child.returncode == 0
    stamped, plain = np.load(path), _results()
    for name, want in plain.items():
        # the same sums in the same order; the compiler may fuse other multiplications and additions
        assert np.abs(stamped[name] - want).max() <= 1e-5 * np.abs(want).max(), name


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    np.savez(sys.argv[1], **_results())
