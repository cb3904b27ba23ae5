"""Short prefixes in the row-split kernel, cut at 64 keys where that leaves compute units idle: prefix lengths at the edges of the
splits and around the line to splits of 128, both head sizes, scores of chunks that a split may not cut."""
import numpy as np
import pytest

from parity_util import check_attention, check_scores, oracle_all
from workloads import make_workload, random_parent_tree

pytestmark = pytest.mark.gpu

CASES = [
    # d, Hq, Hkv, T, L, chunk
    *[(128, 32, 8, 20, L, 32) for L in (33, 63, 64, 65, 127, 512, 1023, 1025)],
    (128, 32, 8, 60, 256, 64), (128, 8, 2, 60, 900, 96), (128, 32, 8, 60, 832, 32), (128, 32, 8, 128, 600, 32),
    *[(64, 12, 12, 60, L, 32) for L in (64, 65, 128, 300, 1024, 1025)],
    (64, 8, 2, 60, 1000, 32), (64, 32, 8, 60, 1000, 32), (64, 6, 3, 20, 500, 160),
]


@pytest.mark.parametrize("d,Hq,Hkv,T,L,chunk", CASES)
def test_short_prefix_splits(d, Hq, Hkv, T, L, chunk):
    from paper_2505_20776_amd import harness as hx
    wl = make_workload("short", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=random_parent_tree(T, 9, np.random.default_rng(L)), chunk_size=chunk, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] d={d} Hq={Hq} Hkv={Hkv} T={T} L={L} chunk={chunk}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    for want_scores in (True, False):
        res = hx.run_verify(wl, want_scores=want_scores, out_dtype="f32")
        assert res["status"] == 0
        check_attention(wl, res, ref_out, ref_lse, "short")
        if want_scores:
            check_scores(res["scores"], ref_scores, "short")
