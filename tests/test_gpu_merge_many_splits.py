"""GPU parity of the merge kernel with one wavefront per four rows, which takes 65 to 256 splits: every type of partial, both
head sizes, both types of output, row counts that are no multiple of four, chains longer than one batch of ancestors."""
import numpy as np
import pytest

import oracle as orc
from parity_util import check_attention
from workloads import chain_tree, make_workload, random_parent_tree

pytestmark = pytest.mark.gpu

# fp32 inputs and output: nothing is rounded below fp32; the bound is derived at the fp32-probability kernel's tests
TOL_F32 = 1e-4

CASES = [
    # dtype, out, d, Hq, Hkv, L, T, splits
    ("f32", "f32", 128, 3, 1, 65 * 64, 5, 65),
    ("f32", "f32", 128, 2, 2, 81 * 64 - 5, 11, 81),         # one split into a sixth round of sixteen
    ("f32", "f32", 64, 2, 1, 256 * 64, 3, 256),
    ("bf16", "bf16", 128, 8, 1, 65 * 64, 9, 65),             # fp16 partials, 72 rows
    ("bf16", "f32", 128, 5, 1, 256 * 64 - 9, 7, 256),        # fp16 partials, 35 rows
    ("bf16", "f32", 128, 4, 1, 66 * 128, 3, 66),             # fp32 partials of the key-split kernel
    ("bf16", "bf16", 64, 4, 2, 129 * 64, 7, 129),
    ("bf16", "f32", 64, 1, 1, 200 * 64, 21, 200),
]


@pytest.mark.parametrize("chain", [False, True])
@pytest.mark.parametrize("dtype,out,d,Hq,Hkv,L,T,splits", CASES)
def test_more_than_64_splits(dtype, out, d, Hq, Hkv, L, T, splits, chain):
    from paper_2505_20776_amd import harness as hx
    parent = chain_tree(T) if chain else random_parent_tree(T, 9, np.random.default_rng(L + T))
    wl = make_workload("merge", seed=L + T, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, parent=parent,
                       chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] {dtype}->{out} d={d} Hq={Hq} Hkv={Hkv} L={L} T={T} splits={splits} chain={chain}", flush=True)
    ref_out, ref_lse, _ = orc.verify_attention(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent)
    res = hx.run_verify(wl, num_splits=splits, out_dtype=out, want_scores=False)
    assert res["status"] == 0 and res["num_splits"] == splits
    if dtype == "f32":
        assert np.abs(res["out"] - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
        assert np.abs(res["lse"] - ref_lse).max() <= TOL_F32
    else:
        check_attention(wl, res, ref_out, ref_lse, "merge")
