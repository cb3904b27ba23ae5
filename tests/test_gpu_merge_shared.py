"""GPU parity of the merge kernel in which four wavefronts share four rows, with fp32 partials: split counts at the edges of
its per-wave shares (1, 2, 4, 8 or 16 splits per wave; 65 go to the other kernel), row counts that are no multiple of four,
chains longer than one batch of ancestors, both head sizes, both types of input and of output."""
import numpy as np
import pytest

import oracle as orc
from parity_util import check_attention
from workloads import chain_tree, make_workload, random_parent_tree

pytestmark = pytest.mark.gpu

# fp32 inputs and output: nothing is rounded below fp32; the bound is derived at the fp32-probability kernel's tests
TOL_F32 = 1e-4

CASES = [
    # dtype, out, d, Hq, Hkv, L, T, splits -> that many splits
    ("f32", "f32", 64, 3, 1, 64, 1, 1),
    ("f32", "f32", 128, 5, 1, 4 * 64, 13, 4),
    ("f32", "f32", 64, 4, 2, 5 * 64 - 3, 33, 5),
    ("f32", "f32", 128, 2, 2, 9 * 64, 17, 9),
    ("f32", "f32", 128, 4, 1, 32 * 64, 9, 32),
    ("f32", "f32", 64, 2, 1, 33 * 64 - 1, 6, 33),
    ("f32", "f32", 128, 3, 1, 64 * 64, 5, 64),
    ("f32", "f32", 64, 1, 1, 65 * 64, 3, 65),
    ("bf16", "bf16", 128, 4, 1, 17 * 128, 7, 17),
    ("bf16", "f32", 128, 4, 2, 64 * 128, 3, 64),
    ("bf16", "bf16", 64, 3, 3, 8 * 64, 11, 8),
    ("bf16", "bf16", 64, 6, 2, 16 * 64 + 1, 21, 17),
    ("bf16", "f32", 64, 1, 1, 2 * 64, 128, 2),
]


@pytest.mark.parametrize("chain", [False, True])
@pytest.mark.parametrize("dtype,out,d,Hq,Hkv,L,T,splits", CASES)
def test_split_shares_and_row_remainders(dtype, out, d, Hq, Hkv, L, T, splits, chain):
    from paper_2505_20776_amd import harness as hx
    parent = chain_tree(T) if chain else random_parent_tree(T, 9, np.random.default_rng(L + T))
    wl = make_workload("merge", seed=L + T, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, parent=parent,
                       chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] {dtype}->{out} d={d} Hq={Hq} Hkv={Hkv} L={L} T={T} splits={splits} chain={chain}", flush=True)
    ref_out, ref_lse, _ = orc.verify_attention(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent)
    res = hx.run_verify(wl, num_splits=splits, out_dtype=out)
    assert res["status"] == 0
    if dtype == "f32":
        assert np.abs(res["out"] - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
        assert np.abs(res["lse"] - ref_lse).max() <= TOL_F32
    else:
        check_attention(wl, res, ref_out, ref_lse, "merge")
