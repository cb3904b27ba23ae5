"""GPU parity of the merge kernel on deep trees: chain lengths at the edges of its batches of ancestors (eight from the walk, then
eight, or four with wide rows, at a time by fourth ancestors), chains of different length in one tree, broken chains, and row
counts whose workgroups are taken from their end (more than 256 of four rows)."""
import numpy as np
import pytest

import oracle as orc
from parity_util import check_attention
from workloads import chain_tree, make_workload

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4      # fp32 inputs and output: derived at the fp32-probability kernel's tests


def _comb(n, step):
    """Every node's parent is the one `step` before: `step` chains side by side, their ends at different depths."""
    return np.asarray([i - step if i >= step else -1 for i in range(n)], dtype=np.int32)


def _branching(n):
    """A spine of every third node with two leaves at each: depths up to n / 3 that differ within four rows of one head."""
    return np.asarray([-1 if i == 0 else (i - 1) // 3 * 3 if i % 3 else i - 3 for i in range(n)], dtype=np.int32)


CASES = [
    # dtype, d, Hq, Hkv, L, parents
    *[("f32", 64, 4, 2, 200, chain_tree(n)) for n in (8, 9, 12, 13, 16, 17, 20, 21, 24, 25, 32, 33, 48, 49)],
    *[("f32", 128, 3, 1, 130, chain_tree(n)) for n in (9, 12, 13, 16, 17, 20, 21, 24, 25, 128)],
    *[("bf16", 128, 8, 2, 700, chain_tree(n)) for n in (17, 31, 36, 64, 128)],
    ("bf16", 64, 5, 5, 300, chain_tree(127)),
    ("f32", 64, 2, 1, 100, _comb(128, 7)),
    ("f32", 128, 1, 1, 100, _comb(61, 3)),
    ("f32", 64, 3, 1, 100, _branching(100)),
    ("bf16", 128, 32, 8, 150, _branching(90)),          # 720 workgroups: a short third 256
    ("f32", 64, 21, 21, 64, _comb(99, 2)),              # 520 workgroups, the last of three rows
    ("f32", 64, 16, 4, 64, chain_tree(65)),             # 260: a short second 256, taken from its end
    ("f32", 64, 21, 7, 64, _comb(51, 2)),               # 268, and the last, which comes first of those, of three rows
    ("bf16", 128, 27, 9, 96, _branching(115)),     # 777: a short fourth 256, its last workgroup of one row
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_deep_trees(case):
    from paper_2505_20776_amd import harness as hx
    dtype, d, Hq, Hkv, L, parent = CASES[case]
    print(f"[case] {dtype} d={d} Hq={Hq} Hkv={Hkv} L={L} T={len(parent)}", flush=True)
    wl = make_workload("deep", seed=case, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, parent=parent,
                       chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    ref_out, ref_lse, _ = orc.verify_attention(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent)
    res = hx.run_verify(wl, out_dtype="f32")
    assert res["status"] == 0
    if dtype == "f32":
        assert np.abs(res["out"] - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
        assert np.abs(res["lse"] - ref_lse).max() <= TOL_F32
    else:
        check_attention(wl, res, ref_out, ref_lse, "deep")


@pytest.mark.parametrize("at,entry", [(5, 9), (9, 9), (18, -7), (40, 2 ** 31 - 1)])
def test_a_broken_entry_in_a_long_chain_is_a_root(at, entry):
    import torch

    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    T, Hq, Hkv, d, L = 60, 4, 2, 64, 150
    fixed = chain_tree(T)
    fixed[at] = -1
    wl = make_workload("broken", seed=at, dtype="f32", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, parent=fixed,
                       chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    ref_out, ref_lse, _ = orc.verify_attention(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent)
    parent = torch.from_numpy(fixed).cuda()
    parent[at] = entry
    buf = hx.make_buffers(dtype="f32", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, n_tree=T, out_dtype="f32")
    to = lambda a: hx.to_device(a, "f32")  # noqa: E731
    sx.verify_attn(buf.desc, to(wl.q), to(wl.k_prefix), to(wl.v_prefix), to(wl.k_tree), to(wl.v_tree), parent, buf.out, buf.lse,
                   buf.workspace)
    torch.cuda.synchronize()
    buf.check_guards()
    assert int(buf.workspace[:4].view(torch.int32)) == 1
    assert np.abs(buf.out.cpu().numpy() - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
    assert np.abs(buf.lse.cpu().numpy() - ref_lse).max() <= TOL_F32
