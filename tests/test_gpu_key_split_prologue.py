"""Key-split prefix kernel: its queries pass through the LDS slot of the third key tile.  Tiles per wave from none to six (the
slot stays empty, is filled once, is used again by the loop), rows from one to 32, groups that are no power of two, queries
with gaps between their heads; against the oracle."""
import numpy as np
import pytest
import torch

from parity_util import check_attention, check_scores, oracle_all
from workloads import make_workload, random_parent_tree

pytestmark = pytest.mark.gpu


# the four waves take the 32-key tiles in turns: 32 keys leave three of them none, 128 give one each, 129 a second to the first
@pytest.mark.parametrize("L,splits", [(32, 1), (63, 1), (128, 1), (129, 1), (256, 1), (300, 1), (384, 1), (385, 1), (512, 1), (641, 1), (768, 1), (900, 2)])
@pytest.mark.parametrize("Hq,Hkv,T", [(1, 1, 1), (6, 2, 7), (5, 1, 6), (8, 2, 8), (31, 1, 1), (2, 2, 32)])
def test_tiles_per_wave(L, splits, Hq, Hkv, T):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    d = 128
    wl = make_workload("prologue", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=random_parent_tree(T, 4, np.random.default_rng(T)), chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] L={L} splits={splits} Hq={Hq} Hkv={Hkv} T={T}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    res = hx.run_verify(wl, num_splits=splits)
    check_attention(wl, res, ref_out, ref_lse, "prologue")
    check_scores(res["scores"], ref_scores, "prologue")
    # heads of 144 elements, one more head per row, whose values must not be taken for queries
    wide = torch.full((T, Hq + 1, d + 16), 1e4, dtype=torch.bfloat16, device="cuda")
    wide[:, :Hq, :d] = hx.to_device(wl.q, "bf16")
    buf = hx.make_buffers(dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, n_tree=T, num_splits=splits,
                          chunk_size=32, want_scores=True)
    buf.desc.q_stride_t, buf.desc.q_stride_h = (Hq + 1) * (d + 16), d + 16
    sx.verify_attn(buf.desc, wide, *(hx.to_device(x, "bf16") for x in (wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree)),
                   torch.from_numpy(np.asarray(wl.parent, dtype=np.int32)).cuda(), buf.out, buf.lse, buf.workspace)
    torch.cuda.synchronize()
    buf.check_guards()
    assert np.array_equal(buf.out.float().cpu().numpy(), res["out"]) and np.array_equal(buf.lse.cpu().numpy(), res["lse"])
