"""GPU parity of the matrix-core prefix kernel with fp32 probabilities (fp32 inputs; bf16 inputs whose chunk size, prefix
length or key stride the bf16 kernels do not take): sizes at the edges of its key tiles (16 keys fp32, 32 bf16; four tiles
per stage), of its row groups (16, 32 or 64 rows) and of its score blocks (4, 8 or 16 keys)."""
import numpy as np
import pytest
import torch

from parity_util import check_scores, oracle_all
from workloads import chain_tree, make_workload, random_parent_tree

pytestmark = pytest.mark.gpu

# Nothing is rounded below fp32 on the way to an fp32 output: a logit of n = 128 products of unit-variance values is off by
# at most n * 2^-24 * sum|q k| / sqrt(n) = 128 * 6e-8 * (128 * 0.64 / 11.3) = 5.6e-5, a probability and the output
# relatively by as much.
TOL_F32 = 1e-4

CASES = [
    # dtype, Hq, Hkv, d, L, T, B, splits
    ("f32", 4, 1, 64, 1, 4, 4, 0),            # one key, 16 rows
    ("f32", 4, 1, 64, 15, 5, 8, 0),           # one short tile, 20 rows: two blocks of 16
    ("f32", 4, 1, 128, 16, 8, 16, 0),         # exactly one tile, 32 rows
    ("f32", 8, 1, 128, 17, 8, 12, 0),         # 64 rows: two row groups of a workgroup
    ("f32", 5, 1, 128, 63, 13, 20, 1),        # 65 rows: a second workgroup with one row
    ("f32", 8, 8, 64, 65, 1, 4, 0),           # one row per KV head, one key past a stage; KV head fastest
    ("f32", 8, 2, 64, 1000, 33, 48, 5),       # ragged splits
    ("f32", 16, 2, 128, 700, 128, 32, 64),    # more splits asked for than stages
    ("bf16", 8, 2, 128, 31, 16, 32, 0),       # shorter than the bf16 kernels' tile
    ("bf16", 8, 2, 128, 33, 9, 4, 0),         # 36 rows, 4-key score blocks, two tiles
    ("bf16", 4, 4, 128, 129, 16, 24, 0),      # 16 rows, 8-key score blocks, one key past a stage
    ("bf16", 32, 8, 128, 1500, 60, 16, 3),
    ("bf16", 8, 2, 64, 63, 20, 12, 0),        # head_dim 64 below its bf16 tile
    ("bf16", 8, 2, 64, 999, 30, 48, 2),
]


@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,T,B,splits", CASES)
def test_tile_row_and_score_block_edges(dtype, Hq, Hkv, d, L, T, B, splits):
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(L * 1000 + T)
    wl = make_workload("f32prob", seed=L + 7 * T, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=random_parent_tree(T, 9, rng), chunk_size=B, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] {dtype} Hq={Hq} Hkv={Hkv} d={d} L={L} T={T} B={B} splits={splits}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    res = hx.run_verify(wl, num_splits=splits, out_dtype="f32")
    assert res["status"] == 0
    assert np.abs(res["out"] - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
    assert np.abs(res["lse"] - ref_lse).max() <= TOL_F32
    check_scores(res["scores"], ref_scores, "fp32 probabilities")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_strided_keys_of_64(dtype):
    """Keys of 64 elements with gaps between them and between the heads (a cache that holds K and V side by side)."""
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    Hq, Hkv, d, L, T = 6, 2, 64, 333, 11
    wl = make_workload("strided64", seed=64, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=chain_tree(T), chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    ref_out, _, _ = oracle_all(wl)
    kv = torch.zeros((Hkv, L + 5, 2 * d), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    kv[:, :L, :d], kv[:, :L, d:] = hx.to_device(wl.k_prefix, dtype), hx.to_device(wl.v_prefix, dtype)
    buf = hx.make_buffers(dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, n_tree=T, out_dtype="f32")
    buf.desc.kp_stride_h, buf.desc.kp_stride_l = (L + 5) * 2 * d, 2 * d
    to = lambda a: hx.to_device(a, dtype)
    sx.verify_attn(buf.desc, to(wl.q), kv, kv[:, :, d:], to(wl.k_tree), to(wl.v_tree), torch.from_numpy(wl.parent).cuda(),
                   buf.out, buf.lse, buf.workspace)
    torch.cuda.synchronize()
    buf.check_guards()
    assert np.abs(buf.out.cpu().numpy() - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()


@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,T,B", [
    ("bf16", 32, 8, 128, 4109, 60, 16),       # eight splits of 17 tiles, the last of ten: key groups of five and four tiles
    ("bf16", 32, 8, 128, 3000, 40, 16), ("bf16", 8, 2, 64, 1000, 20, 12), ("f32", 32, 8, 128, 3333, 25, 64),
    ("f32", 16, 8, 128, 1100, 40, 32), ("f32", 4, 1, 64, 300, 12, 8)])
def test_splits_cut_at_tiles(dtype, Hq, Hkv, d, L, T, B):
    """Automatic split counts cut the prefix at whole tiles of a key group or at stages of all four, requested ones at tiles."""
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(L)
    wl = make_workload("tiles", seed=L, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=random_parent_tree(T, 9, rng), chunk_size=B, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] {dtype} Hq={Hq} Hkv={Hkv} d={d} L={L} T={T} B={B}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    for splits in (0, 6):
        res = hx.run_verify(wl, num_splits=splits, out_dtype="f32")
        assert np.abs(res["out"] - ref_out).max() <= TOL_F32 * np.abs(ref_out).max()
        assert np.abs(res["lse"] - ref_lse).max() <= TOL_F32
        check_scores(res["scores"], ref_scores, "tiles")
