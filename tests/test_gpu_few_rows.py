"""At most 32 query rows per KV head: prefix lengths at the edges of tiles and splits, one row to 32, strided caches, score blocks,
chunks much longer than a split, the same problem with the split count that the automatic call reports, and how far the results
are from 64 bits."""
import numpy as np
import pytest
import torch

from parity_util import check_attention, check_scores, oracle_all
from workloads import chain_tree, make_workload

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, T, L, chunk
    *[(32, 8, 8, L, 32) for L in (32, 33, 63, 64, 65, 512, 1023, 1024, 1025, 2048)],
    (4, 1, 8, 767, 32), (4, 1, 8, 769, 32), (4, 1, 1, 100, 64), (31, 1, 1, 300, 96), (7, 7, 32, 500, 32), (2, 2, 32, 4100, 64),
    (32, 8, 1, 7681, 32), (32, 8, 4, 8192 - 37, 64), (32, 32, 20, 2011, 32), (24, 12, 3, 5400, 160),
    (32, 8, 8, 1024, 1024), (32, 8, 4, 5000, 2048),
]


@pytest.mark.parametrize("Hq,Hkv,T,L,chunk", CASES)
def test_few_rows(Hq, Hkv, T, L, chunk):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    wl = make_workload("few", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, parent=chain_tree(T),
                       chunk_size=chunk, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] Hq={Hq} Hkv={Hkv} T={T} L={L} chunk={chunk}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    auto = hx.run_verify(wl, out_dtype="f32")
    plain = hx.run_verify(wl, want_scores=False, out_dtype="f32")
    splits = sx.num_splits(hx.make_buffers(dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, n_tree=T).desc)
    asked = hx.run_verify(wl, num_splits=splits, out_dtype="f32")
    for res in (auto, plain, asked):
        assert res["status"] == 0
        check_attention(wl, res, ref_out, ref_lse, "few rows")
    for res in (auto, asked):
        check_scores(res["scores"], ref_scores, "few rows")
    again = hx.run_verify(wl, want_scores=False, num_splits=splits, out_dtype="f32")
    assert np.array_equal(again["out"], plain["out"]) and np.array_equal(again["lse"], plain["lse"])
    # a cache with room behind the prefix and between the keys
    to = lambda a: hx.to_device(a, "bf16")  # noqa: E731
    wide = [torch.full((Hkv, L + 3, 136), 3e38, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    wide[0][:, :L, :128], wide[1][:, :L, :128] = to(wl.k_prefix), to(wl.v_prefix)
    buf = hx.make_buffers(dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, n_tree=T, out_dtype="f32")
    buf.desc.kp_stride_h, buf.desc.kp_stride_l = (L + 3) * 136, 136
    sx.verify_attn(buf.desc, to(wl.q), *wide, to(wl.k_tree), to(wl.v_tree), torch.from_numpy(wl.parent).cuda(), buf.out, buf.lse, buf.workspace)
    torch.cuda.synchronize()
    buf.check_guards()
    assert np.array_equal(buf.out.cpu().numpy(), plain["out"]) and np.array_equal(buf.lse.cpu().numpy(), plain["lse"])


@pytest.mark.parametrize("Hq,Hkv,T,L", [(32, 8, 1, 512), (32, 8, 8, 512), (32, 32, 20, 300), (32, 8, 8, 1000)])
def test_distance_from_64_bits(Hq, Hkv, T, L):
    """Only the probabilities are rounded.  One of 8 significant bits is off by 2^-8 / sqrt(3) * 0.72 (the mean of 1 / m over its
    mantissas) = 1.6e-3 of itself, and so is an output that is a sum of many of them.  Each wave of the key-split kernel has one
    tile of 32 keys per split of 128 here, with the tile's largest logit as its reference: that one's probability is exactly one and
    holds half of the sum of squares of 32 unit-variance logits' exponentials, which leaves 1.6e-3 * sqrt(1/2) = 1.15e-3 (measured).
    A reference for two tiles gives 1.43e-3; the bound is half way."""
    from paper_2505_20776_amd import harness as hx
    wl = make_workload("precise", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, parent=chain_tree(T),
                       chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    ref_out, _, _ = oracle_all(wl)
    out = hx.run_verify(wl, out_dtype="f32")["out"]
    assert np.linalg.norm(out - ref_out) <= 1.29e-3 * np.linalg.norm(ref_out)
