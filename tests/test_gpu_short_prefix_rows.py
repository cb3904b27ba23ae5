"""Short prefixes in the row-split kernel: with an automatic split count workgroups of 128 rows, with the same count asked for
those of 256.  A row's arithmetic does not depend on its workgroup, so the results are the same bits; one of the two is held
to the oracle."""
import numpy as np
import pytest

from parity_util import check_attention, check_scores, oracle_all
from workloads import make_workload, random_parent_tree

pytestmark = pytest.mark.gpu


# M = T * Hq / Hkv query rows per KV head: one past 128, the middle, one short of and exactly 256, and past it
@pytest.mark.parametrize("Hq,Hkv,d,L,T", [
    (3, 1, 128, 1024, 43), (32, 8, 128, 2048, 60), (15, 3, 128, 2048, 51), (8, 2, 128, 4096, 64), (4, 1, 128, 1024, 65),
    (4, 1, 128, 2048, 33),
    (8, 2, 64, 2048, 60), (4, 4, 64, 1024, 128), (4, 2, 64, 1024, 128)])
def test_128_row_workgroups_give_the_bits_of_256(Hq, Hkv, d, L, T):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(L + T)
    wl = make_workload("short", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L,
                       parent=random_parent_tree(T, 7, rng), chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    splits = sx.num_splits(sx.make_desc(dtype=sx.SPECEXT_BF16, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, prefix_len=L, n_tree=T,
                                        chunk_size=32, want_scores=True))
    print(f"[case] Hq={Hq} Hkv={Hkv} d={d} L={L} T={T} splits={splits}", flush=True)
    auto, asked = hx.run_verify(wl), hx.run_verify(wl, num_splits=splits)
    for what in ("out", "lse", "scores"):
        assert np.array_equal(auto[what], asked[what]), what
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    check_attention(wl, auto, ref_out, ref_lse, "short prefix")
    check_scores(auto["scores"], ref_scores, "short prefix")


# rows per KV head: one past the key-split kernel's 32, odd counts that leave padding rows in the last wave, whole waves of padding
@pytest.mark.parametrize("Hq,Hkv,L,T", [(1, 1, 4096, 33), (3, 1, 2000, 15), (4, 4, 9000, 65), (3, 1, 9000, 43), (5, 1, 9000, 51), (1, 1, 1000, 5),
                                        (6, 2, 700, 7)])
def test_score_pairs_beside_padding_rows(Hq, Hkv, L, T):
    """Every lane of a wave stores its row's score pair, padding rows that of the last real row: the same bits in every pass, and
    nothing outside of the pairs."""
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(L + T)
    wl = make_workload("pairs", seed=L + T, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L,
                       parent=random_parent_tree(T, 7, rng), chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] Hq={Hq} Hkv={Hkv} L={L} T={T}", flush=True)
    first = hx.run_verify(wl)
    for _ in range(3):
        again = hx.run_verify(wl)
        assert np.array_equal(again["scores"], first["scores"]) and np.array_equal(again["out"], first["out"])
    _, _, ref_scores = oracle_all(wl)
    check_scores(first["scores"], ref_scores, "pairs")


@pytest.mark.parametrize("L,splits,T", [(97, 1, 17), (128, 1, 20), (16 * 32, 1, 32), (16 * 32 + 1, 1, 32), (17 * 32, 1, 18), (1000, 2, 25)])
def test_ring_depths_of_four_waves(L, splits, T):
    """65 to 128 rows: a ring of three stages up to 16 tiles per split, of four beyond; split lengths around both."""
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(L)
    wl = make_workload("ring", seed=L, dtype="bf16", n_q_heads=4, n_kv_heads=1, head_dim=128, prefix_len=L,
                       parent=random_parent_tree(T, 7, rng), chunk_size=32, top_k=4, n_needles=0, value_std=1.0)
    print(f"[case] L={L} splits={splits} T={T}", flush=True)
    ref_out, ref_lse, ref_scores = oracle_all(wl)
    for want_scores in (True, False):
        res = hx.run_verify(wl, num_splits=splits, want_scores=want_scores)
        check_attention(wl, res, ref_out, ref_lse, "ring")
        if want_scores:
            check_scores(res["scores"], ref_scores, "ring")
