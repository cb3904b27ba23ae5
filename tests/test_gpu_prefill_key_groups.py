"""GPU parity of the prefill kernel where its workgroups cut the keys into two or four key groups (pieces of prompts and
short prompts): fewer tiles than key groups, key groups that some or all rows of a wave do not see, the shifted last tile in
every key group, row groups of 64 and 128 with a remainder, fp32 output."""
import numpy as np
import pytest

import oracle as orc
from workloads import quantize

pytestmark = pytest.mark.gpu

CASES = [
    # q_len, kv_len, Hq, Hkv, out
    (64, 64, 4, 1, "f32"),           # two tiles for four key groups; the first rows see only the first
    (33, 33, 1, 1, "bf16"),          # the second tile starts at the last key
    (17, 100, 4, 1, "bf16"),         # 68 rows: 64 + 4; four tiles, the last shifted
    (130, 130, 1, 1, "f32"),         # G = 1: the waves' rows start 32 tokens apart
    (7, 161, 8, 1, "bf16"),          # six tiles: two key groups have one tile more
    (600, 600, 8, 4, "bf16"),        # several row groups per head
    (40, 2000, 16, 2, "f32"),        # a short piece, long context
    (300, 4100, 32, 8, "bf16"),      # 1200 rows per KV head behind 3800 tokens: four key groups
    (1000, 4133, 32, 8, "bf16"),     # fewer, longer workgroups for the chip: two key groups
    (2048, 2048, 8, 8, "bf16"),      # whole prompt, G = 1
]


@pytest.mark.parametrize("tq,n,hq,hkv,out_dtype", CASES)
def test_against_oracle(tq, n, hq, hkv, out_dtype):
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(tq * 7 + n)
    mk = lambda *s: quantize(rng.standard_normal(s).astype(np.float32), "bf16")
    q, k, v = mk(tq, hq, 128), mk(hkv, n, 128), mk(hkv, n, 128)
    print(f"[case] prefill q_len={tq} kv_len={n} Hq={hq} Hkv={hkv} {out_dtype}", flush=True)
    rows = list(range(tq)) if tq * n < 1 << 19 else sorted(set([0, 1, tq - 1] + [int(r) for r in rng.integers(0, tq, size=40)]))
    ref_out, ref_lse = orc.prefill_attention(q, k, v, rows=rows)
    out, lse = hx.run_prefill(q, k, v, out_dtype=out_dtype)
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    # probabilities rounded to bf16 (2^-9 each) against the largest of the values they weigh, and the result once more
    assert np.abs(out[rows] - ref_out[rows]).max() <= 2.0 ** -8 * np.abs(ref_out[rows]).max() * 2
    assert np.abs(lse[:, rows] - ref_lse[:, rows]).max() <= 2e-4
    again, lse2 = hx.run_prefill(q, k, v, out_dtype=out_dtype)
    assert (again == out).all() and (lse2 == lse).all()
