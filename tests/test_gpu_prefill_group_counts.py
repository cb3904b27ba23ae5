"""GPU parity of the prefill kernel at each number of key groups that its launch rule picks, at the edges of the tiling: row
groups with a remainder and waves of padding rows, a ragged last tile, later pieces, groups of one and three query heads, both
output types, strided tensors.  (Many KV heads fill the chip with few tokens, which is what the rule goes by.)"""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import quantize

pytestmark = pytest.mark.gpu


def _key_groups(tq, n, hq, hkv):
    """The rule of launch_prefill_rows: longest workgroup against the launch's work per compute unit, in tiles of 32 keys."""
    G, n_groups = hq // hkv, -(-tq * (hq // hkv) // 256)
    longest = -(-n // 32)
    shortest = -(-(n - tq + -(-256 // G)) // 32)
    share = hkv * n_groups * 0.5 * (longest + min(shortest, longest)) / 256
    periods = {kg: max(longest / kg, share) for kg in (1, 2, 4)}
    if 1.15 * periods[2] >= periods[1]:
        return 1
    return 2 if 1.2 * periods[4] >= periods[2] else 4


CASES = [
    # key groups, q_len, kv_len, Hq, Hkv, out, capacity
    (1, 1, 64, 1024, 512, "f32", 0),         # two rows per KV head: seven waves of padding rows
    (1, 65, 97, 768, 256, "bf16", 0),        # G = 3, 195 rows; the last tile holds one key
    (1, 100, 131, 384, 128, "f32", 0),       # 256 + 44 rows
    (1, 257, 257, 256, 256, "f32", 0),       # G = 1: 256 + 1 rows, eight tiles and one key
    (1, 257, 257, 256, 256, "bf16", 264),
    (1, 77, 205, 512, 128, "bf16", 0),       # 256 + 52 rows
    (1, 250, 1333, 256, 64, "f32", 1400),    # a later piece: 1000 rows, 41 tiles and 21 keys
    (1, 1030, 1030, 96, 32, "f32", 0),       # G = 3: 3090 rows
    (1, 4100, 4100, 32, 8, "f32", 0),        # a long whole prompt
    (2, 100, 100, 512, 64, "f32", 0),        # 800 rows: 6 * 128 + 32
    (2, 40, 1000, 512, 128, "bf16", 1024),
    (2, 150, 1000, 192, 64, "f32", 0),       # G = 3: 450 rows
    (2, 513, 513, 64, 64, "f32", 0),         # G = 1, a last row group of one row
    (2, 2047, 2047, 32, 8, "f32", 0),
    (4, 61, 700, 32, 8, "f32", 704),
]


def _draw(tq, n, hq, hkv):
    rng = np.random.default_rng(tq * 7 + n + hq)
    mk = lambda *s: quantize(rng.standard_normal(s).astype(np.float32), "bf16")  # noqa: E731
    return mk(tq, hq, 128), mk(hkv, n, 128), mk(hkv, n, 128)


def _sampled(tq):
    """Rows at the edges of tiles and row groups, and some more."""
    edges = [0, 1, 31, 32, 63, 64, 85, 86, 127, 128, 255, 256, tq - 34, tq - 2, tq - 1]
    more = np.random.default_rng(tq).integers(0, tq, size=8)
    return sorted({int(r) for r in list(edges) + list(more) if 0 <= r < tq})


def _check(out, lse, ref_out, ref_lse, rows):
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    # probabilities rounded to bf16 (2^-9 each) against the largest of the values they weigh, and the result once more
    assert np.abs(out[rows] - ref_out[rows]).max() <= 2.0 ** -8 * np.abs(ref_out[rows]).max() * 2
    assert np.abs(lse[:, rows] - ref_lse[:, rows]).max() <= 2e-4


@pytest.mark.parametrize("kg,tq,n,hq,hkv,out_dtype,cap", CASES)
def test_against_oracle(kg, tq, n, hq, hkv, out_dtype, cap):
    from paper_2505_20776_amd import harness as hx
    assert _key_groups(tq, n, hq, hkv) == kg
    q, k, v = _draw(tq, n, hq, hkv)
    rows = _sampled(tq)
    print(f"[case] prefill {kg} key groups q_len={tq} kv_len={n} Hq={hq} Hkv={hkv} {out_dtype}", flush=True)
    ref_out, ref_lse = orc.prefill_attention(q, k, v, rows=rows)
    out, lse = hx.run_prefill(q, k, v, out_dtype=out_dtype, kv_capacity=cap)
    _check(out, lse, ref_out, ref_lse, rows)


@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kg,tq,n,hq,hkv", [(1, 65, 97, 768, 256), (2, 40, 1000, 512, 128), (4, 61, 700, 32, 8)])
def test_strided_tensors(kg, tq, n, hq, hkv, out_dtype):
    """K and V of a head side by side, gaps between the heads of q and between the rows of the output, which stay untouched."""
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    assert _key_groups(tq, n, hq, hkv) == kg
    d = 128
    q, k, v = _draw(tq, n, hq, hkv)
    rows = _sampled(tq)
    print(f"[case] prefill strided {kg} key groups {out_dtype}", flush=True)
    ref_out, ref_lse = orc.prefill_attention(q, k, v, rows=rows)
    qd = torch.zeros((tq, hq, d + 8), dtype=torch.bfloat16, device="cuda")
    qd[:, :, :d] = hx.to_device(q, "bf16")
    kv = torch.zeros((hkv, n + 3, 2 * d), dtype=torch.bfloat16, device="cuda")
    kv[:, :n, :d], kv[:, :n, d:] = hx.to_device(k, "bf16"), hx.to_device(v, "bf16")
    out = torch.full((tq, hq + 1, d), 7.0, dtype=torch.bfloat16 if out_dtype == "bf16" else torch.float32, device="cuda")
    lse, base = hx.guarded((hq, tq), torch.float32)
    sx.prefill_attn(qd, kv, kv[:, :, d:], out, lse, hq, hkv, d, tq, n, out_dtype=hx.dtype_code(out_dtype),
                    q_stride_t=hq * (d + 8), q_stride_h=d + 8, kv_stride_h=(n + 3) * 2 * d, kv_stride_l=2 * d,
                    o_stride_t=(hq + 1) * d, o_stride_h=d)
    torch.cuda.synchronize()
    assert hx.guards_intact(base) and (out[:, hq] == 7.0).all()
    _check(out[:, :hq].float().cpu().numpy(), lse.cpu().numpy(), ref_out, ref_lse, rows)
