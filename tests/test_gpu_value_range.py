"""Values at the edge of the range through the prefix kernel with fp32 probabilities and the merge behind it: infinities, logits
and scales near the ends of fp32.  Each case is a call that plain fp32 attention answers."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

# as at the fp32-probability kernel's tests: a logit and with it a probability off by 5.6e-5 at most
TOL = 1e-4


def _run(dtype, q, k, v, *, chunk=16, scale=0.0, splits=0, v_tree=None, parent=None):
    """Output, log-sum-exp and chunk scores of the library and of fp64; the tree's keys are zero."""
    import paper_2505_20776_amd as sx
    dt, code = (torch.bfloat16, sx.SPECEXT_BF16) if dtype == "bf16" else (torch.float32, sx.SPECEXT_F32)
    q, k, v = q.to(dt), k.to(dt), v.to(dt)
    T, hq, d = q.shape
    hkv, L, _ = k.shape
    G = hq // hkv
    kt = torch.zeros((hkv, T, d), dtype=dt)
    vt = torch.zeros((hkv, T, d), dtype=dt) if v_tree is None else v_tree.to(dt)
    parent = [-1] * T if parent is None else parent
    desc = sx.make_desc(dtype=code, out_dtype=sx.SPECEXT_F32, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=L, n_tree=T,
                        chunk_size=chunk, want_scores=True, softmax_scale=scale, num_splits=splits)
    ws = torch.zeros(sx.workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    out, lse = torch.empty((T, hq, d), device="cuda"), torch.empty((hq, T), device="cuda")
    n_chunks = -(-L // chunk)
    scores = torch.empty((T, n_chunks), device="cuda")
    sx.verify_attn(desc, q.cuda(), k.cuda(), v.cuda(), kt.cuda(), vt.cuda(), torch.tensor(parent, dtype=torch.int32).cuda(), out,
                   lse, ws)
    sx.chunk_scores(desc, ws, -1, scores)
    torch.cuda.synchronize()

    sees = torch.zeros((T, T), dtype=torch.bool)
    for i in range(T):
        j = i
        while j >= 0:
            sees[i, j] = True
            j = parent[j]
    ref, ref_lse, ref_p = torch.empty((T, hq, d), dtype=torch.float64), torch.empty((hq, T), dtype=torch.float64), 0.0
    for h in range(hq):
        kk, vv = torch.cat([k[h // G], kt[h // G]]).double(), torch.cat([v[h // G], vt[h // G]]).double()
        s = (q[:, h].double() @ kk.t()) * (scale or 1 / math.sqrt(d))
        s[:, L:].masked_fill_(~sees, -math.inf)
        ref_lse[h] = torch.logsumexp(s, 1)
        p = torch.softmax(s, 1)
        ref_p = ref_p + p[:, :L] / hq
        # a key of probability zero contributes nothing, whatever its value
        ref[:, h] = torch.stack([(p[t, p[t] > 0, None] * vv[p[t] > 0]).sum(0) for t in range(T)])
    size = torch.tensor([min(chunk, L - c * chunk) for c in range(n_chunks)], dtype=torch.float64)
    ref_scores = torch.nn.functional.pad(ref_p, (0, n_chunks * chunk - L)).view(T, n_chunks, chunk).sum(2) / size
    return (out.cpu().double(), lse.cpu().double(), scores.cpu().double()), (ref, ref_lse, ref_scores)


def _check(got, want, tol=TOL, check_scores=True):
    (out, lse, scores), (ref, ref_lse, ref_scores) = got, want
    finite = torch.isfinite(ref)
    assert torch.equal(out[~finite], ref[~finite])            # the same infinities (no case here has a NaN)
    assert torch.isfinite(out[finite]).all()
    assert (out - ref)[finite].abs().max() <= tol * ref[finite].abs().max()
    assert ((lse - ref_lse).abs() <= tol * ref_lse.abs().clamp(min=1)).all()
    assert torch.isfinite(scores).all()
    if check_scores:
        assert (scores - ref_scores).abs().max() <= tol * ref_scores.max()


def _draw(seed, T, hq, hkv, L, d):
    gen = torch.Generator().manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=gen)  # noqa: E731
    return r(T, hq, d), r(hkv, L, d), r(hkv, L, d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("masked,splits", [(16, 0), (48, 1), (64, 0), (300, 2), (333, 0)])
def test_leading_keys_with_logits_of_minus_infinity(dtype, d, masked, splits):
    """Keys switched off by an infinite component: whole tiles, key groups, splits, all of the prefix."""
    q, k, v = _draw(masked + d, 9, 8, 2, 333, d)
    q[:, :, 0] = q[:, :, 0].abs() + 0.1
    k[:, :masked] = 0
    k[:, :masked, 0] = -math.inf
    if masked == 333:
        got, want = _run(dtype, q, k, v, splits=splits)
        assert (got[0] == 0).all() and (got[2] == 0).all()     # the tree's zero values are all there is
        assert (got[1] - want[1]).abs().max() <= TOL
    else:
        _check(*_run(dtype, q, k, v, splits=splits))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("scale", [1e-42, 1e-38, 3e-38, 1e-3, 4.0])
def test_softmax_scales(dtype, d, scale):
    """Down to the smallest scales (an even softmax).  A logit's error grows with the scale: at 4.0 its sum of d products of
    unit variance is off by up to d * 2^-24 * 4 * 0.64 * d = 2.5e-3."""
    q, k, v = _draw(d, 7, 8, 2, 200, d)
    _check(*_run(dtype, q, k, v, scale=scale), tol=TOL if scale < 1 else 2.5e-3)


@pytest.mark.parametrize("dtype,d,scale", [("f32", 64, 0.0), ("f32", 128, 0.0), ("bf16", 64, 0.0), ("bf16", 128, 0.0), ("f32", 64, 2e-4)])
@pytest.mark.parametrize("q0,k0", [(1e19, 4.5e19), (-3e5, -7e5), (3e5, -7e5)])
def test_large_logits(dtype, d, scale, q0, k0):
    """Products of 4.5e38 before the scale and of 2.1e11 (a rounding of it moves the exponent by thousands); every seventh key
    takes all of the weight, or none.  (Scores are taken against the log-sum-exp, in which fp32 holds no weight of one key beside
    2^24 or more.)"""
    q, k, v = _draw(d, 7, 8, 2, 333, d)
    q[:], k[:] = 0, 0
    q[:, :, 0], k[:, ::7, 0] = q0, k0
    _check(*_run(dtype, q, k, v, scale=scale), check_scores=False)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype,L,splits", [("f32", 333, 0), ("f32", 320, 5), ("bf16", 333, 0), ("bf16", 640, 5)])
def test_infinite_values(dtype, d, L, splits):
    """An infinite component of a value that has weight is the output's."""
    q, k, v = _draw(L + d, 9, 8, 2, L, d)
    v[:, 3, 1], v[:, 15, 5], v[:, L // 2, d - 1] = math.inf, -math.inf, math.inf
    _check(*_run(dtype, q, k, v, splits=splits))


@pytest.mark.parametrize("dtype,d,L,splits", [("f32", 64, 64, 1), ("f32", 128, 320, 5), ("f32", 64, 600, 9), ("bf16", 128, 20, 0),
                                              ("bf16", 64, 640, 5)])
def test_infinite_values_in_the_last_split_and_in_the_tree(dtype, d, L, splits):
    """The merge reads the last split and the first node again in place of those that a wave does not have."""
    q, k, v = _draw(L * d, 9, 8, 2, L, d)
    v[:, L - 2, 1] = math.inf
    v_tree = torch.randn((2, 9, d), generator=torch.Generator().manual_seed(L))
    v_tree[:, 0, 2], v_tree[:, 4, 3] = -math.inf, math.inf
    # two roots; nodes 1, 3, 5, 6 do not see node 0
    _check(*_run(dtype, q, k, v, splits=splits, v_tree=v_tree, parent=[-1, -1, 0, 1, 2, 3, 5, 4, 0]))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("size", [2.0 ** 100, 2.0 ** -100])
def test_range_of_values(dtype, d, size):
    """The magnitudes of V that the header promises, behind logits that grow from tile to tile (the reference lags by up to 2^10)."""
    q, k, v = _draw(d, 9, 8, 2, 600, d)
    k *= torch.linspace(0.2, 3, 600)[None, :, None]
    _check(*_run(dtype, q, k, v * size))
