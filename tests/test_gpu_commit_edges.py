"""Commit of accepted rows at the edges of its work split (256 threads, K and V pieces of 16 bytes; several workgroups per
layer and head where these are few, several passes of one workgroup where they are many): rows of other sizes, a count beyond
the launch bound, a bound beyond the tree, nodes outside the tree, strided trees and caches."""
import numpy as np
import pytest
import torch

import oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,heads,T,d,elem,n", [
    (2, 3, 128, 128, 2, 128),     # 16 workgroups per head, a pass each
    (1, 1, 9, 128, 2, 9),         # 8 rows for the first workgroup, one for the second
    (3, 2, 8, 64, 4, 8),          # one workgroup, exactly one pass
    (1, 2, 20, 24, 2, 17),        # rows of 48 bytes: three pieces
    (1, 2, 5, 128, 4, 0),         # nothing accepted
])
def test_commit_passes(layers, heads, T, d, elem, n):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(T * 10 + d)
    L, cap = 37, 37 + T
    dt = {2: torch.int16, 4: torch.int32}[elem]
    npdt = {2: np.int16, 4: np.int32}[elem]
    mk = lambda *s: rng.integers(-2 ** 15, 2 ** 15, size=s).astype(npdt)
    kt, vt, kc, vc = mk(layers, heads, T, d), mk(layers, heads, T, d), mk(layers, heads, cap, d), mk(layers, heads, cap, d)
    path = rng.permutation(T)[:n].astype(np.int32)
    raw = np.full(T, -1, np.int32)
    raw[:n] = path
    k_dev, k_base = hx.guarded(kc.shape, dt)
    v_dev, v_base = hx.guarded(vc.shape, dt)
    k_dev.copy_(torch.from_numpy(kc))
    v_dev.copy_(torch.from_numpy(vc))
    to = lambda a: torch.from_numpy(a).cuda()
    # the count may say more than the bound allows
    sx.commit_tree_kv(to(kt), to(vt), k_dev, v_dev, to(raw), to(np.array([n if n < T else T + 50], np.int32)), T, T, layers,
                      heads, d, elem, L, cap)
    torch.cuda.synchronize()
    assert hx.guards_intact(k_base) and hx.guards_intact(v_base)
    for y in range(layers):
        rk, rv, _ = orc.commit_tree_kv(kc[y], vc[y], kt[y], vt[y], [int(x) for x in path], L)
        assert (k_dev[y].cpu().numpy() == rk).all() and (v_dev[y].cpu().numpy() == rv).all()


@pytest.mark.parametrize("layers,heads,T,bound,n", [
    (1, 2, 8, 128, 5),            # a fixed launch bound behind a small tree: the path has 8 entries
    (1, 1, 4, 128, 4),
    (32, 32, 4, 64, 3),           # one workgroup per head
    (1, 2, 5, 6, 0),
])
def test_launch_bound_beyond_the_tree(layers, heads, T, bound, n):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(T + bound)
    L, cap, d = 11, 11 + bound, 64
    mk = lambda *s: rng.integers(-2 ** 15, 2 ** 15, size=s).astype(np.int16)
    kt, vt, kc, vc = mk(layers, heads, T, d), mk(layers, heads, T, d), mk(layers, heads, cap, d), mk(layers, heads, cap, d)
    path = np.full(T, -1, np.int32)
    path[:n] = rng.permutation(T)[:n]
    k_dev, k_base = hx.guarded(kc.shape, torch.int16)
    v_dev, v_base = hx.guarded(vc.shape, torch.int16)
    k_dev.copy_(torch.from_numpy(kc))
    v_dev.copy_(torch.from_numpy(vc))
    to = lambda a: torch.from_numpy(a).cuda()
    print(f"[case] commit layers={layers} heads={heads} T={T} bound={bound} n={n}", flush=True)
    sx.commit_tree_kv(to(kt), to(vt), k_dev, v_dev, to(path), to(np.array([n], np.int32)), bound, T, layers, heads, d, 2, L, cap)
    torch.cuda.synchronize()
    assert hx.guards_intact(k_base) and hx.guards_intact(v_base)
    for y in range(layers):
        rk, rv, _ = orc.commit_tree_kv(kc[y], vc[y], kt[y], vt[y], [int(x) for x in path[:n]], L)
        assert (k_dev[y].cpu().numpy() == rk).all() and (v_dev[y].cpu().numpy() == rv).all()


@pytest.mark.parametrize("layers,heads,T,n,d", [
    (32, 20, 60, 60, 64),         # 640 heads: one workgroup each, four passes, the last with 12 rows' K and V left
    (33, 16, 33, 33, 24),         # 528 heads, rows of three pieces: 198 items, one pass
    (40, 8, 128, 100, 64),        # 320 heads: one workgroup each, seven passes
    (20, 8, 60, 41, 128),         # 160 heads: three workgroups each, of two passes
])
def test_several_passes_invalid_nodes_and_strides(layers, heads, T, n, d):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(layers + heads)
    L, cap = 5, 5 + T + 2
    mk = lambda *s: torch.from_numpy(rng.integers(-2 ** 15, 2 ** 15, size=s).astype(np.int16))  # noqa: E731
    # tree: K and V rows side by side; cache: eight elements behind every row
    tree, kc, vc = mk(layers, heads, T, 2 * d), mk(layers, heads, cap, d + 8), mk(layers, heads, cap, d + 8)
    path = np.full(T, -1, np.int32)
    path[:n] = rng.permutation(T)[:n]
    path[2:n:7], path[5:n:11] = -1, T + 3          # accepted entries that are no nodes: their cache rows stay
    k_dev, k_base = hx.guarded(kc.shape, torch.int16)
    v_dev, v_base = hx.guarded(vc.shape, torch.int16)
    k_dev.copy_(kc)
    v_dev.copy_(vc)
    t_dev = tree.cuda()
    print(f"[case] commit layers={layers} heads={heads} T={T} n={n} d={d}", flush=True)
    sx.commit_tree_kv(t_dev, t_dev[:, :, :, d:], k_dev, v_dev, torch.from_numpy(path).cuda(),
                      torch.tensor([n], dtype=torch.int32, device="cuda"), T, T, layers, heads, d, 2, L, cap,
                      tree_stride_layer=heads * T * 2 * d, tree_stride_h=T * 2 * d, tree_stride_t=2 * d,
                      cache_stride_layer=heads * cap * (d + 8), cache_stride_h=cap * (d + 8), cache_stride_l=d + 8)
    torch.cuda.synchronize()
    assert hx.guards_intact(k_base) and hx.guards_intact(v_base)
    for r in range(n):
        if 0 <= path[r] < T:
            kc[:, :, L + r, :d], vc[:, :, L + r, :d] = tree[:, :, path[r], :d], tree[:, :, path[r], d:]
    assert torch.equal(k_dev.cpu(), kc) and torch.equal(v_dev.cpu(), vc)
