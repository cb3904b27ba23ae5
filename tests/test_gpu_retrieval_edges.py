"""Edges of the score and selection kernels: lengths around one and four keys per thread of the byte-wise selection, all keys
in one histogram bin, few distinct keys; scores of chunks of one to five blocks with a remainder of heads and chunks, and
the one-launch form against the two calls on both sides of the line between one launch and two."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import check_scores
from workloads import chain_tree, make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 3073, 4095, 4096, 4097])
def test_selection_lengths(n):
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(n)
    few = rng.integers(0, 3, size=n).astype(np.float32)                     # ties across waves and keys of a thread
    close = (np.float32(1.0).view(np.uint32) + rng.integers(0, 200, size=n).astype(np.uint32)).view(np.float32)
    for s in (rng.standard_normal(n).astype(np.float32), few, close, np.full(n, 2.5, np.float32)):
        for k in (1, 63, n // 3, n - 1, n):
            sel, n_out, raw = hx.run_select(s, k)
            assert n_out == k and list(sel) == list(orc.select_chunks(s, k)), f"n={n} k={k}"


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 32, 48, 49, 63, 64, 65])
def test_selection_within_one_wave(n):
    """Up to 64 scores are ranked all against all in steps of 16; ties that fit whole, in part and not at all."""
    from paper_2505_20776_amd import harness as hx
    rng = np.random.default_rng(n)
    two = np.where(rng.random(n) < 0.5, np.float32(0.25), np.float32(0.75)).astype(np.float32)
    mixed = np.where(rng.random(n) < 0.3, rng.random(n), 0.5).astype(np.float32)
    for s in (rng.standard_normal(n).astype(np.float32), two, mixed, np.zeros(n, np.float32), -np.abs(rng.standard_normal(n)).astype(np.float32),
              np.arange(n, dtype=np.float32), np.arange(n, dtype=np.float32)[::-1].copy()):
        for k in range(0, n + 3):
            sel, n_out, raw = hx.run_select(s, k)
            assert n_out == min(k, n) and list(sel) == list(orc.select_chunks(s, k)), f"n={n} k={k}"
            assert (raw[n_out:] == -1).all()


@pytest.mark.parametrize("n_list,n_idx", [(1, 1), (63, 63), (64, 64), (65, 65), (65, 64), (130, 129), (64, 0), (64, 70),
                                          (256, 256), (257, 257), (258, 258), (600, 600), (600, 300), (1030, 1030)])
def test_gather_lists_around_a_wave(n_list, n_idx):
    """List entries from the 65th on are read in a second step, behind more than 256 of them by the whole workgroup; entries that
    contribute fewer or no tokens before and behind."""
    from paper_2505_20776_amd import harness as hx
    B, H, d = 9, 2, 64                      # 72 vectors of 16 bytes per chunk
    C = max(140, n_list + 10)
    L = C * B - 4                           # the last chunk has five tokens
    g = torch.Generator(device="cuda").manual_seed(n_list)
    k = torch.randn((1, H, L, d), device="cuda", generator=g).to(torch.bfloat16)
    v = torch.randn((1, H, L, d), device="cuda", generator=g).to(torch.bfloat16)
    idx = np.random.default_rng(n_list).permutation(C)[:n_list].astype(np.int32)
    idx[0] = C - 1
    idx[n_list // 2] = -1 if n_list > 1 else C - 1
    idx[-1] = C if n_list > 2 else idx[-1]
    used = [int(c) for c in idx[:n_idx] if 0 <= c < C]
    kd, vd, pos, length = hx.run_gather(k, v, idx, B, n_idx=n_idx)
    rk, rv, rpos = orc.gather_draft_kv(k.float().cpu().numpy(), v.float().cpu().numpy(), np.array(used, dtype=np.int32), B)
    assert length == len(rpos) and list(pos[:length]) == list(rpos) and (pos[length:] == -1).all()
    assert (kd[:, :, :length].float().cpu().numpy() == rk).all() and (vd[:, :, :length].float().cpu().numpy() == rv).all()


def test_gather_list_shorter_than_its_room(monkeypatch):
    """The kernel may read all max_idx entries: a list of three with room for seventy is handed over with all of them."""
    from paper_2505_20776_amd import binding, harness as hx
    handed, gather = [], binding.gather_draft_kv

    def note(*args, **kw):
        handed.append((args[4].numel(), args[6]))
        return gather(*args, **kw)

    monkeypatch.setattr(binding, "gather_draft_kv", note)
    g = torch.Generator(device="cuda").manual_seed(1)
    k = torch.randn((1, 2, 700, 64), device="cuda", generator=g).to(torch.bfloat16)
    idx = np.array([5, 0, 21], dtype=np.int32)
    for n_idx in (3, 2, None):
        kd, _, pos, length = hx.run_gather(k, k, idx, 32, n_idx=n_idx, max_idx=70)
        rk, _, rpos = orc.gather_draft_kv(k.float().cpu().numpy(), k.float().cpu().numpy(), idx[:n_idx], 32)
        assert length == len(rpos) and list(pos[:length]) == list(rpos)
        assert (kd[:, :, :length].float().cpu().numpy() == rk).all()
    assert all(size >= max_idx for size, max_idx in handed)


@pytest.mark.parametrize("Hq,Hkv,L,B", [
    (32, 8, 4096, 32),        # 128 chunks, 1024 groups: one launch
    (32, 8, 4097, 32),        # 129 chunks: two
    (32, 8, 4864, 64),        # 76 chunks, 1216 groups: one
    (6, 3, 500, 32),          # 6 heads: two of four lanes have one head more; 16 chunks
    (36, 12, 545, 32),        # 36 heads: nine per lane, one past a round of eight; 18 chunks, the last of one token
    (8, 2, 3000, 96),         # three blocks per chunk
    (8, 8, 2222, 160),        # five blocks per chunk
    (32, 32, 3008, 32),       # 32 heads x 94 blocks = 3008 groups: two launches
    (32, 32, 2976, 32),       # 2976: two
    (8, 8, 6400, 64),         # 100 chunks, 8 x 200 = 1600 groups: one
    (8, 8, 6401, 64),         # 1608: two
])
def test_scores_of_blocks_and_heads(Hq, Hkv, L, B):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    T, k = 5, 6
    wl = make_workload("edges", seed=L, dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L,
                       parent=chain_tree(T), chunk_size=B, top_k=k, n_needles=0, value_std=1.0)
    print(f"[case] scores Hq={Hq} Hkv={Hkv} L={L} B={B}", flush=True)
    ref = orc.chunk_scores(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent, B)
    t = [hx.to_device(a, "bf16") for a in (wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree)]
    buf = hx.make_buffers(dtype="bf16", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, n_tree=T, chunk_size=B,
                          want_scores=True)
    sx.verify_attn(buf.desc, *t, torch.from_numpy(wl.parent).cuda(), buf.out, buf.lse, buf.workspace)
    sx.chunk_scores(buf.desc, buf.workspace, -1, buf.scores)
    C = ref.shape[1]
    path = torch.tensor([0, 3, -1, -1, -1], dtype=torch.int32, device="cuda")
    for row, with_scores in ((4, True), (2, False), (3, True)):
        idx, n_out = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
        sc, base = hx.guarded((C,), torch.float32)
        walk = dict(path=path, n_accept=torch.tensor([2], dtype=torch.int32, device="cuda")) if row == 3 else {}
        sx.chunk_scores_select(buf.desc, buf.workspace, 0 if walk else row, k, idx, n_out, scores=sc if with_scores else None,
                               **walk)
        torch.cuda.synchronize()
        assert hx.guards_intact(base)
        got = buf.scores[row].cpu().numpy()
        if with_scores:
            assert (sc.cpu().numpy() == got).all()                       # the same bits as the call on its own
        assert int(n_out) == k and list(idx.cpu().numpy()) == list(orc.select_chunks(got, k))
    buf.check_guards()
    check_scores(buf.scores.cpu().numpy(), ref, "all rows")


def _launches(call):
    """Kernels that the call launches: the nodes of a captured graph of it."""
    paths = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
    hip = ctypes.CDLL(paths.pop())
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def test_accepted_row_at_the_ends_of_the_path():
    """The row that a walk of 128 nodes ends at: counts around a wavefront's 64 entries, at and beyond both ends, and entries that
    are no node (row 0)."""
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    T, L, B, k = 128, 200, 16, 4
    wl = make_workload("path", seed=5, dtype="f32", n_q_heads=2, n_kv_heads=1, head_dim=64, prefix_len=L, parent=chain_tree(T),
                       chunk_size=B, top_k=k, n_needles=0, value_std=1.0)
    t = [hx.to_device(a, "f32") for a in (wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree)]
    buf = hx.make_buffers(dtype="f32", n_q_heads=2, n_kv_heads=1, head_dim=64, prefix_len=L, n_tree=T, chunk_size=B, want_scores=True)
    sx.verify_attn(buf.desc, *t, torch.from_numpy(wl.parent).cuda(), buf.out, buf.lse, buf.workspace)
    sx.chunk_scores(buf.desc, buf.workspace, -1, buf.scores)
    order = np.random.default_rng(0).permutation(T).astype(np.int32)
    order[[10, 70]] = -1, 128
    path = torch.from_numpy(order).cuda()
    for count in (-3, 0, 1, 2, 11, 63, 64, 65, 71, 127, 128, 129, 2 ** 30):
        last = min(count, T) - 1
        row = int(order[last]) if last >= 0 and 0 <= order[last] < T else 0
        n_acc = torch.tensor([count], dtype=torch.int32, device="cuda")
        one, both = (torch.zeros(buf.scores.shape[1], device="cuda") for _ in range(2))
        idx, n_out = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
        sx.chunk_scores_accepted(buf.desc, buf.workspace, path, n_acc, one)
        sx.chunk_scores_select(buf.desc, buf.workspace, 0, k, idx, n_out, scores=both, path=path, n_accept=n_acc)
        torch.cuda.synchronize()
        assert torch.equal(one, buf.scores[row]) and torch.equal(both, buf.scores[row]), count
    buf.check_guards()


# both sides of the line between one launch and two: 128 chunks, 1600 pair groups
@pytest.mark.parametrize("Hkv,L,B,with_scores,launches", [
    (8, 4096, 32, True, 1), (8, 4097, 32, True, 2), (8, 5120, 64, True, 1), (16, 2560, 64, True, 1), (32, 1600, 32, True, 1),
    (8, 6400, 64, True, 1), (8, 6401, 64, True, 2), (8, 12000, 128, True, 2), (8, 12000, 128, False, 1), (2, 32768, 32, False, 1)])
def test_launches_of_scores_and_selection(Hkv, L, B, with_scores, launches):
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    T, d, k = 2, 128, 4
    g = torch.Generator(device="cuda").manual_seed(L)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    buf = hx.make_buffers(dtype="bf16", n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=d, prefix_len=L, n_tree=T, chunk_size=B, want_scores=True)
    sx.verify_attn(buf.desc, rn(T, Hkv, d), rn(Hkv, L, d), rn(Hkv, L, d), rn(Hkv, T, d), rn(Hkv, T, d),
                   torch.tensor([-1, 0], dtype=torch.int32, device="cuda"), buf.out, buf.lse, buf.workspace)
    sc = torch.empty(-(-L // B), dtype=torch.float32, device="cuda") if with_scores else None
    idx, n_out = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    assert _launches(lambda: sx.chunk_scores_select(buf.desc, buf.workspace, 1, k, idx, n_out, scores=sc)) == launches


@pytest.mark.parametrize("dtype,B,L", [
    ("f32", 80, 700),             # five blocks of 16: the first length dealt to four quads; a last chunk of four blocks
    ("f32", 128, 1024), ("f32", 144, 1000), ("f32", 256, 1030),             # 8, 9, 16 blocks; a last chunk of one block
    ("f32", 272, 600), ("f32", 512, 1500), ("f32", 528, 1100), ("f32", 1024, 2050),     # 17, 32, 33, 64
    ("f32", 1040, 2100), ("f32", 8192, 5000), ("f32", 4100, 4200),         # 65; one chunk of 313; 1025 blocks of four keys
    ("bf16", 1024, 4100), ("bf16", 16384, 9000),                           # 32 blocks of 32 keys; one chunk of 282
])
def test_chunks_of_many_score_blocks(dtype, B, L):
    """Every split of a chunk's blocks over quads, against the oracle, and the one-launch form against the two calls."""
    import paper_2505_20776_amd as sx
    from paper_2505_20776_amd import harness as hx
    T, Hq, Hkv = 3, 6, 2
    wl = make_workload("blocks", seed=B + L, dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L,
                       parent=chain_tree(T), chunk_size=B, top_k=2, n_needles=0, value_std=1.0)
    print(f"[case] chunk scores {dtype} B={B} L={L}", flush=True)
    ref = orc.chunk_scores(wl.q, wl.k_prefix, wl.v_prefix, wl.k_tree, wl.v_tree, wl.parent, B)
    buf = hx.make_buffers(dtype=dtype, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, prefix_len=L, n_tree=T, chunk_size=B,
                          want_scores=True)
    to = lambda a: hx.to_device(a, dtype)  # noqa: E731
    sx.verify_attn(buf.desc, to(wl.q), to(wl.k_prefix), to(wl.v_prefix), to(wl.k_tree), to(wl.v_tree),
                   torch.from_numpy(wl.parent).cuda(), buf.out, buf.lse, buf.workspace)
    sx.chunk_scores(buf.desc, buf.workspace, -1, buf.scores)
    check_scores(buf.scores.cpu().numpy(), ref, f"B={B}")
    C = buf.scores.shape[1]
    for row in range(T):
        one, one_base = hx.guarded((C,), torch.float32)
        idx, n_out = torch.empty(2, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
        sx.chunk_scores_select(buf.desc, buf.workspace, row, 2, idx, n_out, scores=one)
        again = torch.empty_like(idx)
        sx.chunk_scores_select(buf.desc, buf.workspace, row, 2, again, n_out, scores=None)
        assert torch.equal(one, buf.scores[row]) and hx.guards_intact(one_base)
        assert torch.equal(idx, again) and int(n_out) == min(2, C)
        assert list(idx[:int(n_out)].cpu().numpy()) == list(orc.select_chunks(one.cpu().numpy(), 2))
    torch.cuda.synchronize()
    buf.check_guards()
