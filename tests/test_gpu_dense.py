"""The dense form of the exact top-k on the fused shapes (slices, ragged
ranges, partly filled query groups, bucket maxima) against its own scores
ranked by torch and against float64 (MI355X only)."""
import dataclasses

import pytest
import torch

import synth
from paper_2407_15462_amd import mol
from parity_helpers import cuda_inputs, log

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS
SHAPES = {"exact_32k": W["exact_32k"], "exact_1m": W["exact_1m"], "hybrid_8m": W["hybrid_8m"],
          "paper_books": W["paper_books"]}


# every number of slices and its edges (2, 4, 8 queries), a last group with
# one to sixteen queries, items that end inside a step, a tile and a bucket
# block, rows with and without bucket maxima
@pytest.mark.parametrize("wl", list(SHAPES))
@pytest.mark.parametrize("B,N,k", [
    (1, 1, 1), (1, 20011, 100), (2, 333, 100), (3, 16384, 128), (4, 65537, 7), (5, 31, 31), (8, 16449, 100),
    (9, 20000, 100), (17, 16500, 128), (33, 1000, 64), (40, 24186, 100),
])
def test_dense_topk_equals_ranked_scores(wl, B, N, k):
    spec = SHAPES[wl].scaled(B=B, N=N, clusters=max(1, N // 200))
    log(f"[dense] {wl} B={B} N={N} k={k}")
    inp = cuda_inputs(spec, seed=B + N)
    for flags in (0, mol.MOL_FLAG_BF16X2_GATING):
        prob = mol.Problem.from_inputs(inp, flags=flags)
        phi = mol.score(prob)
        s, i = mol.topk_exact(prob, k)
        ns, ni = torch.empty_like(s), torch.empty_like(i)
        mol.mol_topk_exact_noalloc(prob, k, ns, ni)          # the per-range list form
        torch.cuda.synchronize()
        ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
        assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])
        assert torch.equal(ns, s) and torch.equal(ni, i)
        f32 = mol.score(mol.Problem.from_inputs(inp, flags=mol.MOL_FLAG_F32_GATING))
        assert (phi - f32).abs().max() <= 2e-5               # the chains' stated error at std 0.1, ten times over


def test_dense_topk_ties_across_ranges():
    """Identical items spread over every range: ranked by index; more of them
    than the selection's list holds."""
    spec = dataclasses.replace(W["exact_32k"], B=5, N=40000, clusters=64)
    inp = cuda_inputs(spec, seed=3)
    at = torch.randperm(spec.N, generator=torch.Generator().manual_seed(1))[:6000].cuda()
    inp.X[:, at] = inp.X[:, at[:1]]
    inp.a_x[at] = inp.a_x[at[:1]]
    inp.Q[:] = inp.X[:, at[0]].repeat(2, 1)[None]            # the tied items come first
    prob = mol.Problem.from_inputs(inp)
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, 100)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :100]) and torch.equal(i.long(), wi[:, :100])


def _ordered(v, i):
    """descending scores, ascending ids among equals"""
    return bool(((v[:, 1:] < v[:, :-1]) | ((v[:, 1:] == v[:, :-1]) & (i[:, 1:] > i[:, :-1]))).all())


# lists ranked from dense dot products: rows with and without bucket maxima, k
# on both sides of 512 and at its largest, a ragged last tile, and (the last) a
# problem whose dense scores pass the buffer's limit (the sampled-threshold form)
@pytest.mark.parametrize("B,Pq,Px,d,N,kp", [
    (3, 4, 4, 96, 3001, 50), (5, 2, 3, 96, 20011, 128), (2, 4, 4, 768, 16447, 5), (3, 1, 1, 64, 4000, 600),
    (4, 1, 1, 32, 200001, 2048), (2, 1, 1, 128, 60001, 513), (1, 1, 1, 64, 50000, 512), (64, 4, 4, 96, 140001, 60),
])
def test_dense_lists(B, Pq, Px, d, N, kp):
    log(f"[lists] B={B} P={Pq}x{Px} d={d} N={N} k'={kp}")
    g = torch.Generator(device="cuda").manual_seed(N)
    Q = torch.nn.functional.normalize(torch.randn((B, Pq, d), generator=g, device="cuda"), dim=-1).bfloat16()
    X = torch.nn.functional.normalize(torch.randn((Px, N, d), generator=g, device="cuda"), dim=-1).bfloat16()
    dots, ids = mol.topk_per_embd(mol.Problem(Q, X), kp)
    torch.cuda.synchronize()
    for b in range(0, B, max(1, B // 3)):
        s = torch.stack([Q[b].double() @ X[px].double().t().contiguous() for px in range(Px)], 1).view(Pq * Px, N)
        want = torch.topk(s, kp, dim=1).values
        got = torch.gather(s, 1, ids[b].long())
        # float32 sums of d products of unit rows
        tol = d * 2.0 ** -24
        assert (dots[b].double() - got).abs().max() <= tol and (got - want).abs().max() <= 2 * tol
        assert all(torch.unique(ids[b, p]).numel() == kp for p in range(Pq * Px))
        assert _ordered(dots[b], ids[b])


# the small-batch per-component form: lists on both sides of its appending
# scan's bucket rule (2 k' buckets), every width and list capacity, ragged
# ranges; and a batch whose lists overflow their key buffers (identical items)
@pytest.mark.parametrize("B,Px,d,N,kp,ties", [
    (1, 1, 32, 700, 10, 0), (32, 8, 32, 33001, 200, 0), (3, 4, 64, 8192, 128, 0), (3, 4, 64, 8191, 129, 0),
    (32, 4, 128, 24186, 100, 0), (5, 2, 128, 20000, 256, 0), (31, 8, 64, 50001, 5, 0), (4, 8, 32, 40000, 100, 3000),
])
def test_small_batch_lists(B, Px, d, N, kp, ties):
    log(f"[small lists] B={B} P=8x{Px} d={d} N={N} k'={kp} ties={ties}")
    g = torch.Generator(device="cuda").manual_seed(N + kp)
    X = torch.nn.functional.normalize(torch.randn((Px, N, d), generator=g, device="cuda"), dim=-1).bfloat16()
    Q = torch.nn.functional.normalize(torch.randn((B, 8, d), generator=g, device="cuda"), dim=-1).bfloat16()
    if ties:
        at = torch.randperm(N, generator=torch.Generator().manual_seed(2))[:ties].cuda()
        X[:, at] = X[:, at[:1]]
        Q[0] = X[torch.arange(8) % Px, at[0]]
        Q[1] = 0
    dots, ids = mol.topk_per_embd(mol.Problem(Q, X), kp)
    torch.cuda.synchronize()
    tol = d * 2.0 ** -24
    for b in range(B):
        s = torch.stack([Q[b].double() @ X[px].double().t().contiguous() for px in range(Px)], 1).view(8 * Px, N)
        want = torch.topk(s, kp, dim=1).values
        got = torch.gather(s, 1, ids[b].long())
        assert (dots[b].double() - got).abs().max() <= tol and (got - want).abs().max() <= 2 * tol
        assert _ordered(dots[b], ids[b])


# dots and gating in one kernel (P_x = 4): every vector tile (32, 64, 128, and
# more than one), ragged items, one to many K steps, padded hidden units, with
# and without side logits of aligned rows; the pair-wise kernels (the
# allocation-free form takes them) give the same bits
@pytest.mark.parametrize("B,Pq,d,H,N,k", [
    (1, 4, 768, 64, 20011, 100), (8, 4, 768, 64, 70, 50), (9, 4, 64, 64, 3001, 100), (32, 4, 768, 64, 16449, 128),
    (33, 4, 96, 48, 2000, 64), (75, 4, 32, 32, 1025, 100), (17, 2, 128, 100, 2100, 33), (40, 1, 64, 128, 999, 10),
    (3, 2, 1024, 17, 65, 65),
])
def test_dots_phi_equals_pairwise_kernels(B, Pq, d, H, N, k):
    log(f"[dots_phi] B={B} P={Pq}x4 d={d} H={H} N={N} k={k}")
    spec = dataclasses.replace(W["exact_32k"], name="pairwise", B=B, N=N, Pq=Pq, Px=4, d=d, H=H,
                               clusters=max(1, N // 100))
    inp = cuda_inputs(spec, seed=N)
    for flags in (0, mol.MOL_FLAG_BF16X2_GATING):
        prob = mol.Problem.from_inputs(inp, flags=flags)
        s, i = mol.topk_exact(prob, k)
        bs, bi = mol.topk_exact_bounded(prob, k, s[:, k - 1].contiguous())
        every = torch.arange(N, dtype=torch.int32, device="cuda").repeat(B, 1)
        if N <= 16384:                                       # the two kernels, through the rerank of all items
            rs, ri, _ = mol.rerank(prob, every, k)
            assert torch.equal(rs, s) and torch.equal(ri, i)
        assert torch.equal(bs, s) and torch.equal(bi, i)
        f32 = mol.score(mol.Problem.from_inputs(inp, flags=mol.MOL_FLAG_F32_GATING))
        want = torch.topk(f32, k, dim=1).values
        got = torch.gather(f32, 1, i.long())
        assert (s - got).abs().max() <= 2e-5 and (got - want).abs().max() <= 4e-5


def test_dense_slabs_of_queries():
    """A batch whose dense scores pass the buffer and whose list form would
    leave CUs idle runs in slabs of queries: the rows of the allocation-free
    (list) form, bit for bit, the last slab included."""
    spec = W["exact_32k"].scaled(B=1090, N=131101, clusters=512)
    inp = cuda_inputs(spec, seed=8)
    for flags in (0, mol.MOL_FLAG_BF16X2_GATING):
        prob = mol.Problem.from_inputs(inp, flags=flags)
        # slabs: about half a gigabyte of scores; the list form needs a few MB
        assert mol.mol_workspace_size(prob, mol.MOL_OP_TOPK_EXACT, k=50) > 256 << 20
        s, i = mol.topk_exact(prob, 50)
        ns, ni = torch.empty_like(s), torch.empty_like(i)
        mol.mol_topk_exact_noalloc(prob, 50, ns, ni)
        torch.cuda.synchronize()
        assert torch.equal(ns, s) and torch.equal(ni, i)


def test_workspace_without_room_for_dense_scores():
    """A workspace kept for a larger batch can be smaller than the dense form
    of this batch: the calls take the lists and return the same rows."""
    spec = W["exact_32k"].scaled(B=40, N=70001, clusters=256)
    prob = mol.Problem.from_inputs(cuda_inputs(spec, seed=5))
    small = mol.workspace(prob, mol.MOL_OP_TOPK_BOUNDED, k=50)      # the lists' size
    assert small.numel() < mol.mol_workspace_size(prob, mol.MOL_OP_TOPK_EXACT, k=50)
    s, i = mol.topk_exact(prob, 50)
    ls, li = mol.topk_exact(prob, 50, ws=small)
    torch.cuda.synchronize()
    assert torch.equal(s, ls) and torch.equal(i, li)
    with pytest.raises(mol.MolError):
        mol.topk_exact(prob, 50, ws=small[:-256])


# lists of more than 256 keys are ranked by bins of the score range: the bin
# limit (64 keys of one score), more (the bitonic network), more than the list
# holds (the radix search), and k with a few and with all keys above it
@pytest.mark.parametrize("ties,kp,N", [
    (0, 300, 3000), (63, 300, 20011), (65, 1000, 60001), (64, 513, 50000), (3000, 2048, 60001), (5000, 2048, 200001),
    (0, 2048, 200001),
])
def test_long_lists_with_ties(ties, kp, N):
    log(f"[long lists] ties={ties} k'={kp} N={N}")
    g = torch.Generator(device="cuda").manual_seed(N + ties)
    Q = torch.nn.functional.normalize(torch.randn((3, 1, 64), generator=g, device="cuda"), dim=-1).bfloat16()
    X = torch.nn.functional.normalize(torch.randn((1, N, 64), generator=g, device="cuda"), dim=-1).bfloat16()
    if ties:
        at = torch.randperm(N, generator=torch.Generator().manual_seed(4))[:ties].cuda()
        X[:, at] = torch.nn.functional.normalize(Q[0, 0].float() + 2 * X[0, at[0]].float(), dim=-1).bfloat16()
    dots, ids = mol.topk_per_embd(mol.Problem(Q, X), kp)
    torch.cuda.synchronize()
    s = Q[:, 0].double() @ X[0].double().t().contiguous()
    want = torch.topk(s, kp, dim=1).values
    got = torch.gather(s, 1, ids[:, 0].long())
    tol = 64 * 2.0 ** -24                                    # float32 sums of 64 products of unit rows
    assert (dots[:, 0].double() - got).abs().max() <= tol and (got - want).abs().max() <= 2 * tol
    assert _ordered(dots[:, 0], ids[:, 0]) and all(torch.unique(ids[b, 0]).numel() == kp for b in range(3))
