"""The float32 scoring kernel and the dense-row top-k against float64
references, at the sizes where their tiles and branches end (MI355X only)."""
import pytest
import torch

from paper_2407_15462_amd import mol
from parity_helpers import log

pytestmark = pytest.mark.gpu


def _problem(B, N, Pq, Px, d, H, dtype, flags=0, seed=0, offset=0, std=0.5):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def unit(*shape):
        v = torch.randn(shape, generator=g, device="cuda")
        return (v / v.norm(dim=-1, keepdim=True)).to(dtype)

    def off(t):   # the same values `offset` elements past a 16-byte boundary
        buf = torch.empty(t.numel() + offset, dtype=t.dtype, device="cuda")
        buf[offset:] = t.reshape(-1)
        return buf[offset:].view(t.shape)

    P = Pq * Px
    r = lambda *s: std * torch.randn(s, generator=g, device="cuda")   # noqa: E731
    t = (off(unit(B, Pq, d)), off(unit(Px, N, d)), off(r(B, P)), off(r(N, P)), r(H, P).to(dtype), r(H),
         r(P, H).to(dtype), r(P))
    return mol.Problem(*t, flags=flags), t


def _phi64(t):
    Q, X, a_q, a_x, W1, b1, W2, b2 = (x.double() for x in t)
    B, Pq, d = Q.shape
    Px, N, _ = X.shape
    s = torch.stack([Q.reshape(B * Pq, d) @ X[px].t().contiguous() for px in range(Px)], 1)   # [B Pq][Px][N]
    s = s.view(B, Pq * Px, N).permute(0, 2, 1).reshape(B * N, Pq * Px)
    u = s @ W1.t().contiguous() + b1
    lg = (u * torch.sigmoid(u)) @ W2.t().contiguous() + b2
    lg = lg.view(B, N, -1) + a_q[:, None] + a_x[None]
    return (torch.softmax(lg, -1) * s.view(B, N, -1)).sum(-1), s.view(B, N, -1)


def _rel(got, want):
    return (got.double() - want).norm() / want.norm()


# P at and around 16, 32 and 64; H not a multiple of 16 and the largest; d
# whole chunks, a partial chunk, odd (element reads); batches that leave a
# partial query block; items that leave a partial tile
@pytest.mark.parametrize("B,N,Pq,Px,d,H,dtype,offset", [
    (1, 33, 1, 1, 8, 1, torch.float32, 0),
    (9, 1000, 4, 4, 64, 32, torch.float32, 0),
    (5, 517, 4, 4, 20, 17, torch.float32, 0),
    (3, 300, 3, 5, 7, 40, torch.float32, 0),
    (3, 129, 17, 1, 64, 33, torch.float32, 1),
    (6, 257, 8, 4, 36, 64, torch.float32, 0),
    (5, 130, 8, 8, 64, 64, torch.float32, 0),
    (2, 70, 2, 32, 96, 256, torch.float32, 0),
    (1, 700, 7, 9, 1024, 16, torch.float32, 0),
    (2, 70, 64, 1, 16, 250, torch.bfloat16, 0),
    (5, 333, 8, 8, 64, 64, torch.bfloat16, 0),
    (3, 100, 5, 3, 40, 48, torch.bfloat16, 0),
    (3, 100, 4, 4, 33, 48, torch.bfloat16, 3),
])
def test_f32_scores_topk_rerank(B, N, Pq, Px, d, H, dtype, offset):
    log(f"[f32] B={B} N={N} P={Pq}x{Px} d={d} H={H} {dtype} offset={offset}")
    prob, t = _problem(B, N, Pq, Px, d, H, dtype, mol.MOL_FLAG_F32_GATING, seed=B * N, offset=offset)
    phi = mol.score(prob)
    part = mol.score(prob, 7, N - 11)
    k = min(N, 20)
    s, i = mol.topk_exact(prob, k)
    bs, bi = mol.topk_exact_bounded(prob, k, s[:, k - 1].contiguous())
    cand = torch.randint(-2, N, (B, 67), device="cuda", dtype=torch.int32,
                         generator=torch.Generator(device="cuda").manual_seed(4))
    rs, ri, rn = mol.rerank(prob, cand, k)
    ms, mi = mol.topk_maxdot(prob, k)
    ps, pi = mol.topk_per_embd(prob, k)
    torch.cuda.synchronize()
    want, dots = _phi64(t)
    # Float32 errors seen over these rows: 2-norm up to 1.1e-6 of the result's,
    # largest up to 5.5e-6 of its RMS, dots (|s| <= 1) up to 1.8e-7.  The bounds
    # are two, three and five times that; the two-term chain is past the first
    # two where a shape has it (3.7e-6 and 3.1e-5), the f16 chain far past.
    rel, worst, tol = 2e-6, 1.5e-5, 1e-6
    assert _rel(phi, want) <= rel and (phi.double() - want).abs().max() <= worst * want.square().mean().sqrt()
    if dtype == torch.bfloat16 and Pq == 8:
        for flags in (0, mol.MOL_FLAG_BF16X2_GATING):
            assert _rel(mol.score(mol.Problem(*t, flags=flags)), want) > rel
    assert torch.equal(part, phi[:, 7:N - 4])
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])     # the kernel's own scores, exactly
    assert torch.equal(bs, s) and torch.equal(bi, i)
    for b in range(B):
        ids = torch.unique(cand[b][cand[b] >= 0].long())
        assert int(rn[b]) == ids.numel()
        o = torch.sort(phi[b, ids], descending=True, stable=True)
        n = min(k, ids.numel())
        assert torch.equal(rs[b, :n], o.values[:n]) and torch.equal(ri[b, :n].long(), ids[o.indices[:n]])
        assert bool((ri[b, n:] == -1).all())
    assert (ms.double() - torch.sort(dots.amax(-1), dim=1, descending=True).values[:, :k]).abs().max() <= tol
    top = torch.sort(dots.permute(0, 2, 1), dim=2, descending=True).values[..., :k]
    assert (ps.double() - top).abs().max() <= tol
    got = torch.gather(dots.permute(0, 2, 1), 2, pi.long())
    assert (ps.double() - got).abs().max() <= tol


# rows shorter than a workgroup, around it, and long; k at both ends of the
# kernel's range; more tied items than the LDS list holds (the radix finish)
@pytest.mark.parametrize("N,k,ties", [
    (1, 1, 0), (63, 63, 0), (700, 512, 0), (1025, 100, 0), (4099, 512, 0), (40001, 1, 0), (40001, 300, 9000),
    (40001, 512, 40001), (40001, 100, 39950),
])
def test_dense_topk_is_exact(N, k, ties):
    log(f"[dense topk] N={N} k={k} ties={ties}")
    prob, t = _problem(3, N, 2, 2, 16, 16, torch.float32, seed=N + k)
    X = t[1]
    if ties:   # identical items: equal scores, ranked by index
        at = torch.randperm(N, generator=torch.Generator().manual_seed(1))[:ties].cuda()
        X[:, at] = X[:, at[:1]]
        t[3][at] = t[3][at[:1]]
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, k)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])


# both workgroup sizes of the selection: rows up to four values a thread of the
# small one and more, few and many rows, k around half its threads, with and
# without bucket maxima; rows ranked whole and just not; more tied items than
# the small list holds (the radix finish)
@pytest.mark.parametrize("B,N,k,ties", [
    (2, 128, 128, 0), (2, 129, 128, 0), (5, 1024, 128, 0), (5, 1025, 128, 0), (5, 1024, 129, 0), (513, 1025, 128, 0),
    (512, 1025, 1, 0), (600, 3001, 129, 0), (600, 16383, 128, 0), (520, 20011, 100, 0), (520, 20011, 10, 4000),
    (600, 2000, 100, 1500), (3, 1000, 128, 900), (513, 172, 172, 0), (513, 1024, 512, 0), (513, 1024, 513, 0),
    (512, 1024, 200, 0), (600, 1000, 300, 900), (513, 1025, 200, 0), (257, 3072, 128, 0),
    (257, 3073, 128, 0), (256, 3072, 10, 0), (300, 3000, 50, 1200),
])
def test_dense_topk_workgroups(B, N, k, ties):
    log(f"[dense topk] B={B} N={N} k={k} ties={ties}")
    prob, t = _problem(B, N, 2, 2, 16, 16, torch.float32, seed=N + k)
    if ties:
        at = torch.randperm(N, generator=torch.Generator().manual_seed(1))[:ties].cuda()
        t[1][:, at] = t[1][:, at[:1]]
        t[3][at] = t[3][at[:1]]
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, k)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])


# more tied items than the list holds: a query of zeros, ties of the best item,
# ties behind k / 3 others, two blocks, and ties of a negative score behind five
# positive ones; both workgroup sizes, with and without bucket maxima
@pytest.mark.parametrize("B,N,k", [(3, 9000, 100), (3, 20011, 200), (2, 200003, 100), (2, 300003, 2000), (2, 300003, 1),
                                   (600, 3001, 100), (520, 20000, 128)])
@pytest.mark.parametrize("tied", ["all", "best", "behind", "two", "negative"])
def test_dense_topk_ties(B, N, k, tied):
    log(f"[dense topk ties] B={B} N={N} k={k} {tied}")
    prob, t = _problem(B, N, 2, 2, 16, 16, torch.float32, seed=N + k)
    Q, X, a_x = t[0], t[1], t[3]
    order = torch.argsort(mol.score(prob)[0], descending=True)

    def tie(at, to):
        X[:, at] = X[:, to:to + 1].clone()
        a_x[at] = a_x[to:to + 1].clone()

    if tied == "all":
        Q.zero_()
    elif tied == "negative":
        tie(order[5:N - 500], int(order[N - 500]))
    else:
        first = k // 3 if tied == "behind" else 0
        if tied == "two":
            tie(order[1:k // 2], int(order[0]))
            first = k // 2
        tie(order[first:N - 300], int(order[first]))
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, k)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])


@pytest.mark.parametrize("B,N,k", [(2, 200003, 100), (520, 20000, 100), (2, 300003, 2000)])
def test_dense_topk_of_sorted_rows(B, N, k):
    """The best items side by side: more items reach the threshold than the
    list holds, in buckets that it does."""
    prob, t = _problem(B, N, 2, 2, 16, 16, torch.float32, seed=N + k)
    order = torch.argsort(mol.score(prob)[0], descending=True)
    t[1].copy_(t[1][:, order].clone())
    t[3].copy_(t[3][order].clone())
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, k)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :k]) and torch.equal(i.long(), wi[:, :k])


def test_long_rows_without_scores():
    """Every column excluded, or all but a few, of more buckets than the
    selection collects."""
    prob, _ = _problem(2, 300001, 2, 2, 16, 16, torch.float32, seed=1)
    m, at = mol.topk_maxdot(prob, 6)
    s, i = mol.topk_exact_bounded(prob, 100, torch.tensor([torch.inf, (m[1, 4] + 0.01).item()], device="cuda"))
    torch.cuda.synchronize()
    assert bool((i[0] == -1).all()) and bool(torch.isneginf(s[0]).all())
    n = int((i[1] >= 0).sum())
    assert n < 100 and bool((i[1, n:] == -1).all()) and set(i[1, :n].tolist()) <= set(range(prob.N))
    assert torch.equal(s[1, :n], mol.score(prob)[1, i[1, :n].long()])


def test_rerank_of_tied_candidates():
    """A query of zeros: the k smallest ids of more candidates than the list holds."""
    prob, t = _problem(3, 100003, 2, 2, 16, 16, torch.float32)
    t[0][1].zero_()
    cand = torch.stack([torch.randperm(prob.N, generator=torch.Generator().manual_seed(b))[:9001] for b in range(3)])
    s, i, nu = mol.rerank(prob, cand.int().cuda(), 100)
    torch.cuda.synchronize()
    assert nu.tolist() == [9001] * 3
    assert torch.equal(i[1].long().cpu(), torch.sort(cand[1]).values[:100]) and bool((s[1] == 0).all())
    phi = mol.score(prob)
    for b in (0, 2):
        assert torch.equal(s[b], torch.sort(phi[b, cand[b].cuda()], descending=True).values[:100])


@pytest.mark.parametrize("B", [1, 8, 16])     # four, two and one slices of bucket maxima
def test_query_of_zeros(B):
    """Every item tied, of more buckets than the selection collects: the first k.
    Then the corpus in the order of a query's scores."""
    g = torch.Generator(device="cuda").manual_seed(1)
    r = lambda *s: 0.1 * torch.randn(s, generator=g, device="cuda")   # noqa: E731
    Q, X = r(B, 8, 32).bfloat16(), r(8, 400003, 32).bfloat16()
    Q[B - 1] = 0
    prob = mol.Problem(Q, X, r(B, 64), r(400003, 64), r(64, 64).bfloat16(), r(64), r(64, 64).bfloat16(), r(64))
    s, i = mol.topk_exact(prob, 100)
    torch.cuda.synchronize()
    assert bool((s[B - 1] == 0).all()) and torch.equal(i[B - 1].long().cpu(), torch.arange(100))
    if B > 1:
        order = torch.argsort(mol.score(prob)[0], descending=True)
        prob = mol.Problem(Q, X[:, order].contiguous(), r(B, 64), r(400003, 64), *[x.zero_() for x in (
            r(64, 64).bfloat16(), r(64), r(64, 64).bfloat16(), r(64))])
    phi = mol.score(prob)
    s, i = mol.topk_exact(prob, 100)
    torch.cuda.synchronize()
    ws, wi = torch.sort(phi, dim=1, descending=True, stable=True)
    assert torch.equal(s, ws[:, :100]) and torch.equal(i.long(), wi[:, :100])
