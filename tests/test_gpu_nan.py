"""Scores that overflow to NaN: ranked behind every number where sort keys rank
them, in the dense forms as in the streamed ones (MI355X only)."""
import pytest
import torch

from paper_2407_15462_amd import mol
from parity_helpers import log

pytestmark = pytest.mark.gpu


def _problem(B, N, Pq, Px, d, H, dtype, flags=0, scale=3e5, qscale=1.0, every=7):
    """Unit rows, but every `every`-th item so large that its dots overflow."""
    g = torch.Generator(device="cuda").manual_seed(1)

    def randn(*shape):
        return 0.3 * torch.randn(shape, generator=g, device="cuda")

    def unit(*shape):
        return torch.nn.functional.normalize(torch.randn(shape, generator=g, device="cuda"), dim=-1)

    P = Pq * Px
    Q, X = unit(B, Pq, d) * qscale, unit(Px, N, d)
    X[:, ::every] *= scale
    return mol.Problem(Q.to(dtype), X.to(dtype), randn(B, P), randn(N, P), randn(H, P).to(dtype), randn(H),
                       randn(P, H).to(dtype), randn(P), flags=flags)


def _check_rows(s, i, n, every=7):
    """Every one of n items once: numbers descending, then NaN by index, all of
    them among the large items."""
    s, i = s.reshape(-1, s.shape[-1]), i.reshape(-1, i.shape[-1])
    nan = torch.isnan(s)
    assert bool(nan.any()) and torch.equal(torch.sort(i, dim=1).values.long(), torch.arange(n).repeat(len(i), 1).cuda())
    for b in range(len(s)):
        m = int(nan[b].sum())
        assert not bool(nan[b, :n - m].any())
        assert bool((s[b, 1:n - m] <= s[b, :n - m - 1]).all())
        assert bool((i[b, n - m:] % every == 0).all()) and bool((i[b, n - m + 1:] > i[b, n - m:-1]).all())


BIG = dict(scale=1e30, qscale=1e12)   # past float32


# the f16 and two-term chains in the pair-wise kernels, dots and gating in one
# kernel, float32; with and without bucket maxima
@pytest.mark.parametrize("N,shape,kw", [
    (1000, (6, 6, 64, 64, torch.bfloat16), {}),
    (1000, (4, 3, 64, 64, torch.bfloat16), {}),
    (1000, (6, 6, 64, 64, torch.bfloat16), dict(flags=mol.MOL_FLAG_BF16X2_GATING, **BIG)),
    (1000, (4, 4, 64, 64, torch.bfloat16), {}),
    (1000, (4, 4, 64, 32, torch.float32), BIG),
    (1000, (8, 8, 64, 64, torch.bfloat16), dict(flags=mol.MOL_FLAG_F32_GATING, **BIG)),
])
def test_nan_scores_come_last(N, shape, kw):
    log(f"[nan] N={N} {shape} {kw}")
    prob = _problem(3, N, *shape, **kw)
    s, i = mol.topk_exact(prob, N)
    _check_rows(s, i, N)
    low = torch.full((prob.B,), -torch.finfo(torch.float32).max, device="cuda")
    bs, bi = mol.topk_exact_bounded(prob, N, low)
    if shape[4] == torch.float32 or kw.get("flags") == mol.MOL_FLAG_F32_GATING:
        assert torch.equal(bi, i) and torch.equal(torch.nan_to_num(bs), torch.nan_to_num(s))
    none = mol.topk_exact_bounded(prob, 10, torch.full_like(low, torch.inf))[1][:, 0]
    every = torch.arange(N, dtype=torch.int32, device="cuda").repeat(prob.B, 1)
    rs, ri, _ = mol.rerank(prob, every, N)
    _check_rows(rs, ri, N)
    # Algorithm 1: where G holds a NaN score (finite dots: the large items lead
    # the lists), the smallest score is NaN, no bound, and the exact rows follow
    ts, ti, tb = mol.topk_two_pass(prob, 20)
    torch.cuda.synchronize()
    assert torch.equal(ti, i[:, :20]) and torch.equal(ts, s[:, :20])
    if not kw:
        assert bool(torch.isnan(tb).all()) and bool((none == -1).all())


def test_nan_behind_bucket_maxima():
    """Long rows: fewer numbers than k in all, a bucket of nothing but NaN, and
    a row of 16,384 items that has enough numbers."""
    N = 20000
    for every, k in ((1, 100), (7, 100)):
        prob = _problem(3, N, 4, 4, 64, 64, torch.bfloat16, every=every)
        s, i = mol.topk_exact(prob, k)
        torch.cuda.synchronize()
        nan = torch.isnan(s)
        assert bool((i >= 0).all())
        for b in range(prob.B):
            m = int(nan[b].sum())
            assert torch.unique(i[b]).numel() == k and not bool(nan[b, :k - m].any())
            assert m == 0 or bool((i[b, k - m + 1:] > i[b, k - m:-1]).all())


@pytest.mark.parametrize("shape", [(6, 6, 64, 16, torch.bfloat16), (4, 4, 96, 16, torch.bfloat16)])
def test_nan_dots_come_last(shape):
    prob = _problem(2, 1000, *shape, scale=3e37, qscale=1e12)
    if shape[2] == 96:
        s, i = mol.topk_per_embd(prob, 1000)
    else:
        s, i = mol.topk_maxdot(prob, 1000)
    torch.cuda.synchronize()
    _check_rows(s, i, 1000)


def test_running_lists_drop_nan():
    """The P_q = 8 kernels with k <= 128: never ranked, the rest padded, the
    same rows from the dense form and the lists."""
    prob = _problem(3, 128, 8, 4, 64, 64, torch.bfloat16)
    s, i = mol.topk_exact(prob, 128)
    ns, ni = torch.empty_like(s), torch.empty_like(i)
    mol.mol_topk_exact_noalloc(prob, 128, ns, ni)
    torch.cuda.synchronize()
    assert torch.equal(s, ns) and torch.equal(i, ni)
    assert not bool(torch.isnan(s).any()) and bool((i == -1).any(dim=1).all())
