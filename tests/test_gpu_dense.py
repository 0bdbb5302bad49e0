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
