"""The fused rerank at the ends of a wave's chunk of candidates, against the
dense scores of the same problem (MI355X only)."""
import pytest
import torch

import synth
from paper_2407_15462_amd import mol
from parity_helpers import cuda_inputs, log

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


# candidates of a query: one step of a wave (1 to 16), a step and one more, a
# whole chunk of 32 and one more, and several chunks with a one-step tail; a
# query without any
@pytest.mark.parametrize("wl", ["exact_32k", "exact_1m", "hybrid_8m", "paper_books"])
@pytest.mark.parametrize("flags", [0, mol.MOL_FLAG_BF16X2_GATING])
def test_rerank_chunk_ends(wl, flags):
    counts = [1, 15, 16, 17, 31, 32, 33, 0, 64, 65, 97, 128]
    C = max(counts)                              # = k, the largest of the fused rerank
    log(f"[rerank ends] {wl} flags={flags} counts={counts}")
    spec = W[wl].scaled(B=len(counts), N=5003, clusters=16)
    prob = mol.Problem.from_inputs(cuda_inputs(spec, seed=29), flags=flags)
    phi = mol.score(prob)
    cand = torch.full((spec.B, C), -1, dtype=torch.int32, device="cuda")
    gen = torch.Generator().manual_seed(3)
    for b, n in enumerate(counts):
        cand[b, C - n:] = torch.randperm(spec.N, generator=gen)[:n].int().cuda()
    s, i, nu = mol.rerank(prob, cand, C)
    torch.cuda.synchronize()
    assert nu.tolist() == counts
    for b, n in enumerate(counts):
        ids = i[b, :n].long()
        assert torch.equal(torch.sort(ids).values, torch.sort(cand[b, C - n:].long()).values)
        # both chains' stated error at std 0.1, ten times over
        assert n == 0 or (s[b, :n] - phi[b, ids]).abs().max() <= 2e-5
        assert bool((s[b, 1:n] <= s[b, :max(n - 1, 0)]).all())
        assert bool((i[b, n:] == -1).all()) and bool(torch.isneginf(s[b, n:]).all())
