"""Every entry point in the least workspace that it takes gives the rows of the
preferred form (MI355X only)."""
import re

import pytest
import torch

from paper_2407_15462_amd import mol
from parity_helpers import log

pytestmark = pytest.mark.gpu


def _problem(B, N, Pq, Px, d, H, dtype=torch.bfloat16, flags=0, ties=0):
    g = torch.Generator(device="cuda").manual_seed(B + N)

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    def unit(*shape):
        return torch.nn.functional.normalize(randn(*shape), dim=-1).to(dtype)

    P = Pq * Px
    Q, X = unit(B, Pq, d), unit(Px, N, d)
    if ties:                                                 # more equal items than a list's key buffer holds
        at = torch.randperm(N, generator=torch.Generator().manual_seed(2))[:ties].cuda()
        X[:, at] = X[:, at[:1]]
        Q[0] = X[torch.arange(Pq) % Px, at[0]]
    return mol.Problem(Q, X, 0.1 * randn(B, P), 0.1 * randn(N, P), (0.1 * randn(H, P)).to(dtype), 0.1 * randn(H),
                       (0.1 * randn(P, H)).to(dtype), 0.1 * randn(P), flags=flags)


def _least(call):
    """Workspace of the size that `call` asks for when handed one byte."""
    with pytest.raises(mol.MolError) as e:
        call(torch.empty(1, dtype=torch.uint8, device="cuda"))
    assert e.value.status == mol.MOL_EWORKSPACE
    return torch.empty(int(re.search(r"needs (\d+)", str(e.value)).group(1)), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("what,args,kw,k", [
    ("exact", (40, 70001, 8, 4, 64, 64), {}, 50),                           # dense -> per-range lists
    ("exact", (4, 109036, 1, 1, 128, 64), {}, 1174),                        # key tiles -> dense rows
    ("exact", (1024, 100000, 6, 6, 64, 64), {}, 100),                       # dense -> key tiles
    ("bounded", (1024, 100000, 6, 6, 64, 64), {}, 100),
    ("maxdot", (128, 1 << 20, 4, 4, 32, 16), {"dtype": torch.float32}, 100),
    ("per_embd", (3, 200003, 1, 1, 64, 16), {}, 300),                       # dense -> the kernel, one range
    ("per_embd", (3, 50001, 8, 4, 64, 16), {"ties": 3000}, 100),            # appending form, one range for overflows
    ("per_embd", (40, 50001, 8, 8, 32, 16), {"ties": 3000}, 128),           # pruned form, the same
    ("per_embd", (128, 109739, 4, 4, 96, 16), {}, 50),                      # sampled threshold -> key tiles
    ("two_pass", (64, 20011, 6, 6, 64, 64), {}, 40),
    ("two_pass", (9, 20011, 8, 4, 64, 64), {"flags": mol.MOL_FLAG_F32_GATING}, 25),
])
def test_least_workspace_gives_the_same_rows(what, args, kw, k):
    log(f"[least workspace] {what} {args} {kw} k={k}")
    prob = _problem(*args, **kw)
    bound = torch.full((prob.B,), -1.0, device="cuda")
    call = {
        "exact": lambda ws: mol.topk_exact(prob, k, ws=ws),
        "bounded": lambda ws: mol.topk_exact_bounded(prob, k, bound, ws=ws),
        "maxdot": lambda ws: mol.topk_maxdot(prob, k, ws=ws),
        "per_embd": lambda ws: mol.topk_per_embd(prob, k, ws=ws),
        "two_pass": lambda ws: mol.topk_two_pass(prob, k, ws=ws)[:2],
    }[what]
    best = call(None)
    ws = _least(call)
    least = call(ws)
    torch.cuda.synchronize()
    # component dots are sums of d float32 products of unit rows in an order of
    # their own in each kernel; the MoL scores' chain is the same in all forms
    # of a shape (the rerank behind the two-pass bound aside, which only sets it)
    if what == "per_embd":
        assert (best[0] - least[0]).abs().max() <= prob.d * 2.0 ** -24
        same = best[1] == least[1]
        assert bool(((best[0] - least[0])[~same].abs() <= prob.d * 2.0 ** -24).all()) and same.float().mean() > 0.98
    else:
        assert torch.equal(best[0], least[0]) and torch.equal(best[1], least[1])
    with pytest.raises(mol.MolError):
        call(ws[:-256])


def test_rerank_without_room_for_the_dots():
    """Scored in float32: within the gating chain's stated error of the
    preferred form (2e-6 at std 0.1), ten times over."""
    prob = _problem(9, 5003, 6, 6, 64, 64)
    cand = torch.randint(-1, prob.N, (prob.B, 300), dtype=torch.int32, device="cuda",
                         generator=torch.Generator(device="cuda").manual_seed(1))
    best = mol.rerank(prob, cand, 300)
    least = mol.rerank(prob, cand, 300, ws=_least(lambda ws: mol.rerank(prob, cand, 300, ws=ws)))
    torch.cuda.synchronize()
    assert torch.equal(best[2], least[2])
    for b in range(prob.B):
        n = int(best[2][b])
        o, p = torch.argsort(best[1][b, :n]), torch.argsort(least[1][b, :n])
        assert torch.equal(best[1][b, o], least[1][b, p])
        assert (best[0][b, o] - least[0][b, p]).abs().max() <= 2e-5
