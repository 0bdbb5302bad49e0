"""A workspace kept for a larger batch serves every smaller one: the least that
an entry point takes for the smaller batch is within what mol_workspace_size
gives for the larger.  Sizes only: nothing is launched (CPU only)."""
import ctypes
import re

import pytest

from paper_2407_15462_amd import mol

FAKE = 256   # every call below stops at its workspace check


def _problem(B, N, Pq, Px, d, H, dtype=mol.MOL_BF16, flags=0):
    return mol.MolProblemC(B, N, Pq, Px, d, H, dtype, *([FAKE] * 8), flags)


def _size(c, op, k, C):
    out = ctypes.c_size_t(0)
    assert mol.load().mol_workspace_size(ctypes.byref(c), op, k, k, C, ctypes.byref(out)) == mol.MOL_OK
    return out.value


def _least(c, op, k, C):
    """Bytes that the entry point asks for when handed 16."""
    lib, r, ws = mol.load(), ctypes.byref(c), (FAKE, 16, None)
    rc = {
        mol.MOL_OP_TOPK_EXACT: lambda: lib.mol_topk_exact(r, k, FAKE, FAKE, *ws),
        mol.MOL_OP_TOPK_BOUNDED: lambda: lib.mol_topk_exact_bounded(r, k, FAKE, FAKE, FAKE, *ws),
        mol.MOL_OP_TOPK_TWO_PASS: lambda: lib.mol_topk_two_pass(r, k, 0, FAKE, FAKE, None, *ws),
        mol.MOL_OP_TOPK_MAXDOT: lambda: lib.mol_topk_maxdot(r, k, FAKE, FAKE, *ws),
        mol.MOL_OP_TOPK_PER_EMBD: lambda: lib.mol_topk_per_embd(r, k, FAKE, FAKE, *ws),
        mol.MOL_OP_RERANK: lambda: lib.mol_rerank(r, FAKE, C, None, 0, k, FAKE, FAKE, None, *ws),
    }[op]()
    assert rc == mol.MOL_EWORKSPACE
    return int(re.search(rb"needs (\d+)", lib.mol_last_error()).group(1))


F32 = dict(dtype=mol.MOL_F32)


# (operation, N, shape, options, k, C): corpora whose dense forms end within
# the batches below, shapes with and without their own kernels, k on both sides
# of the kernels' limits
@pytest.mark.parametrize("op,N,shape,opt,k,C", [
    (mol.MOL_OP_TOPK_PER_EMBD, 1 << 20, (1, 1, 64, 1), {}, 300, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 8388608, (1, 1, 128, 1), {}, 500, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 1 << 20, (8, 8, 64, 1), {}, 300, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 674044, (1, 1, 32, 1), {}, 500, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 1273943, (4, 4, 64, 1), {}, 585, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 109739, (4, 4, 768, 1), {}, 50, 0),
    (mol.MOL_OP_TOPK_PER_EMBD, 100003, (8, 4, 64, 1), {}, 128, 0),
    (mol.MOL_OP_TOPK_BOUNDED, 100000, (6, 6, 64, 64), {}, 100, 0),
    (mol.MOL_OP_TOPK_BOUNDED, 1008018, (64, 1, 64, 64), {}, 4, 0),
    (mol.MOL_OP_TOPK_BOUNDED, 100000, (4, 4, 768, 64), {"flags": mol.MOL_FLAG_F32_GATING}, 12, 0),
    (mol.MOL_OP_TOPK_MAXDOT, 1 << 20, (8, 8, 64, 1), F32, 100, 0),
    (mol.MOL_OP_TOPK_MAXDOT, 121592, (6, 6, 64, 1), {}, 70, 0),
    (mol.MOL_OP_TOPK_TWO_PASS, 100000, (6, 6, 64, 64), {}, 100, 0),
    (mol.MOL_OP_TOPK_TWO_PASS, 537014, (8, 4, 64, 64), {"flags": mol.MOL_FLAG_F32_GATING}, 25, 0),
    (mol.MOL_OP_TOPK_TWO_PASS, 283186, (8, 8, 64, 96), {}, 9, 0),
    (mol.MOL_OP_TOPK_EXACT, 1 << 20, (8, 8, 64, 64), {}, 100, 0),
    (mol.MOL_OP_TOPK_EXACT, 24186, (8, 4, 128, 128), {}, 100, 0),
    (mol.MOL_OP_TOPK_EXACT, 53585, (2, 32, 96, 256), {}, 500, 0),
    (mol.MOL_OP_TOPK_EXACT, 65537, (4, 4, 64, 32), F32, 10, 0),
    (mol.MOL_OP_RERANK, 1 << 20, (16, 4, 64, 64), {}, 70, 7317),
    (mol.MOL_OP_RERANK, 1 << 20, (8, 8, 64, 64), {}, 235, 16384),
])
def test_workspace_of_a_larger_batch_is_enough(op, N, shape, opt, k, C):
    batches = [1, 2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 40, 53, 64, 66, 74, 100, 128, 129, 199, 200, 255, 256, 257,
               500, 512, 641, 1000, 1024, 1025, 1170, 1171, 2000, 2048, 2656, 4095, 4096, 5000]
    if op == mol.MOL_OP_TOPK_EXACT and shape[0] == 8:
        # the fused shapes' lists (a few MB) follow the ranges that fill the
        # chip, whose number falls where a batch begins another query group
        batches = [B for B in batches if B & (B - 1) == 0]
    size = {B: _size(_problem(B, N, *shape, **opt), op, k, C) for B in batches}
    for i, B in enumerate(batches):
        least = _least(_problem(B, N, *shape, **opt), op, k, C)
        assert least <= size[B]
        for larger in batches[i + 1:]:
            assert least <= size[larger], f"B = {B} needs {least} bytes, {size[larger]} are kept for {larger}"


# the same over k: the dense forms' rule and buffers change with it
@pytest.mark.parametrize("op,B,N,shape,opt", [
    (mol.MOL_OP_TOPK_EXACT, 5, 109036, (1, 1, 128, 64), {}),
    (mol.MOL_OP_TOPK_EXACT, 32, 20000, (8, 8, 64, 64), {}),
    (mol.MOL_OP_TOPK_MAXDOT, 643, 47421, (1, 1, 33, 16), {}),
    (mol.MOL_OP_TOPK_PER_EMBD, 141, 1716, (4, 4, 64, 32), {}),
    (mol.MOL_OP_TOPK_PER_EMBD, 8, 160706, (1, 1, 128, 64), {}),
    (mol.MOL_OP_TOPK_BOUNDED, 64, 20000, (6, 6, 64, 64), {}),
])
def test_workspace_of_a_longer_list_is_enough(op, B, N, shape, opt):
    ks = [k for k in (1, 5, 64, 100, 128, 129, 200, 256, 257, 300, 512, 513, 700, 1024, 1025, 2048, 2049, 5000, 8192)
          if k <= N]
    c = _problem(B, N, *shape, **opt)
    size = {k: _size(c, op, k, 0) for k in ks}
    for i, k in enumerate(ks):
        least = _least(c, op, k, 0)
        for larger in ks[i:]:
            assert least <= size[larger], f"k = {k} needs {least} bytes, {size[larger]} are kept for {larger}"
