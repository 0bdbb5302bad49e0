"""Static check of gfx950 assembly: the counted wait in front of LDS reads of
direct global -> LDS copies admits no more outstanding vector-memory
operations than are certain to be younger than the last of those copies.

Vector-memory operations complete in order, so s_vmcnt(n) proves that the
copies have landed only if at least n operations were issued behind them on
every path.  The certain ones are those in the copies' own basic block: an
operation behind a branch may be skipped."""
from __future__ import annotations

import re
from typing import List, Tuple


def _lines(func: str):
    for ln in func.split("\n"):
        s = ln.strip()
        if s.startswith(";;#ASM"):
            yield s
            continue
        s = s.split(";")[0].strip()
        if s and (not s.startswith(".") or s.startswith(".LBB")):
            yield s


def copy_waits(asm: str, kernel: str) -> List[Tuple[str, int, int]]:
    """(function, admitted by the wait, certainly younger than the copies) of
    every function whose name contains ``kernel``.  The explicit wait stands
    alone between two empty asm statements (compiler barriers)."""
    out = []
    for func in re.split(r"\n(?=_Z\w+:)", asm)[1:]:
        func = func.split(".Lfunc_end")[0]
        name = func.split(":")[0]
        if kernel not in name:
            continue
        lines = list(_lines(func))
        younger, n, open_ = [], 0, False
        for s in lines:
            op = s.split()[0]
            if op.startswith("global_load_lds"):
                n, open_ = 0, True
            elif open_ and re.match(r"(global|buffer|flat)_", op):
                n += 1
            elif open_ and (s.startswith(".LBB") or op.startswith(("s_cbranch", "s_branch", "s_endpgm"))):
                younger.append(n)
                open_ = False
        text = "\n".join(lines)
        waits = re.findall(r";;#ASMSTART\n;;#ASMEND\ns_waitcnt vmcnt\((\d+)\)\n;;#ASMSTART\n;;#ASMEND\n", text)
        assert younger and waits, name
        out.append((name, max(int(w) for w in waits), min(younger)))
    return out


def copy_drains(asm: str, kernel: str) -> List[Tuple[str, int]]:
    """(function, number of runs of copies that a vector-memory wait follows
    before the block's last MFMA) where the copies and MFMAs share a block."""
    out = []
    for func in re.split(r"\n(?=_Z\w+:)", asm)[1:]:
        func = func.split(".Lfunc_end")[0]
        name = func.split(":")[0]
        if kernel not in name:
            continue
        blocks, blk = [], []
        for s in _lines(func):
            if s.startswith(".LBB") or s.split()[0].startswith(("s_cbranch", "s_branch", "s_endpgm")):
                blocks.append(blk)
                blk = []
            else:
                blk.append(s)
        shared, drained = 0, 0
        for blk in blocks:
            copies = [i for i, s in enumerate(blk) if s.startswith("global_load_lds")]
            mfmas = [i for i, s in enumerate(blk) if s.startswith("v_mfma")]
            if not copies or not mfmas:
                continue
            shared += 1
            drained += any(s.startswith("s_waitcnt") and "vmcnt" in s for s in blk[copies[0]:mfmas[-1]])
        assert shared, name
        out.append((name, drained))
    return out
