"""gfx950 assembly of the rerank kernel: its wait for the gathered operands
holds whatever follows the copies (CPU only: hipcc cross-compiles)."""
import os

import pytest

from test_mfma_hazards import HIPCC, _asm
from vmem_waits import copy_waits


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_rerank_waits_for_its_gathers(tmp_path):
    waits = copy_waits(_asm("mol_rerank.hip", str(tmp_path)), "k_mol_rerank")
    assert len(waits) == 8                       # four shapes, two gating chains
    for name, admitted, younger in waits:
        assert admitted <= younger, f"{name}: vmcnt({admitted}) with {younger} operations behind the copies"
