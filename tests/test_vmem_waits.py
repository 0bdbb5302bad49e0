"""gfx950 assembly of the rerank kernel: its wait for the gathered operands
holds whatever follows the copies, and nothing waits for them before it (CPU
only: hipcc cross-compiles)."""
import os

import pytest

from test_mfma_hazards import HIPCC, _asm
from vmem_waits import copy_drains, copy_waits


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_rerank_waits_for_its_gathers(tmp_path):
    asm = _asm("mol_rerank.hip", str(tmp_path))
    waits = copy_waits(asm, "k_mol_rerank")
    assert len(waits) == 8                       # four shapes, two gating chains
    for name, admitted, younger in waits:
        assert admitted <= younger, f"{name}: vmcnt({admitted}) with {younger} operations behind the copies"
    # the gathers of the next step stay in flight under the step's own chain
    for name, drained in copy_drains(asm, "k_mol_rerank"):
        assert drained == 0, f"{name}: the copies are waited for before the MFMAs"
