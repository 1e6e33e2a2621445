"""XOR responses over blocks so wide that their column slices take several
launches."""
import pytest

from _util import banner

pytestmark = pytest.mark.gpu


def test_wide_blocks(gpu):
    import torch
    import paper_2510_03631_amd as qp
    rows, W = 2, (1 << 29) + 5
    banner(f"chor wide {rows}x{W}")
    DB = torch.empty((rows, W), dtype=torch.int32, device="cuda")
    DB.random_(-(1 << 31), (1 << 31) - 1)
    Q = torch.tensor([[1], [3]], dtype=torch.int32, device="cuda")
    out = qp.chor_answer(DB, Q)
    assert torch.equal(out[0], DB[0])
    assert torch.equal(out[1], DB[0].bitwise_xor_(DB[1]))
