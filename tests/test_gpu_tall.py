"""The single query on databases of very many short rows."""
import pytest

from _util import banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C", [((1 << 28) - 3, 1), ((1 << 29) + 3, 1)])
def test_answer_tall(gpu, R, C):
    import torch
    import paper_2510_03631_amd as qp
    banner(f"tall {R}x{C}")
    D = torch.empty((R, C), dtype=torch.uint8, device="cuda")
    D.random_(0, 256)
    q = torch.tensor([-1640531527], dtype=torch.int32, device="cuda")
    with qp.Database(D) as db:
        a = db.answer(q)
    ref = D[:, 0].to(torch.int32).mul_(q)          # wraps modulo 2^32
    assert torch.equal(a, ref)
