"""The allocation-free batched answer at the edges of its scratch: equality
with the oracle."""
import numpy as np
import pytest

import oracle
import workload
from _util import banner, to_dev_u32, to_dev_u8, to_host_u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qp(gpu):
    import paper_2510_03631_amd as p
    return p


@pytest.mark.parametrize("R,C", [((1 << 21) + 5, 7), ((1 << 21) + 1, 8), (1 << 20, 16)])
@pytest.mark.parametrize("B", [3, 4])
def test_noalloc_tall_narrow(qp, R, C, B):
    """Small batches on tall, narrow databases of up to 16 MiB."""
    import torch
    banner(f"noalloc {R}x{C} B={B}")
    g = np.random.default_rng(R + C + B)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, B))
    with qp.Database(to_dev_u8(D)) as db:
        out = torch.empty((R, B), dtype=torch.int32, device="cuda")
        got = to_host_u32(db.answer_batch_noalloc(to_dev_u32(Q), out))
    assert np.array_equal(got, oracle.answer_batch(D, Q))


# Rows, columns, row padding and queries of calls whose split product's
# partials pass the scratch beside the limb planes (tests/test_plans.py checks
# the piece counts: cut to 11, 4, one and one piece).
CUT = [(168, 85906, 0, 130), (355, 86016, 0, 183), (234, 130684, 0, 78), (624, 64400, 0, 224),
       (556, 65098, 6, 243)]


@pytest.mark.parametrize("R,C,pad,B", CUT)
def test_noalloc_cut_plans(qp, R, C, pad, B):
    import torch
    banner(f"noalloc cut {R}x{C} pad={pad} B={B}")
    g = np.random.default_rng(R + C + B)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, B))
    buf = torch.zeros((R, C + pad), dtype=torch.uint8, device="cuda")
    buf[:, :C] = to_dev_u8(D)
    with qp.Database(buf[:, :C]) as db:
        out = torch.empty((R, B), dtype=torch.int32, device="cuda")
        got = to_host_u32(db.answer_batch_noalloc(to_dev_u32(Q), out))
        assert np.array_equal(got, to_host_u32(db.answer_batch(to_dev_u32(Q))))
    assert np.array_equal(got[::37], oracle.answer_batch(D[::37], Q))
