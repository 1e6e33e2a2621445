"""The built-in choice of tile and split for shapes and batches around the
lines where it changes: narrow tiles on rows of any length, the few-query
stream up to 16 MiB, few rows with many columns (many pieces), and the same
answers from the allocation-free call.  Results are whole numbers: equality."""
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


@pytest.mark.parametrize("R,C,pad", [(3, 70001, -70001 % 16), (130, 4099, 13), (129, 40007, 9),
                                     (4096, 4096, 0), (4097, 4096, 0), (300, 60000, 0),
                                     (300, 60000, 3)])
def test_default_choice(qp, R, C, pad):
    import torch
    banner(f"default tiles {R}x{C} pad={pad}")
    g = np.random.default_rng(R + C + pad)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, 70))
    D[-1], Q[:, 0], Q[:, 1] = 0xFF, 0xFFFFFFFF, 0
    ref = oracle.answer_batch(D, Q)
    store = torch.zeros((R, C + pad), dtype=torch.uint8, device="cuda")
    store[:, :C] = to_dev_u8(D)
    with qp.Database(store[:, :C]) as db:
        for B in (1, 2, 3, 4, 5, 8, 9, 16, 17, 33, 70):
            q = to_dev_u32(np.ascontiguousarray(Q[:, :B]))
            assert np.array_equal(to_host_u32(db.answer_batch(q)), ref[:, :B]), B
            assert np.array_equal(to_host_u32(db.answer_batch_qmajor(q.t().contiguous())),
                                  ref[:, :B].T), B
            out = torch.zeros((R, B), dtype=torch.int32, device="cuda")
            db.answer_batch_noalloc(q, out)
            assert np.array_equal(to_host_u32(out), ref[:, :B]), B
