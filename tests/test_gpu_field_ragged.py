"""The field form's small batches on databases above 16 MiB whose rows are
aligned but no multiple of 16 long (and unaligned ones): equality with the
oracle."""
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


@pytest.mark.parametrize("R,C,pitch", [(4096, 8200, 8208), (1700, 10007, 10240), (2100, 8003, 8003)])
def test_field_ragged_rows(qp, R, C, pitch):
    import torch
    g = np.random.default_rng(R + C)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, 4))
    buf = torch.zeros((R, pitch), dtype=torch.uint8, device="cuda")
    buf[:, :C] = to_dev_u8(D)
    with qp.Database(buf[:, :C]) as db:
        for B in (1, 2, 3, 4):
            banner(f"field ragged {R}x{C} pitch={pitch} B={B}")
            q = np.ascontiguousarray(Q[:, :B])
            got = to_host_u32(db.answer_batch_modp(to_dev_u32(q), workload.FTR_PRIME))
            assert np.array_equal(got, oracle.answer_batch_mod(D, q, workload.FTR_PRIME)), B
