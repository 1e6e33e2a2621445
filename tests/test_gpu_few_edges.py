"""The small-batch stream on both sides of its tile and split rules: equality
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


@pytest.mark.parametrize("R,C", [(16383, 300), (16385, 300), (16390, 4097), (700, 9001), (300, 4097),
                                 (2304, 7777), (1030, 16289), (5, 70001)])
def test_few_edges(qp, R, C):
    banner(f"few edges {R}x{C}")
    g = np.random.default_rng(R + C)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, 2))
    with qp.Database(to_dev_u8(D)) as db:
        for B in (1, 2):
            q = np.ascontiguousarray(Q[:, :B])
            assert np.array_equal(to_host_u32(db.answer_batch(to_dev_u32(q))),
                                  oracle.answer_batch(D, q)), B
            assert np.array_equal(to_host_u32(db.answer_batch_modp(to_dev_u32(q), workload.FTR_PRIME)),
                                  oracle.answer_batch_mod(D, q, workload.FTR_PRIME)), B
