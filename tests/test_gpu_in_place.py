"""Batched answers written over their own queries: the queries are read before
anything is stored over them.  Equality with the oracle."""
import numpy as np
import pytest

import oracle
import workload
from _util import banner, to_dev_u32, to_dev_u8, to_host_u32

pytestmark = pytest.mark.gpu
P = 4294967291


@pytest.fixture(scope="module")
def qp(gpu):
    import paper_2510_03631_amd as p
    return p


@pytest.mark.parametrize("N", [15, 257, 1024, 2100])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 9])
def test_answers_over_queries(qp, N, B):
    banner(f"in place {N}x{N} B={B}")
    g = np.random.default_rng(N + B)
    D = workload.db_bytes(g, N, N)
    Q = workload.uniform_u32(g, (N, B))
    ref = oracle.answer_batch(D, Q)
    with qp.Database(to_dev_u8(D)) as db:
        q = to_dev_u32(Q)
        assert np.array_equal(to_host_u32(db.answer_batch(q, out=q)), ref)
        q = to_dev_u32(Q)
        assert np.array_equal(to_host_u32(db.answer_batch_noalloc(q, q)), ref)
        q = to_dev_u32(np.ascontiguousarray(Q.T))
        assert np.array_equal(to_host_u32(db.answer_batch_qmajor(q, out=q)), ref.T)
        if B <= 4:
            q = to_dev_u32(Q)
            assert np.array_equal(to_host_u32(db.answer_batch_modp(q, P, out=q)),
                                  oracle.answer_batch_mod(D, Q, P))
