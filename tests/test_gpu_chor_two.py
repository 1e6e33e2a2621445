"""Two XOR queries on databases large enough to be streamed: whole and ragged
row and word counts, padded and unaligned rows, sparse and dense selectors.
Equality with the oracle."""
import numpy as np
import pytest

import oracle
import workload
from _util import banner, to_dev_u32, to_host_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,W,pad", [(1 << 18, 768, 0), (239999, 777, 0), (380001, 500, 3),
                                        (65536, 2804, 4)])
def test_two_queries_streamed(gpu, rows, W, pad):
    import paper_2510_03631_amd as qp
    banner(f"chor two {rows}x{W} pad={pad}")
    DB_d = workload.device_u32((rows, W + pad), workload.SEED_BASE + 62, "cuda")[:, :W]
    DB = DB_d.cpu().numpy().view(np.uint32)
    g = workload.rng(workload.SEED_BASE + rows)
    Q = workload.chor_query_words(g, rows, 4)
    Q[2] = 0
    Q[2, [0, 7, -1]] = 1, 1 << 31, 1
    Q[3] = 0xFFFFFFFF
    if rows % 32:
        Q[:, -1] |= np.uint32(0xFFFFFFFF) << np.uint32(rows % 32)   # bits past the last row
    for pair in ([0, 1], [2, 3]):
        got = to_host_u32(qp.chor_answer(DB_d, to_dev_u32(Q[pair])))
        assert np.array_equal(got, oracle.chor_answer_batch(DB, Q[pair])), pair
