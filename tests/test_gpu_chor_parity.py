"""XOR responses on the matrix cores at the edges of their tiles: query groups
of 32 and 64, column slices of 32 and 64 words, chunks of 128 rows, slabs, and
the largest count one accumulator holds.  Results are whole numbers: equality."""
import numpy as np
import pytest

import oracle
import workload
from _util import banner, to_dev_u32, to_host_u32

pytestmark = pytest.mark.gpu
M32 = 1 << 32


@pytest.fixture(scope="module")
def qp(gpu):
    import paper_2510_03631_amd as p
    return p


@pytest.mark.parametrize("B", [2, 32, 33, 64, 65, 129])
@pytest.mark.parametrize("rows,W,pad", [(127, 31, 0), (128, 32, 1), (129, 33, 0), (767, 63, 0),
                                        (768, 65, 5), (1000, 64, 0), (6401, 97, 3)])
def test_parity_edges(qp, rows, W, pad, B):
    banner(f"parity rows={rows} W={W} pad={pad} B={B}")
    g = np.random.default_rng(rows + W + B)
    DB = g.integers(0, M32, size=(rows, W + pad), dtype=np.uint32)
    Q = workload.chor_query_words(g, rows, B)
    got = to_host_u32(qp.chor_answer(to_dev_u32(DB)[:, :W], to_dev_u32(Q)))
    assert np.array_equal(got, oracle.chor_answer_batch(DB[:, :W], Q))


def test_parity_full_accumulator(qp):
    """Every selector and database bit set over 2^18 rows, a few taken out:
    counts around 2^18, the most one accumulator takes.  16384 queries of 64
    words fill the chip with one slab of all rows."""
    import torch
    banner("parity full accumulator")
    rows, W, B = 1 << 18, 64, 1 << 14
    DB = torch.full((rows, W), -1, dtype=torch.int32, device="cuda")
    DB[-1, 3] = 0
    DB[5, 7] = 0x12345678
    Q = torch.full((B, rows // 32), -1, dtype=torch.int32, device="cuda")
    Q[1::2, 100] = 0x7FFFFFFE
    out = to_host_u32(qp.chor_answer(DB, Q))
    ref = oracle.chor_answer_batch(DB.cpu().numpy().view(np.uint32),
                                   Q[:2].cpu().numpy().view(np.uint32))
    assert np.array_equal(out[0::2], np.broadcast_to(ref[0], (B // 2, W)))
    assert np.array_equal(out[1::2], np.broadcast_to(ref[1], (B // 2, W)))
