"""XOR responses on the matrix cores through the unclamped main loop, in each of
the kernel's forms: up to 32 queries (two column groups) and more, rows through
registers and straight to LDS, streamed past the last-level cache or not, and
one call of more rows than an accumulator counts.  Random data; sampled queries
against the oracle, and linearity over all of them."""
import numpy as np
import pytest

import oracle
import workload
from _util import banner, to_dev_u32, to_host_u32

pytestmark = pytest.mark.gpu
PAIR = 256                      # rows of a pair of chunks
FAST_ROWS = 4 * PAIR            # a slab of this many runs the main loop


def slab_rows(rows, W, B):
    """The launch rule's rows per slab."""
    tile, width = (32, 64) if B <= 32 else (64, 32)
    per_slab = -(-B // tile) * -(-W // width)
    pairs, lo = -(-rows // PAIR), -(-rows // (1 << 18))
    n = min(range(lo, max(lo, min(pairs, 64)) + 1),
            key=lambda n: -(-per_slab * n // 256) * (-(-pairs // n) + 3))
    return -(-pairs // n) * PAIR


@pytest.fixture(scope="module")
def words(gpu):
    """384 MiB of random words, on the device and the host."""
    d = workload.device_u32((1 << 17, 768), workload.SEED_BASE + 70, "cuda").view(-1)
    return d, d.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("rows,W,pitch,B", [
    (1 << 17, 768, 768, 2), (1 << 17, 768, 768, 17), (131071, 768, 768, 32),   # TM = 1, streamed
    (50001, 768, 768, 32), (40000, 777, 777, 5),                               # TM = 1
    (1 << 17, 768, 768, 33), (131001, 764, 768, 64),                           # LDS, streamed
    (60001, 768, 768, 100),                                                    # LDS
    (1 << 17, 767, 768, 40), (129000, 777, 777, 64),                           # registers, streamed
    (60001, 777, 777, 100), (70003, 769, 770, 65)])                            # registers
def test_main_loop(words, rows, W, pitch, B):
    import torch
    import paper_2510_03631_amd as qp
    banner(f"chor fast rows={rows} W={W} pitch={pitch} B={B}")
    assert slab_rows(rows, W, B) >= FAST_ROWS
    DB_d = torch.as_strided(words[0], (rows, W), (pitch, 1))
    DB = words[1][:rows * pitch].reshape(rows, pitch)[:, :W]
    g = workload.rng(workload.SEED_BASE + rows + B)
    Q = workload.chor_query_words(g, rows, B)
    out = to_host_u32(qp.chor_answer(DB_d, to_dev_u32(Q)))
    for b in sorted({0, B // 2, B - 1}):
        assert np.array_equal(out[b], oracle.chor_answer(DB, Q[b])), b
    for t in range(4):
        pick = g.random(B) < 0.5
        assert np.array_equal(np.bitwise_xor.reduce(out[pick], axis=0),
                              oracle.chor_answer(DB, np.bitwise_xor.reduce(Q[pick], axis=0))), t


def test_more_rows_than_an_accumulator_counts(words):
    """2^18 + 37 rows where the queries alone fill the chip: two slabs."""
    import torch
    import paper_2510_03631_amd as qp
    rows, W, B = (1 << 18) + 37, 64, 1 << 14
    banner(f"chor fast rows={rows} W={W} B={B}")
    assert slab_rows(rows, W, B) < rows <= 2 * slab_rows(rows, W, B)
    DB_d = torch.as_strided(words[0], (rows, W), (W, 1))
    DB = words[1][:rows * W].reshape(rows, W)
    Q_d = workload.device_u32((B, (rows + 31) // 32), workload.SEED_BASE + 71, "cuda")
    out = to_host_u32(qp.chor_answer(DB_d, Q_d))
    Q = Q_d[::1021].cpu().numpy().view(np.uint32)
    assert np.array_equal(out[::1021], oracle.chor_answer_batch(DB, Q))
