"""Column sums taken inside the batched product (tiles of up to 128 limb
rows): the query words whose centred sums are largest either way, split and
whole products, ragged columns, and both sides of the size from which the
ingest sums instead.  Results are whole numbers: equality."""
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


def answers(qp, D, Q, batches, names_of):
    """Every kernel of names_of(B) on the first B queries, against one oracle call."""
    ref = oracle.answer_batch(D, Q)
    ref_p = oracle.answer_batch_mod(D, Q, P)
    with qp.Database(to_dev_u8(D)) as db:
        for B in batches:
            q = to_dev_u32(np.ascontiguousarray(Q[:, :B]))
            for name in names_of(B):
                try:
                    db.set_variant(B, name)
                except qp.PirError:
                    continue
                assert np.array_equal(to_host_u32(db.answer_batch(q)), ref[:, :B]), (B, name)
                got = to_host_u32(db.answer_batch_modp(q, P))
                assert np.array_equal(got, ref_p[:, :B]), (B, name)


@pytest.mark.parametrize("R,C", [(1, 16), (127, 144), (129, 1008), (256, 20000), (513, 4096)])
def test_column_sums(qp, R, C):
    banner(f"column sums {R}x{C}")
    g = np.random.default_rng(R * 7 + C)
    D = workload.db_bytes(g, R, C)
    D[0], D[-1] = 0x80, 0xFF
    Q = workload.uniform_u32(g, (C, 37))
    Q[:, 0], Q[:, 1], Q[:, 2], Q[:, 3] = 0, 0x80808080, 0x7F7F7F7F, 0xFFFFFFFF
    answers(qp, D, Q, (4, 7, 8, 9, 32, 37),
            lambda B: ["auto"] + [n for n in qp.variant_names(B)
                                  if n.startswith("narrow") or "128x128" in n])


@pytest.mark.parametrize("R", [16384, 16385])
def test_who_sums(qp, R):
    banner(f"column sums {R}x16384")
    g = np.random.default_rng(R)
    D = workload.db_bytes(g, R, 16384)
    Q = workload.uniform_u32(g, (16384, 4))
    Q[:, 0], Q[:, 1] = 0xFFFFFFFF, 0
    answers(qp, D, Q, (4,), lambda B: ["ring_128x128_k128_s2"])
