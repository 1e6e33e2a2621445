"""Answers stored four rows at a time (query-major answers, and the client
steps' epilogues inside the product): row counts around multiples of four and
of the tiles, split and whole products, every layout, and unaligned operands,
which take the other route.  Results are whole numbers: equality."""
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


@pytest.mark.parametrize("R,C", [(4, 16), (6, 5008), (128, 300), (132, 4096), (257, 2048),
                                 (300, 33)])
def test_query_major_rows(qp, R, C):
    import torch
    banner(f"query-major {R}x{C}")
    g = np.random.default_rng(R + C)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (70, C))
    ref = oracle.answer_batch(D, np.ascontiguousarray(Q.T)).T
    with qp.Database(to_dev_u8(D)) as db:
        for B in (3, 8, 16, 33, 70):
            Qd = to_dev_u32(Q[:B])
            for name in ["auto"] + [n for n in qp.variant_names(B) if n.startswith("narrow")]:
                try:
                    db.set_variant(B, name)
                except qp.PirError:
                    continue
                got = to_host_u32(db.answer_batch_qmajor(Qd))
                assert np.array_equal(got, ref[:B]), (B, name)
            # Answers at an address that is not 16-byte aligned.
            out = torch.zeros(B * R + 1, dtype=torch.int32, device="cuda")[1:].view(B, R)
            assert np.array_equal(to_host_u32(db.answer_batch_qmajor(Qd, out=out)), ref[:B]), B


@pytest.mark.parametrize("n", [1, 3, 32, 33, 64, 100, 128, 257])
@pytest.mark.parametrize("rows", [4, 130, 1000, 4100])
def test_client_products(qp, rows, n):
    """Byte planes narrower than, equal to and wider than a k-tile."""
    import torch
    banner(f"client products rows={rows} n={n}")
    g = np.random.default_rng(rows * 3 + n)
    M = workload.uniform_u32(g, (rows, n))
    M[0] = 0xFFFFFFFF
    M[-1] = 0x80808080
    S = workload.uniform_u32(g, (130, n))
    S[0] = 0xFFFFFFFF
    S[-1] = 0
    E = workload.lwe_error(g, (130, rows))
    cols = g.integers(0, rows, size=130).astype(np.uint32)
    cols[:2] = (0, rows - 1)
    ans = workload.uniform_u32(g, (130, rows))
    queries = np.stack([oracle.lwe_query(M, S[b], E[b], int(cols[b])) for b in range(130)])
    decoded = np.stack([oracle.lwe_decode(ans[b], M, S[b]) for b in range(130)])
    with qp.ClientMatrix(to_dev_u32(M)) as m:
        for B in (1, 5, 32, 33, 64, 130):
            Sd, Ed = to_dev_u32(S[:B]), to_dev_u32(E[:B].view(np.uint32))
            cd, ad = to_dev_u32(cols[:B]), to_dev_u32(ans[:B])
            assert np.array_equal(to_host_u32(m.query(Sd, Ed, cd)), queries[:B]), B
            assert np.array_equal(m.decode(Sd, ad).cpu().numpy(), decoded[:B]), B
        # Errors and answers at unaligned addresses.
        B = 5
        store = torch.zeros(B * rows + 1, dtype=torch.int32, device="cuda")
        view = store[1:].view(B, rows)
        view.copy_(to_dev_u32(E[:B].view(np.uint32)))
        Sd, cd = to_dev_u32(S[:B]), to_dev_u32(cols[:B])
        assert np.array_equal(to_host_u32(m.query(Sd, view, cd)), queries[:B])
        view.copy_(to_dev_u32(ans[:B]))
        assert np.array_equal(m.decode(Sd, view).cpu().numpy(), decoded[:B])
