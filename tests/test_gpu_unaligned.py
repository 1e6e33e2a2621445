"""Databases whose rows start anywhere and have any length: the byte stream's
chunks, slices, column splits and ragged last pieces, and the refresh.
Results are whole numbers: equality with the oracle."""
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


def resident(D: np.ndarray, pad: int, shift: int):
    """D on the device with rows `pad` bytes apart more than their length,
    starting `shift` bytes past an aligned address; nothing after the last
    row's bytes belongs to the tensor."""
    import torch
    R, C = D.shape
    store = torch.zeros(shift + (R - 1) * (C + pad) + C, dtype=torch.uint8, device="cuda")
    view = torch.as_strided(store, (R, C), (C + pad, 1), shift)
    view.copy_(to_dev_u8(D))
    return view


@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 0), (9, 5)])
@pytest.mark.parametrize("R,C", [(1, 1), (5, 15), (9, 16), (70, 17), (3, 1023), (33, 1025),
                                 (130, 4097), (300, 8193), (17, 40001)])
def test_stream_ragged(qp, R, C, pad, shift):
    banner(f"stream {R}x{C} pad={pad} shift={shift}")
    g = np.random.default_rng(R * 31 + C + pad)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, 4))
    with qp.Database(resident(D, pad, shift)) as db:
        for name in qp.variant_names(0):
            db.set_variant(0, name)
            a = to_host_u32(db.answer(to_dev_u32(Q[:, 0])))
            assert np.array_equal(a, oracle.answer(D, Q[:, 0])), name
        for B in (1, 2, 3, 4):
            db.set_variant(B, "few")
            q = np.ascontiguousarray(Q[:, :B])
            assert np.array_equal(to_host_u32(db.answer_batch(to_dev_u32(q))),
                                  oracle.answer_batch(D, q)), B
            assert np.array_equal(to_host_u32(db.answer_batch_modp(to_dev_u32(q), P)),
                                  oracle.answer_batch_mod(D, q, P)), B


@pytest.mark.parametrize("R,C", [(16385, 16391), (3001, 90001)])
def test_stream_large_ragged(qp, R, C):
    """The large database's row blocks, whole and split by columns."""
    banner(f"stream large {R}x{C}")
    D_d = workload.device_db(R, C, workload.SEED_BASE + 5, "cuda")
    D = D_d.cpu().numpy()
    q = workload.uniform_u32(workload.rng(3), (C,))
    with qp.Database(D_d) as db:
        assert np.array_equal(to_host_u32(db.answer(to_dev_u32(q))), oracle.answer(D, q))
        out = to_host_u32(db.answer_batch(to_dev_u32(q[:, None])))
        assert np.array_equal(out[:, 0], oracle.answer(D, q))


@pytest.mark.parametrize("pad,shift", [(0, 0), (7, 3)])
@pytest.mark.parametrize("R,C,m", [(3, 5, 3), (40, 16, 1), (300, 4111, 37), (50, 70003, 2)])
def test_refresh_ragged(qp, R, C, m, pad, shift):
    """A refresh writes the rows and their sums (which the batched product
    reads), and nothing beside them."""
    import torch
    banner(f"refresh {R}x{C} m={m} pad={pad} shift={shift}")
    g = np.random.default_rng(R + C + m)
    D = workload.db_bytes(g, R, C)
    rows = workload.distinct_rows(g, R, m)
    new = workload.db_bytes(g, m, C)
    Q = workload.uniform_u32(g, (C, 5))
    view = resident(D, pad, shift)
    with qp.Database(view) as db:
        listed = to_dev_u32(np.concatenate([rows, [R]]).astype(np.uint32))   # one past the end
        db.update_rows(listed[:m], to_dev_u8(new))
        if m < R:
            db.update_rows(listed[m:], torch.zeros((1, C), dtype=torch.uint8, device="cuda"))
        D[rows] = new
        assert np.array_equal(view.cpu().numpy(), D)
        assert np.array_equal(to_host_u32(db.answer_batch(to_dev_u32(Q))),
                              oracle.answer_batch(D, Q))


@pytest.mark.parametrize("pad,shift", [(0, 0), (9, 5), (None, 0)])
@pytest.mark.parametrize("R,C", [(1, 1), (3, 15), (40, 17), (127, 127), (129, 129), (257, 255),
                                 (300, 1000), (513, 4113)])
def test_batch_ragged(qp, R, C, pad, shift):
    """The batched product's tiles, split-K pieces and ragged last k-tile on
    unaligned rows and (pad None) on aligned rows of odd length, and the
    incremental hint on some of the rows."""
    if pad is None:
        pad = -C % 16
    banner(f"batch {R}x{C} pad={pad} shift={shift}")
    g = np.random.default_rng(R * 17 + C + pad)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, 130))
    D[0], Q[:, 0] = 0x80, 0x80808080            # the centred products' extremes
    D[-1], Q[:, -1] = 0xFF, 0xFFFFFFFF
    ref = oracle.answer_batch(D, Q)
    with qp.Database(resident(D, pad, shift)) as db:
        for B in (3, 32, 33, 64, 130):
            q = to_dev_u32(np.ascontiguousarray(Q[:, -B:]))
            assert np.array_equal(to_host_u32(db.answer_batch(q)), ref[:, -B:]), B
            assert np.array_equal(to_host_u32(db.answer_batch_qmajor(q.t().contiguous())),
                                  ref[:, -B:].T), B
        rows = workload.distinct_rows(g, R, (R + 2) // 3)
        H = to_dev_u32(np.zeros((R, 130), dtype=np.uint32))
        got = to_host_u32(db.hint_update_rows(to_dev_u32(rows), to_dev_u32(Q), H))
        want = np.zeros_like(ref)
        want[rows] = ref[rows]
        assert np.array_equal(got, want)


def test_noalloc_keeps_fitting(qp):
    """256 queries on an unaligned database: the split product's partials
    (over 80 MB) do not fit the fixed scratch, the whole product does."""
    import torch
    banner("noalloc 20000x1007 B=256")
    R, C, B = 20000, 1007, 256
    g = np.random.default_rng(8)
    D = workload.db_bytes(g, R, C)
    Q = workload.uniform_u32(g, (C, B))
    with qp.Database(to_dev_u8(D)) as db:
        out = torch.empty((R, B), dtype=torch.int32, device="cuda")
        got = to_host_u32(db.answer_batch_noalloc(to_dev_u32(Q), out))
        assert np.array_equal(got, to_host_u32(db.answer_batch(to_dev_u32(Q))))
    assert np.array_equal(got[::997], oracle.answer_batch(D[::997], Q))
