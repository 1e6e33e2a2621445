"""The batched calls' plans (status, kernel, split-K pieces, scratch) over
shapes, alignments and forms, from the library's own planner on the CPU."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_03631_amd")
OK, SHAPE, UNSUPPORTED = 0, 2, 5
P = 4294967291


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    """Run the planner on a list of calls; one list of words for each."""
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "native", "plan_probe.cpp"),
                    "-o", exe, os.path.join(PKG, "libqpir.so"), "-L/opt/rocm/lib", "-lamdhip64",
                    f"-Wl,-rpath,{PKG},-rpath,/opt/rocm/lib"], check=True)

    def run(calls):
        text = "".join(" ".join(str(x) for x in c) + "\n" for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        lines = [l.split() for l in out.splitlines()]
        assert len(lines) == len(calls)
        return lines
    return run


def pitch16(C):
    return (C + 15) // 16 * 16


def test_field_form_serves_up_to_four_queries_everywhere(probe):
    """Aligned and unaligned rows, lengths that are and are not multiples of
    16, below and above 16 MiB; more queries need rows of whole 16-byte
    pieces at aligned addresses."""
    rng = random.Random(1)
    calls = []
    for R, C in [(4096, 8200), (20000, 10007), (1000, 100), (3, 5), (4096, 8192), (30000, 30000)] + [
            (rng.randint(1, 1 << 18), rng.randint(1, 1 << 16)) for _ in range(300)]:
        for B in (1, 2, 3, 4, 5, 8, 64, 200):
            for pitch, aligned in ((pitch16(C), 1), (C, int(C % 16 == 0)), (pitch16(C), 0)):
                calls.append(("batch", R, C, pitch, aligned, B, P, 0, 0))
    for c, r in zip(calls, probe(calls)):
        served = c[5] <= 4 or (c[4] and c[2] % 16 == 0)
        assert int(r[0]) == (OK if served else UNSUPPORTED), (c, r)


def test_noalloc_serves_what_its_planes_allow(probe):
    """Three and more queries are refused only where the limb planes (4 bytes
    a query and column, queries and columns padded) alone pass the scratch."""
    rng = random.Random(2)
    calls = []
    for R, C in [(1 << 24, 1), (2808755, 2), (7000000, 1), (1 << 21, 8), (1 << 22, 4)] + [
            (rng.randint(1, 1 << rng.randint(4, 24)), rng.randint(1, 1 << rng.randint(3, 17)))
            for _ in range(300)]:
        for B in (3, 4, 5, 16, 64, 200):
            calls.append(("noalloc", R, C, pitch16(C), 1, B))
            calls.append(("noalloc", R, C, C, int(C % 16 == 0), B))
    for c, r in zip(calls, probe(calls)):
        Bp = 32 if c[5] <= 32 else (c[5] + 63) // 64 * 64
        planes = 4 * Bp * ((c[2] + 255) // 256 * 256) + 8 * Bp + 512
        if planes <= 64 << 20:
            assert int(r[0]) == OK, (c, r)


def test_single_query_grid_fits(probe):
    """A launch holds fewer than 2^32 threads along x, for any row count up
    to 2^30 (and beyond)."""
    calls = [("answer", R, C, C, int(C % 16 == 0), 0)
             for R in (1, 1 << 20, (1 << 28) - 15, (1 << 28) - 3, 1 << 28, 1 << 29, (1 << 29) + 3,
                       (1 << 30) - 1, (1 << 31) - 200)
             for C in (1, 2, 16, 100, 256, 1 << 10)]
    for c, r in zip(calls, probe(calls)):
        assert int(r[1]) * int(r[3]) < 1 << 32, (c, r)


def test_single_query_fills_the_chip(probe):
    """Large databases of any shape run in about as many workgroups as
    CUs (the last round at most an eighth empty): few rows by splitting
    their columns."""
    calls = [("answer", R, C, C, int(C % 16 == 0), 0)
             for R, C in [(64, 1 << 22), (1, 1 << 28), (16, 1 << 25), (300, 10 ** 6), (500, 600000),
                          (1000, 300000), (1100, 300000), (2000, 131072), (4352, 42752),
                          (3072, 1 << 18), (6320, 24320)]]
    for c, r in zip(calls, probe(calls)):
        assert int(r[1]) * int(r[2]) >= 224, (c, r)


@pytest.mark.parametrize("R,C,B,rows,whole", [
    (1024, 1024, 1, 16, True), (2048, 3001, 2, 16, True), (4096, 4096, 2, 16, True),
    (3072, 8192, 1, 16, False), (3072, 8192, 2, 64, False), (3000, 11008, 2, 64, False),
    (16384, 1500, 1, 64, True), (16384, 1500, 2, 64, True), (100000, 160, 1, 64, True),
    (100000, 160, 2, 64, True), (8192, 8192, 1, 64, False), (8192, 8192, 4, 64, False)])
def test_small_batch_stream_tiles(probe, R, C, B, rows, whole):
    """The measured faster of 16 and 64 rows a workgroup, and one launch where
    a split costs more than it gives."""
    r = probe([("few", R, C, C, int(C % 16 == 0), B)])[0]
    assert int(r[0]) == rows and (int(r[1]) == 1) == whole, r


def test_workspace_holds_every_plan(probe):
    """No call needs more than the workspace reported for its batch, whatever
    its rows, form and pinned kernel, and the whole database's largest call
    and the gathered ones of every tile count come near it."""
    rng = random.Random(3)
    calls = []
    for _ in range(4000):
        R = max(1, round(2 ** rng.uniform(0, 18)))
        C = max(1, round(2 ** rng.uniform(4, 18)))
        C = max(16, C // 16 * 16) if rng.random() < 0.5 else C
        aligned = int(rng.random() < 0.7)
        B = rng.choice((rng.randint(3, 16), rng.randint(17, 64), rng.randint(65, 300)))
        mod = P if rng.random() < 0.3 else 0
        for m in (0, 1, R, rng.randint(1, R), min(R, 128 * rng.randint(1, 40)),
                  min(R, 256 * rng.randint(1, 600))):
            calls.append(("batch", R, C, pitch16(C) if aligned else C, aligned, B, 0 if m else mod, m,
                          rng.choice((0, 0, rng.randint(1, 25)))))
    for c, r in zip(calls, probe(calls)):
        assert int(r[0]) in (OK, UNSUPPORTED) and int(r[4]) <= int(r[5]), (c, r)


def test_workspace_is_no_larger_than_plans_need(probe):
    """Short rows: splitting them gains little, so little is reserved for it
    (megabytes; without the product's times in the bound these took 134, 80
    and 107)."""
    calls = [("batch", 194870, 482, 482, 0, 128, 0, 0, 0), ("batch", 122601, 207, 207, 0, 41, 0, 0, 0),
             ("batch", 96382, 511, 512, 1, 51, 0, 0, 0)]
    for c, r in zip(calls, probe(calls)):
        assert int(r[5]) < 8 << 20, (c, r)


def ktile(name):
    return 128 if "_k128" in name or name.startswith("reg") else 64


def test_fitting_keeps_the_field_forms_pieces(probe):
    """The field form's accumulators cover at most 2^17 columns a piece: a
    plan cut to a scratch keeps that (and then passes the scratch)."""
    calls = [("fit", R, C, C, 1, B, P, scratch)
             for R, C in ((3072, 1 << 18), (500, 1 << 20), (40000, 1 << 18), (3072, 1 << 15))
             for B in (5, 40, 200) for scratch in (1 << 16, 1 << 24, 1 << 28)]
    for c, r in zip(calls, probe(calls)):
        assert int(r[2]) * ktile(r[0]) <= 1 << 17, (c, r)


def test_fitting_cuts_to_what_the_scratch_holds(probe):
    """Plans whose partials pass the scratch get the pieces that fit, down to
    one, and are left alone where they fit."""
    rng = random.Random(4)
    calls, cut, whole = [], 0, 0
    for _ in range(6000):
        R, C = round(2 ** rng.uniform(4, 16)), round(2 ** rng.uniform(8, 18))
        B, aligned = rng.randint(5, 200), rng.randint(0, 1)
        base = ("fit", R, C, pitch16(C) if aligned else C, aligned, B, 0)
        calls += [base + (1 << 60,), base + (round(2 ** rng.uniform(14, 29)),)]
    out = probe(calls)
    for c, full, r in zip(calls[1::2], out[0::2], out[1::2]):
        splits, kts, need = (int(x) for x in r[1:])
        part, ktiles = 4 * c[1] * c[5], -(-c[2] // ktile(r[0]))
        planes = int(full[3]) - (part * int(full[1]) if int(full[1]) > 1 else 0)
        assert splits * kts >= ktiles and (splits - 1) * kts < ktiles, (c, r)
        assert need == planes + (part * splits if splits > 1 else 0), (c, full, r)
        if int(full[3]) <= c[7]:
            assert r == full
        else:
            assert need <= max(c[7], planes), (c, full, r)
            if int(full[1]) > 1:
                assert splits < int(full[1]), (c, full, r)
                cut += splits > 1
                whole += splits == 1
    assert cut > 50 and whole > 50


@pytest.mark.parametrize("R,C,pad,B,pieces", [
    (168, 85906, 0, 130, "some"), (355, 86016, 0, 183, "some"), (234, 130684, 0, 78, "one"),
    (624, 64400, 0, 224, "one"), (556, 65098, 6, 243, "one")])
def test_noalloc_calls_that_are_cut(probe, R, C, pad, B, pieces):
    """The calls that tests/test_gpu_noalloc_shapes.py runs do pass the scratch
    uncut, and are cut to fewer pieces or to one."""
    pitch = C + pad
    full, r = probe([("fit", R, C, pitch, int(pitch % 16 == 0), B, 0, 1 << 60),
                     ("noalloc", R, C, pitch, int(pitch % 16 == 0), B)])
    assert int(full[3]) > 64 << 20 and int(r[0]) == OK and int(r[4]) <= 64 << 20
    assert int(r[2]) == 1 if pieces == "one" else 1 < int(r[2]) < int(full[1])


def test_kept_tile_choice(probe):
    """A handle's kept choice is the choice of a fresh handle, for each batch
    size and form, in any order."""
    rng = random.Random(5)
    kept, fresh = [], []
    for _ in range(500):
        R, C = round(2 ** rng.uniform(4, 16)), round(2 ** rng.uniform(4, 16)) // 16 * 16
        k = rng.randint(2, 8)
        B, other = rng.randint(2 ** (k - 1) + 1, 2 ** k), rng.randint(2 ** (k - 1) + 1, 2 ** k)
        kept.append(("kept", R, C, C, 1, B, P, other))
        fresh += [("batch", R, C, C, 1, b, m, 0, 0) for b, m in ((B, 0), (B, P), (other, 0))]
    out = probe(fresh)
    for i, r in enumerate(probe(kept)):
        a, b, c = (f"{x[0]}:{x[1]}" for x in out[3 * i:3 * i + 3])
        assert r == [a, b, c, a, b], (kept[i], r)


@pytest.mark.parametrize("R,C,few", [
    (1024, 1024, True), (4096, 4096, True), (3277, 1017, True), (13312, 72, True), (16384, 1, True),
    (16385, 64, False), (65536, 256, False), (1 << 20, 16, False), (30000, 3000, False)])
@pytest.mark.parametrize("B", [3, 4])
def test_stream_or_tile_for_three_and_four_queries(probe, R, C, few, B):
    """The dot4 stream up to 16 MiB, rows below 1024 bytes counted as 1024."""
    r = probe([("batch", R, C, pitch16(C), 1, B, 0, 0, 0)])[0]
    assert (r[1] == "few") == few


@pytest.mark.parametrize("R,C,B,splits", [(17784, 2343, 2, 2), (16384, 2048, 2, 1),
                                          (6144, 4352, 1, 1), (3072, 8192, 1, 4), (200, 100000, 1, 25)])
def test_small_batch_stream_pieces(probe, R, C, B, splits):
    assert int(probe([("few", R, C, C, int(C % 16 == 0), B)])[0][1]) == splits
