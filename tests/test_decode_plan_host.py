"""Launch plans of the decode kernel (token-axis splits of Eq. (3)) and where their partial results
lie in a workspace, from the library's own planning code; no GPU needed."""
import os
import random
import shutil
import subprocess

import pytest

from paper_2412_12706_amd import kvqp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FIELDS = ("accepted", "splits", "waves", "part_bytes", "part_off", "counters", "stated", "half", "chunks", "least")
PRICED, EQUAL_HEADS, OWN_COUNTS = 0, 1, 2        # the planner's answer; what a call launches, heads alike or with counts of their own
COUNTER_ROOM = 65536 * 4                         # opens every workspace of the stated size


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans([(batch, hq, hkv, n, bits, group, outliers, decode_splits, workspace bytes, key axis (0), form (PRICED)), ...]) -> dicts"""
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    if not os.path.exists(kvqp.LIB_PATH):
        from paper_2412_12706_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    lib_dir = os.path.dirname(kvqp.LIB_PATH)
    r = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                        "-I" + os.path.join(lib_dir, "csrc"), os.path.join(ROOT, "tests", "sanitize", "plan_driver.cpp"),
                        "-L" + lib_dir, "-lkvqp", "-Wl,-rpath," + lib_dir, "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]

    def ask(problems):
        r = subprocess.run([exe], input="".join(" ".join(map(str, (p + (0, PRICED))[:11])) + "\n" for p in problems), capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-3000:]
        rows = [dict(zip(FIELDS, map(int, line.split()))) for line in r.stdout.splitlines()]
        assert len(rows) == len(problems)
        return rows
    return ask


@pytest.mark.parametrize("hq,hkv,n,bits,group,outliers,splits", [
    (32, 8, 2048, 4, 32, 0, 0), (32, 8, 8192, 2, 32, 0, 0), (32, 8, 8192, 16, 32, 0, 0), (64, 8, 3000, 4, 128, 0, 0),
    (16, 8, 1000, 8, 64, 0, 0), (8, 8, 4096, 4, 32, 0, 0), (32, 8, 5000, 4, 32, 1, 0), (32, 8, 4096, 4, 32, 0, 7)])
def test_partials_stay_clear_of_every_counter_of_calls_that_share_a_workspace(plans, hq, hkv, n, bits, group, outliers, splits):
    """One workspace of the larger stated size, two batch sizes in turn: neither call's partial
    results may lie over the other's arrival counters, which have to be zero when it starts."""
    def problem(b, ws=0):
        return (b, hq, hkv, n, bits, group, outliers, splits, ws)
    own = {b: r for b, r in zip(range(1, 65), plans([problem(b) for b in range(1, 65)]))}
    pairs = [(a, b) for a in own for b in own if a != b]
    shared = [max(own[a]["stated"], own[b]["stated"]) for a, b in pairs]
    split = 0
    for (a, b), ws, p in zip(pairs, shared, plans([problem(a, ws) for (a, _), ws in zip(pairs, shared)])):
        assert p["accepted"] and p["splits"] == own[a]["splits"]
        if p["splits"] > 1:
            split += 1
            assert p["part_off"] >= max(own[a]["counters"], own[b]["counters"]), (a, b, p)
            assert p["part_off"] % 16 == 0 and p["part_off"] + p["part_bytes"] <= ws, (a, b, p)
    assert split > 500


@pytest.mark.parametrize("hq,hkv,n,bits", [(32, 8, 2048, 4), (16, 8, 1200, 4), (64, 8, 8192, 2)])
def test_smaller_workspaces_than_stated_are_taken_and_not_overrun(plans, hq, hkv, n, bits):
    """Down to the arrival counters and the plain rule's partials, and no further."""
    for b in (1, 3, 12, 19, 40, 44):
        whole = plans([(b, hq, hkv, n, bits, 32, 0, 0, 0)])[0]
        sizes = sorted({whole["counters"] + i * whole["stated"] // 40 // 16 * 16 for i in range(40)} | {whole["stated"]})
        rows = plans([(b, hq, hkv, n, bits, 32, 0, 0, ws) for ws in sizes])
        taken = [(ws, p) for ws, p in zip(sizes, rows) if p["accepted"]]
        assert taken and [p["accepted"] for p in rows] == sorted(p["accepted"] for p in rows)
        for ws, p in taken:
            assert p["part_bytes"] == 0 or (p["part_off"] >= p["counters"] and p["part_off"] + p["part_bytes"] <= ws), (b, ws, p)


def price(heads, gq, bits, group, outliers, n, waves, splits):
    """Predicted microseconds of a launch, in 64 bits, and the number of splits it comes to."""
    max_waves, n_cu = (12 if bits <= 4 and gq <= 4 and not outliers else 8), 256
    n_chunks = -(-n // 64)
    chunks = -(-n_chunks // splits)
    cut = -(-n_chunks // chunks)
    wgs, per_cu = heads * cut, max_waves // waves
    rounds, deep = -(-wgs // (n_cu * per_cu)), -(-wgs // n_cu)
    simd = 0.25 * waves * min(deep, per_cu)
    chunk = {2: 1.31 + 0.27 * simd, 4: 1.40 + 0.10 * simd, 8: 1.48 + 0.21 * simd, 16: 0.0}[bits]
    token = 512 if bits == 16 else 2 * (16 * bits + 512 // group) + (32 if outliers else 0)
    chip = heads * n * token * 1e-6 / 7.15
    streams = (rounds * -(-chunks // waves) * chunk * (1.47 if gq == 8 else 1)) ** 2 + chip ** 2 + (chip * deep * n_cu / wgs / 1.44) ** 2
    return 2.4 + 4.99 * rounds + streams ** 0.5 + (0.85 + 0.02 * cut * gq if cut > 1 else 0), cut


def test_the_search_passes_over_no_better_launch_shape(plans):
    """The planner's search, which leaves out numbers of splits that cannot win, against all pairs."""
    rng = random.Random(17)
    problems = []
    for _ in range(4000):
        bits = rng.choice([2, 4, 8, 16])
        problems.append((rng.randint(1, 80), rng.choice([1, 2, 4, 8]), rng.choice([1, 4, 8]), int(2 ** rng.uniform(0, 17)), bits,
                         rng.choice([32, 64, 128]), rng.choice([0, 0, 1]) if bits < 16 else 0))
    rows = plans([(b, hkv * gq, hkv, n, bits, g, o, 0, 0) for b, gq, hkv, n, bits, g, o in problems])
    other = 0
    for (b, gq, hkv, n, bits, g, o), row in zip(problems, rows):
        heads, max_waves, n_chunks = b * hkv, (12 if bits <= 4 and gq <= 4 and not o else 8), -(-n // 64)
        share = 256 * max_waves // heads
        waves = min(share, n_chunks)                                         # the plain rule
        if waves <= max_waves:
            plain = (max(4, waves // 4 * 4), 1)
        else:
            nw = max(4, min(max_waves, max(waves * heads // 256 // 4 * 4, -(-(-(-waves // 16)) // 4) * 4)))
            plain = (nw, -(-waves // nw))
        part = heads * gq * 1024                                             # bytes of a split's partials
        choice = [price(heads, gq, bits, g, o, n, w, s) for s in (1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32)
                  if s <= n_chunks and s <= -(-share // 4) and (s == 1 or row["counters"] + s * part <= 8 << 20)
                  for w in range(4, max_waves + 1, 4)]
        here = price(heads, gq, bits, g, o, n, row["waves"], row["splits"])[0]
        best = min([p for p, _ in choice], default=1e9)
        was, cut = price(heads, gq, bits, g, o, n, *plain)
        if best < 0.96 * was * (1 - 1e-5):
            other += 1
            assert here <= best * (1 + 1e-5), (b, gq, hkv, n, bits, g, o, row)
        elif best > 0.96 * was * (1 + 1e-5):
            assert (row["waves"], row["splits"]) == (plain[0], cut), (b, gq, hkv, n, bits, g, o, row)
    assert other > 800


def test_chunks_of_32_cover_the_tokens_within_the_stated_workspace(plans):
    """The form that small calls launch in place of the priced one: its workgroups take every token once, its partial results lie
    clear of all counters inside a workspace of the stated size, and it asks for no more than the plain rule."""
    rng = random.Random(23)
    problems = []
    for _ in range(20000):
        bits = rng.choice([2, 4, 8, 16])
        hkv = rng.choice([1, 2, 4, 8])
        problems.append((int(2 ** rng.uniform(0, 6)), hkv * rng.choice([1, 2, 4, 8]), hkv, int(2 ** rng.uniform(0, 13.2)), bits, rng.choice([32, 64, 128]),
                         int(bits < 16 and rng.random() < 0.1), rng.choice([0, 0, 0, 3]), 0, rng.choice([0, 1])))
    halves = split = 0
    for p, priced, row, own in zip(problems, *(plans([p + (form,) for p in problems]) for form in (PRICED, EQUAL_HEADS, OWN_COUNTS))):
        b, hq, hkv, n, bits, _, outliers, splits = p[:8]
        assert row["accepted"] and own["accepted"] and not own["half"] and row["least"] == priced["least"] == own["least"], p
        if not row["half"]:
            assert row == priced, p
            continue
        halves += 1
        split += row["splits"] > 1
        assert bits != 16 and not outliers and not splits and row["waves"] == 8, p
        assert row["splits"] <= 16 and b * hkv * row["splits"] <= 256, p
        assert (row["splits"] - 1) * row["chunks"] * 32 < n <= row["splits"] * row["chunks"] * 32 and row["chunks"] <= 16, p
        assert row["part_bytes"] == (b * hq * row["splits"] * 1024 if row["splits"] > 1 else 0), p
        assert row["part_off"] >= COUNTER_ROOM and row["part_off"] + row["part_bytes"] <= row["stated"], p
    assert halves > 2000 and split > 1000


@pytest.mark.parametrize("hq,hkv,n,bits", [(32, 8, 1024, 4), (8, 1, 3000, 8), (8, 8, 700, 2), (64, 8, 4000, 4)])
def test_chunks_of_32_give_way_in_a_smaller_workspace(plans, hq, hkv, n, bits):
    """A workspace that holds the plain rule's partials is taken, and one that has no room for this form's behind the counters gets
    the plain rule's launch."""
    for b in (1, 2):
        whole, plain = (plans([(b, hq, hkv, n, bits, 32, 0, 0, 0, 1, form)])[0] for form in (EQUAL_HEADS, OWN_COUNTS))
        assert whole["half"] and whole["part_bytes"] > 0
        room = COUNTER_ROOM + whole["part_bytes"]
        sizes = sorted({whole["least"] - 16, whole["least"], room - 16, room, whole["stated"]} | {whole["least"] + i * (room - whole["least"]) // 20 for i in range(20)})
        for ws, row in zip(sizes, plans([(b, hq, hkv, n, bits, 32, 0, 0, ws, 1, EQUAL_HEADS) for ws in sizes])):
            assert row["accepted"] == (ws >= whole["least"]), (b, ws)
            if not row["accepted"]:
                continue
            assert row["half"] == (ws >= room), (b, ws, row)
            assert row["half"] or all(row[f] == plain[f] for f in ("splits", "waves", "chunks", "part_bytes")), (b, ws, row)
            assert row["part_bytes"] == 0 or (row["part_off"] >= row["counters"] and row["part_off"] + row["part_bytes"] <= ws), (b, ws, row)


@pytest.mark.parametrize("hq,hkv,n,bits,group,axis,half", [
    (8, 8, 300, 2, 128, 0, 0), (8, 8, 300, 2, 128, 1, 1), (8, 8, 300, 2, 32, 0, 1), (8, 8, 256, 2, 128, 0, 1), (32, 8, 600, 2, 64, 0, 1), (32, 8, 800, 2, 64, 0, 0),
    (16, 8, 380, 4, 64, 0, 0), (32, 8, 380, 4, 64, 0, 1), (64, 8, 1100, 4, 128, 0, 1), (32, 8, 1100, 4, 128, 0, 0), (32, 8, 1024, 4, 32, 0, 1),
    (16, 8, 280, 8, 64, 0, 1), (16, 8, 450, 8, 64, 0, 0), (2, 2, 7700, 8, 64, 0, 0), (32, 8, 6700, 8, 64, 0, 1), (32, 8, 6700, 4, 64, 0, 0),
    (32, 8, 8192, 4, 32, 0, 1), (32, 8, 8193, 4, 32, 1, 0), (16, 16, 4180, 4, 64, 0, 0), (16, 16, 4180, 4, 64, 1, 1)])
def test_chunks_of_32_are_left_where_they_are_slower(plans, hq, hkv, n, bits, group, axis, half):
    """Both sides of each line of the rule: per-channel keys in wide groups, a second chunk of 32 beside waves that have a SIMD each."""
    assert plans([(1, hq, hkv, n, bits, group, 0, 0, 0, axis, EQUAL_HEADS)])[0]["half"] == half
