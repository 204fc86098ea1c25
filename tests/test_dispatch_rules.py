"""The rules by which an entry point chooses among its kernels: calls that were measured to lose by a form do not take it, and every kernel
that is compiled for the reduce is one that some call takes.  The rules are read from the library's own headers by tests/dispatch_rules_check.cpp; the
kernels that there are, from the built library's symbols.  No GPU."""
import os
import re
import subprocess

import pytest

from paper_2107_14575_amd import build as dq_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(dq_build.LIB_PATH):
        pytest.skip("needs the built library")
    exe = str(tmp_path_factory.mktemp("rules") / "dispatch_rules_check")
    flags = [f for f in dq_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-O3", "-Wall")]
    where = os.path.dirname(dq_build.LIB_PATH)
    cmd = [HIPCC, *flags, "-O1", "-x", "hip", os.path.join(ROOT, "tests", "dispatch_rules_check.cpp"), "-I", os.path.join(ROOT, "include"), "-I", dq_build.CSRC,
           "-L", where, "-ldq", f"-Wl,-rpath,{where}", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    found = {}
    for line in out.stdout.splitlines():
        kind, *values = line.split()
        found.setdefault(kind, []).append(tuple(int(v) for v in values))
    return found


@pytest.fixture(scope="module")
def form(rules):
    """(tiles, workers, width, update) -> (workers to a word, level loads streamed, model passes through)"""
    return {row[:4]: row[4:] for row in rules["reduce"]}


# tiles, workers, width (0: a table), update: calls in which the other form took 1.03 to 1.3 of the time
ONE_WORKER = [(800, 8, 1, 0), (600, 4, 3, 1), (600, 2, 4, 1), (800, 2, 1, 1), (512, 16, 4, 0), (680, 16, 2, 1), (1000, 10, 1, 0), (1366, 4, 1, 1),
              (800, 1, 6, 1), (8192, 1, 3, 0), (32768, 16, 3, 0), (32768, 16, 8, 0), (6000, 3, 7, 0), (4096, 32, 4, 0), (6000, 64, 2, 0), (8192, 64, 5, 1), (6000, 32, 1, 1),
              (8192, 24, 1, 1), (600, 4, 0, 1), (800, 2, 0, 0), (470, 4, 0, 1), (680, 13, 0, 0), (680, 13, 0, 1), (720, 24, 7, 0), (650, 4, 7, 1), (800, 5, 7, 1), (800, 4, 6, 0), (6000, 64, 0, 1), (6000, 2, 0, 0)]
TWO_WORKERS = [(513, 64, 5, 1), (1366, 8, 6, 1), (1532, 16, 8, 1), (300, 20, 2, 1), (384, 20, 5, 0), (32768, 16, 4, 0), (8192, 16, 7, 0), (32768, 16, 0, 0), (3072, 47, 7, 1), (1000, 24, 0, 1), (6000, 8, 4, 1), (16384, 4, 5, 1),
               (800, 47, 0, 1), (1532, 16, 0, 1), (4096, 8, 0, 1), (300, 47, 0, 1)]


def test_reduces_take_the_form_that_was_measured_to_be_faster(form):
    assert {c for c in ONE_WORKER if form[c][0] != 1} == set()
    assert {c for c in TWO_WORKERS if form[c][0] != 2} == set()


def test_where_level_loads_are_streamed(form):
    """Widths 5 to 7 (and tables): with update the hint where messages and model together exceed 100 MB or, with W = 1 and up to 32 workers, 128 MB; without,
    with W = 2 only, where messages alone exceed 640 MB."""
    for (tiles, workers, width, update), (two, streamed, once) in form.items():
        messages = tiles * 1024 * workers * ((width or 6) + 1)
        if update:
            want = (two == 2 or workers <= 32) and messages + tiles * 32768 > (100 if two == 2 else 128) << 20
        else:
            want = two == 2 and messages > 640 << 20
        assert bool(streamed) == ((width or 6) in (5, 6, 7) and want)
        assert bool(once) == (bool(update) and tiles * 8192 > 24 << 20)


def test_every_reduce_kernel_is_one_that_a_call_takes(form, rules):
    names = subprocess.run(["nm", "-C", dq_build.LIB_PATH], capture_output=True, text=True, check=True).stdout
    one = {tuple(v) for v in re.findall(r"::k_unpack_dequant_reduce<(\d), (\w+), (\w+), (\w+), (\d)>", names)}
    table = {tuple(v) for v in re.findall(r"::k_unpack_dequant_reduce_v<(\w+), (\w+), (\w+), (\d)>", names)}
    each = {tuple(v) for v in re.findall(r"::k_unpack_dequant_reduce_w<(\w+), (\w+), (\w+)>", names)}
    said = {False: "false", True: "true"}
    want_one, want_table, want_each = set(), set(), set()
    for (_, _, width, update), (two, streamed, once) in form.items():
        flags = said[bool(update)], said[bool(streamed)], said[bool(once)]
        if width:
            want_one.add((str(width), *flags, str(two)))
        else:
            want_table.add((*flags, str(two)))
    for _, _, _, update, two, streamed, once in rules["rows"]:
        assert two == 1
        want_each.add((said[bool(update)], said[bool(streamed)], said[bool(once)]))
    assert one == want_one and len(one) > 40
    assert table == want_table
    assert each == want_each


def test_norms_of_small_tensors_are_no_stream(rules):
    """Fewer resident workgroups for many that are nearly full only: at 384 to 3000 values an item they took 1.04 to 1.4 of the time."""
    assert {row[:3]: bool(row[3]) for row in rules["norm"]} == {
        (n, padded, n): n >= 8192 and padded >= 3584 * n for n, padded, _, _ in rules["norm"]}
    assert any(row[3] for row in rules["norm"])


def test_sign_messages_of_small_tensors_take_four_tiles(rules):
    """Chunk by chunk only where at least half of the chunks are of one tensor: at none, 18 and 32 % of them it took 1.05 to 1.15, 1.0 to 1.05 and 1.0 to 1.04."""
    assert {row[0]: bool(row[2]) for row in rules["whole"]} == {0: False, 18: False, 32: False, 49: False, 50: True, 51: True, 100: True}
