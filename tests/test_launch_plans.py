"""The host rules that lay a launch out, over the whole range of sizes they are asked for
(compiled from the library's own header, no GPU needed)."""
import os
import subprocess

import pytest

from paper_2306_14048_amd import build as hb

MAIN = r"""
#include <math.h>
#include <stdio.h>
#include "h2o_internal.h"
int main()
{
    int what, a, b, c, d;
    while (scanf("%d %d %d %d %d", &what, &a, &b, &c, &d) == 5) {
        if (what == 0) {
            const SelectPlan p = select_plan(a, b, c, d != 0);
            printf("%d %d %d\n", p.parts, p.part_slots, (int)p.wide);
        } else if (what == 2) {
            printf("%d %d\n", (int)small_blocks(a, b, c, d), (int)head_slots(a));
        } else if (what == 3) {
            printf("%d\n", compact_parts(a, b, c));
        } else {
            printf("%d %d %d\n", (int)two_groups(a, b, c, false, d), (int)groups_apart(a, b, c, d), (int)head_slots(a));
        }
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans(list of (rule, a, b, c, d)) -> the rule's answers, a tuple of ints each"""
    d = tmp_path_factory.mktemp("plans")
    src, exe = str(d / "plans.hip"), str(d / "plans")
    with open(src, "w") as f:
        f.write(MAIN)
    flags = [f for f in hb.FLAGS if f not in ("-fPIC", "-fvisibility=hidden", "-O3")]
    subprocess.run(["hipcc", *flags, "-O1", src, "-o", exe], check=True, capture_output=True)

    def ask(queries):
        text = "\n".join(" ".join(str(int(x)) for x in q) for q in queries)
        env = dict(os.environ, HIP_VISIBLE_DEVICES="")
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, env=env).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return ask


def test_selection_gives_every_workgroup_a_cu(plans):
    """Beyond 4096 candidates a workgroup's time is its selection: never two on one of the 256 CUs while
    heads could be spread otherwise, and then sixteen waves, whatever the head count."""
    q = [(0, h, k, n, 0) for h in [*range(1, 258), 300, 512, 3584] for k in (1, 64, 700, 1000, 3277, 4096)
         for n in (4097, 8193, 16384, 16385, 28672, 28673, 40000, 65536) if n > k]
    for (_, h, k, n, _), (parts, slots, wide) in zip(q, plans(q)):
        assert parts >= 1 and parts * slots >= k and (parts - 1) * slots < k, (h, k, n)
        assert parts == 1 or h * parts <= 256, (h, k, n, parts)
        assert wide == (h <= 256 or n > 16384), (h, k, n)
        if n <= 28672 and h <= 128 and k >= 8192 // h:       # nor are CUs left idle that a head could use
            assert h * (parts + 1) > 256 or parts * slots < k + slots, (h, k, n, parts)


def test_selection_of_few_candidates_and_in_place(plans):
    q = [(0, h, k, n, 0) for h in range(1, 300) for k in (1, 64, 700, 3277) for n in (k + 1, 4096)]
    for (_, h, k, n, _), (parts, slots, wide) in zip(q, plans(q)):
        assert not wide and parts * slots >= k > (parts - 1) * slots, (h, k, n)
        assert parts <= (256 + h - 1) // h and (parts == 1 or slots >= 16), (h, k, n)
    q = [(0, h, k, n, 1) for h in (1, 12, 56, 128, 256, 257, 3584) for k in (64, 4096) for n in (4096, 4097, 16385, 69000)]
    for (_, h, k, n, _), (parts, slots, wide) in zip(q, plans(q)):
        assert (parts, slots) == (1, k) and wide == (n > 4096 and (h <= 256 or n > 16384)), (h, k, n)


def test_columns_of_the_compression_in_place(plans):
    """Workgroups per head: powers of two (columns are found with masks), lines of 128 bytes, K's columns or V's, at
    least 64 KiB of rows each and no more than there are CUs."""
    q = [(3, h, k, rowb, 0) for h in [*range(1, 270), 512, 3584] for rowb in (128, 256, 512)
         for k in (1, 255, 256, 300, 511, 512, 513, 819, 1023, 1024, 1025, 2048, 4095, 4096)]
    seen = set()
    for (_, h, k, rowb, _), (parts,) in zip(q, plans(q)):
        seen.add(parts)
        assert parts & (parts - 1) == 0 and 1 <= parts <= 2 * rowb // 128, (h, k, rowb)
        if parts > 1:
            assert k * rowb >= 131072 and h * parts <= 256 and 2 * k * rowb // parts >= 65536, (h, k, rowb)
        elif k * rowb >= 131072:
            assert h > 128, (h, k, rowb)
    assert seen == {1, 2, 4, 8}


def test_attention_groups_apart_have_a_cu_of_their_own(plans):
    """At d = 64 the groups one phase apart leave no room for a second workgroup on their CU: few more
    block slots than two rounds of the CUs, and one round where blocks are equally heavy.  (All blocks of
    a head run on one XCD: a single long prompt has eight times its blocks in slots.)"""
    q = [(1, h, nq, nq + old, d) for d in (64, 128) for h in [*range(1, 66), 96, 128, 192, 256, 320, 400, 512]
         for nq in (1, 100, 128, 256, 500, 800, 1024, 1100, 1200, 1531, 1650, 2048, 2300, 3000, 5000, 8200, 16000, 65536)
         for old in (0, 410, 2000, 4000)]
    some = {64: 0, 128: 0}
    for (_, h, nq, nk, d), (few, apart, heads8) in zip(q, plans(q)):
        slots = heads8 * ((nq + 127) // 128)
        if not few or not apart:
            continue
        some[d] += 1
        if d == 64:
            assert slots <= (512 if nk < 4000 else 576), (h, nq, nk)
            assert slots <= 256 or 2 * nk < 3 * nq, (h, nq, nk)
        else:
            assert slots <= 256 or nk >= 1100, (h, nq, nk, d)
    assert min(some.values()) > 300
    want = {(1, 16000, 64): 0, (1, 65536, 64): 0, (20, 3000, 64): 0, (36, 1650, 64): 0, (8, 8000, 64): 1, (32, 1531, 64): 1,
            (1, 65536, 128): 1, (32, 1531, 128): 1, (36, 800, 128): 0, (320, 100, 64): 0, (8, 500, 64): 1}
    got = plans([(1, h, n, n, d) for h, n, d in want])
    assert [g[1] for g in got] == list(want.values())


def test_binary32_blocks_of_64_rows(plans):
    """At d = 128 a workgroup of 64 rows has a CU to itself: not where its second group has no rows, nor where
    twice the blocks take more rounds of the 256 CUs, nor as many with all of them equally heavy."""
    q = [(2, h, rows, st, d) for d in (64, 128) for h in [*range(1, 330, 3), 400, 512, 576, 640, 641, 1024]
         for rows in (1, 16, 32, 33, 64, 65, 96, 97, 128, 129, 192, 200, 256, 300, 512, 700, 1024, 2500, 4096)
         for st in {1, 16, 32, 33, 150, 400, rows, rows + 100, rows + 400, rows + 4000, max(1, rows - 100), max(1, rows - 400)}]
    some = 0
    for (_, h, rows, st, d), (small, heads8) in zip(q, plans(q)):
        slots, slots128 = heads8 * ((rows + 63) // 64), heads8 * ((rows + 127) // 128)
        if d == 64:
            assert small == (slots <= 512), (h, rows, st)
            continue
        some += small
        if small:
            assert st > 32 and slots <= 640 and -(-slots // 256) <= 2 * -(-slots128 // 256), (h, rows, st)
            assert rows <= 64 or rows > 128 or slots <= 256 or (rows > 96 and h > 256), (h, rows, st)
        elif slots <= 256:
            assert st <= 32, (h, rows, st)
    assert some > 500
    # (heads, rows, streamed) on either side: whole prompts, then statistics and column sums of chunks
    want = {(8, 32, 32): 0, (512, 17, 17): 0, (8, 33, 33): 1, (640, 64, 64): 1, (641, 64, 64): 0, (128, 128, 128): 1,
            (129, 65, 65): 0, (256, 100, 100): 0, (264, 96, 96): 0, (264, 97, 97): 1, (320, 128, 128): 1, (128, 129, 129): 1,
            (192, 192, 192): 1, (200, 129, 129): 0, (128, 256, 256): 1, (128, 300, 300): 1, (32, 1000, 1000): 1, (32, 1300, 1300): 0,
            (32, 700, 1700): 1, (128, 192, 292): 1, (128, 150, 550): 0, (48, 512, 912): 1, (64, 512, 1512): 0, (256, 100, 500): 0,
            (64, 292, 192): 1, (128, 250, 150): 0, (32, 550, 300): 1, (32, 550, 150): 0, (40, 400, 150): 1, (64, 433, 33): 0}
    got = plans([(2, h, rows, st, 128) for h, rows, st in want])
    assert [g[0] for g in got] == list(want.values())
