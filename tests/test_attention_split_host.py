"""The device code that cuts a batch's attention into parts of its key ranges (laps_dev_attn_split), run on the CPU with the
launches that laps_attn_plan_info gives for random batches: the parts of every query-row block cover its key tiles once and in
order, none is empty, they stay inside the table and inside the partial results, and where a block is cut follows from its own
length and the launch alone, whatever it is batched with."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2601_11589_amd import api

KT, PAGE, ROWS = 64, 16, 128


@pytest.fixture(scope="module")
def driver(tmp_path_factory, repo_root):
    exe = str(tmp_path_factory.mktemp("split") / "attn_split")
    build = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            os.path.join(repo_root, "tests", "attn_split_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr

    def run(batches):
        lines = [" ".join(map(str, [b["split"], b["min"], b["group"], b["pages"], ROWS, b["max_items"], len(b["new"])]
                              + b["new"] + b["pre"])) for b in batches]
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [tables(b, list(map(int, line.split()))) for b, line in zip(batches, r.stdout.splitlines(), strict=True)]

    return run


def tables(b, v):
    entry = [tuple(v[i:i + 4]) for i in range(0, len(v), 4)]
    desc, parts = entry[:2 * b["max_items"] + 2], entry[2 * b["max_items"] + 2:]
    assert len(parts) == 2 * b["max_items"] * b["split"] + 2
    return desc, parts


def check(b, desc, parts):
    """Returns the number of parts and of blocks."""
    n, cap = b["max_items"], b["max_items"] * b["split"]
    assert desc[-2:] == parts[-2:] == [(-7,) * 4] * 2      # nothing behind either table
    item, live = 0, set()
    for s, (new, pre) in enumerate(zip(b["new"], b["pre"])):
        h = max(0, min(pre, b["pages"] * PAGE - new))
        for r0 in range(0, new * b["group"], ROWS):
            keys = h + (min(r0 + ROWS, new * b["group"]) - 1) // b["group"] + 1
            tiles = -(-keys // KT)
            who, (row, first, used, _) = desc[2 * item], desc[2 * item + 1]
            assert who == (s, r0 // ROWS, new, h) and row == sum(b["new"][:s])
            each = -(-tiles // max(1, min(tiles // b["min"], b["split"])))        # from the block's own length
            assert used == -(-tiles // each) and (used - 1) * each < tiles <= used * each
            assert used == 1 or each >= b["min"]
            for z in range(used):
                assert parts[2 * (first + z)] == who and parts[2 * (first + z) + 1] == (row, z, each, used)
                assert first + z not in live and first + z < cap
                live.add(first + z)
            item += 1
    assert all(desc[2 * k][0] == -1 for k in range(item, n))
    assert all((parts[2 * k][0] >= 0) == (k in live) for k in range(cap))
    return len(live), item


def plan(new, pages, n_q, n_kv, hd):
    out = (C.c_int64 * 6)()
    assert api.lib().laps_attn_plan_info(*[C.c_int32(v) for v in (len(new), sum(new), n_q, n_kv, hd, pages)], out) == 0
    return dict(zip(("rows", "max_items", "split", "min", "table_bytes", "partial_bytes"), out))


def batch(new, pre, heads, pages=None):
    """None where the launch is not split."""
    n_q, n_kv, hd = heads
    pages = pages or max(1, max((n + p + PAGE - 1) // PAGE for n, p in zip(new, pre)))
    p = plan(new, pages, *heads)
    if p["split"] == 1:
        return None
    # a thread an item deals out the parts, and each has its place among the partial results
    assert p["rows"] == ROWS and p["max_items"] < 256 and p["min"] in (1, 4)
    assert p["max_items"] * p["split"] * n_kv * ROWS * (hd + 2) * 4 <= p["partial_bytes"]
    return dict(new=list(new), pre=list(pre), group=n_q // n_kv, pages=pages, max_items=p["max_items"], split=p["split"], min=p["min"])


HEADS = [(40, 8, 128), (28, 4, 128), (4, 2, 64), (8, 1, 64), (1, 1, 128)]


def test_parts_cover_random_batches_once(driver):
    rng = random.Random(3)
    batches = []
    while len(batches) < 1000:
        n = rng.randint(1, rng.choice([1, 3, 20, 60]))
        new = [rng.choice([0, 1, rng.randint(1, 64), rng.randint(1, 300)]) for _ in range(n)]
        pre = [rng.choice([0, rng.randint(0, 4096), rng.randint(0, 20000)]) for _ in range(n)]
        wide = max(1, max((a + p + PAGE - 1) // PAGE for a, p in zip(new, pre)))
        # as wide as the batch needs, wider, or prefixes that the table cannot hold
        b = batch(new, pre, rng.choice(HEADS), rng.choice([wide, wide, wide + 7, max(29, wide // 2)])) if sum(new) else None
        if b:
            batches.append(b)
    seen = [check(b, *t) for b, t in zip(batches, driver(batches))]
    assert sum(p > i for p, i in seen) > 500 and sum(p == i for p, i in seen) > 20
    assert {b["min"] for b in batches} == {1, 4} and max(b["max_items"] for b in batches) > 200


@pytest.mark.parametrize("new,pre,pages", [([1], [0], 29), ([1], [1 << 20], 29), ([1] * 254, [4000] * 254, 251), ([0, 0, 5], [9, 9, 63], 29),
                                           ([255], [4096 * 16], 5000)])
def test_parts_at_the_edges(driver, new, pre, pages):
    b = batch(new, pre, (1, 1, 128), pages)
    check(b, *driver([b])[0])


def test_a_request_is_cut_alike_whatever_it_is_batched_with(driver):
    """In a captured shape of four turns the launch is the same for any lengths."""
    rng = random.Random(5)
    for heads in HEADS[:2]:
        shape = batch([32] * 4, [4096] * 4, heads)
        same = [dict(shape, new=[20] + [rng.randint(1, 32) for _ in range(3)], pre=[2000] + [rng.choice([0, 500, 4096]) for _ in range(3)])
                for _ in range(20)]
        cuts = set()
        for desc, parts in driver(same):
            _, first, used, _ = desc[1]
            cuts.add(tuple(parts[2 * (first + z) + 1][1:] for z in range(used)))
        assert len(cuts) == 1 and len(next(iter(cuts))) > 1
