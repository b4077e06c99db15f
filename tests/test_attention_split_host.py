"""The device code that describes a batch's attention work items and cuts their key ranges into parts (laps_dev_attn_desc), run on
the CPU with the launches that laps_attn_plan_info gives for random batches: every query-row block has its entry, the parts cover
its key tiles once and in order, none is empty, they stay inside the launch's grid and inside the partial results, and where a
block is cut follows from its own length and the launch alone, whatever it is batched with."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2601_11589_amd import api

KT, PAGE = 64, 16


@pytest.fixture(scope="module")
def driver(tmp_path_factory, repo_root):
    exe = str(tmp_path_factory.mktemp("split") / "attn_split")
    build = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            os.path.join(repo_root, "tests", "attn_split_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr

    def run(batches):
        lines = [" ".join(map(str, [b["split"], b["min"], b["group"], b["pages"], b["rows"], b["max_items"], len(b["new"])]
                              + b["new"] + b["pre"])) for b in batches]
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out = []
        for b, line in zip(batches, r.stdout.splitlines(), strict=True):
            v = list(map(int, line.split()))
            out.append([tuple(v[i:i + 4]) for i in range(0, len(v), 4)])
        return out

    return run


def check(b, desc):
    """Returns the number of parts and of blocks."""
    n = b["max_items"]
    assert len(desc) == 2 * n + 2 and desc[-2:] == [(-7,) * 4] * 2      # nothing behind the table
    item = total = 0
    for s, (new, pre) in enumerate(zip(b["new"], b["pre"])):
        h = max(0, min(pre, b["pages"] * PAGE - new))
        for r0 in range(0, new * b["group"], b["rows"]):
            who, (row, parts, each, _) = desc[2 * item], desc[2 * item + 1]
            assert who == (s, r0 // b["rows"], new, h) and row == sum(b["new"][:s])
            item, total = item + 1, total + parts
            if b["split"] == 1:
                assert parts == 1
                continue
            keys = h + (min(r0 + b["rows"], new * b["group"]) - 1) // b["group"] + 1
            tiles = -(-keys // KT)
            assert each == -(-tiles // max(1, min(tiles // b["min"], b["split"])))        # from the block's own length
            assert 1 <= parts <= b["split"] and (parts - 1) * each < tiles <= parts * each
            assert parts == 1 or each >= b["min"]
    assert item <= n and all(desc[2 * k][0] == -1 for k in range(item, n))
    return total, item


def batch(new, pre, heads, pages=None):
    n_q, n_kv, hd = heads
    pages = pages or max(1, max((n + p + PAGE - 1) // PAGE for n, p in zip(new, pre)))
    out = (C.c_int64 * 6)()
    assert api.lib().laps_attn_plan_info(*[C.c_int32(v) for v in (len(new), sum(new), n_q, n_kv, hd, pages)], out) == 0
    rows, max_items, split, least, table_bytes, partial_bytes = out
    if split > 1:      # every part has its place among the partial results
        assert rows == 128 and least in (1, 4) and max_items * split * n_kv * rows * (hd + 2) * 4 <= partial_bytes
    return dict(new=list(new), pre=list(pre), group=n_q // n_kv, pages=pages, rows=rows, max_items=max_items, split=split, min=least)


HEADS = [(40, 8, 128), (28, 4, 128), (4, 2, 64), (8, 1, 64), (1, 1, 128)]


def test_parts_cover_random_batches_once(driver):
    rng = random.Random(3)
    batches = []
    while len(batches) < 1200:
        n = rng.randint(1, rng.choice([1, 3, 20, 60, 300]))
        new = [rng.choice([0, 1, rng.randint(1, 64), rng.randint(1, 300)]) for _ in range(n)]
        pre = [rng.choice([0, rng.randint(0, 4096), rng.randint(0, 20000)]) for _ in range(n)]
        wide = max(1, max((a + p + PAGE - 1) // PAGE for a, p in zip(new, pre)))
        if sum(new):      # as wide as the batch needs, wider, or prefixes that the table cannot hold
            batches.append(batch(new, pre, rng.choice(HEADS), rng.choice([wide, wide, wide + 7, max(29, wide // 2)])))
    seen = [(b["split"], *check(b, t)) for b, t in zip(batches, driver(batches))]
    assert sum(p > i for _, p, i in seen) > 500 and sum(p == i and s > 1 for s, p, i in seen) > 20
    assert sum(s == 1 for s, _, _ in seen) > 200 and max(i for _, _, i in seen) > 256
    assert {b["min"] for b in batches if b["split"] > 1} == {1, 4}


@pytest.mark.parametrize("new,pre,pages", [([1], [0], 29), ([1], [1 << 20], 29), ([1] * 254, [4000] * 254, 251), ([0, 0, 5], [9, 9, 63], 29),
                                           ([255], [4096 * 16], 5000)])
def test_parts_at_the_edges(driver, new, pre, pages):
    b = batch(new, pre, (1, 1, 128), pages)
    assert b["split"] > 1
    check(b, driver([b])[0])


def test_a_request_is_cut_alike_whatever_it_is_batched_with(driver):
    """In a captured shape of four turns the launch is the same for any lengths."""
    rng = random.Random(5)
    for heads in HEADS[:2]:
        shape = batch([32] * 4, [4096] * 4, heads)
        same = [dict(shape, new=[20] + [rng.randint(1, 32) for _ in range(3)], pre=[2000] + [rng.choice([0, 500, 4096]) for _ in range(3)])
                for _ in range(20)]
        cuts = {tuple(desc[1][1:3]) for desc in driver(same)}
        assert len(cuts) == 1 and next(iter(cuts))[0] > 1
