"""The device code that cuts a batch's attention into parts of its key ranges (laps_dev_attn_split), run on the CPU over random
batches: the parts of every query-row block cover its key tiles once and in order, none is empty, they never pass the table's
end, and no part is longer than the equal length the batch allows."""
import os
import random
import subprocess

import pytest

KT, PAGE, WGS = 64, 16, 512


@pytest.fixture(scope="module")
def driver(tmp_path_factory, repo_root):
    exe = str(tmp_path_factory.mktemp("split") / "attn_split")
    build = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            os.path.join(repo_root, "tests", "attn_split_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr

    def run(batches):
        lines = [" ".join(map(str, [b["split"], b["min"], b["kv"], b["group"], b["pages"], b["rows"], b["max_items"], len(b["new"])]
                              + b["new"] + b["pre"])) for b in batches]
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [list(map(int, line.split())) for line in r.stdout.splitlines()]

    return run


def check(b, v):
    """Returns the number of parts and of blocks."""
    entry = [tuple(v[i:i + 4]) for i in range(0, len(v), 4)]
    n, cap = b["max_items"], b["max_items"] * b["split"]
    desc, parts = entry[:2 * n + 2], entry[2 * n + 2:]
    assert len(parts) == 2 * cap + 2 and desc[-2:] == parts[-2:] == [(-7,) * 4] * 2      # nothing behind either table
    item, live, longest, total = 0, set(), 0, 0
    for s, (new, pre) in enumerate(zip(b["new"], b["pre"])):
        h = max(0, min(pre, b["pages"] * PAGE - new))
        for r0 in range(0, new * b["group"], b["rows"]):
            keys = h + (min(r0 + b["rows"], new * b["group"]) - 1) // b["group"] + 1
            tiles = -(-keys // KT)
            who, (row, first, used, _) = desc[2 * item], desc[2 * item + 1]
            assert who == (s, r0 // b["rows"], new, h) and row == sum(b["new"][:s]) and used >= 1
            each = parts[2 * first + 1][2]
            for z in range(used):
                assert parts[2 * (first + z)] == who and parts[2 * (first + z) + 1] == (row, z, each, used)
                assert first + z not in live
                live.add(first + z)
            assert (used - 1) * each < tiles <= used * each
            longest, total, item = max(longest, each), total + tiles, item + 1
    assert all(desc[2 * k][0] == -1 for k in range(item, n))
    assert all((parts[2 * k][0] >= 0) == (k in live) for k in range(cap))
    # equal lengths: what fills the chip, or the shortest worth a workgroup, where the table has the places
    fill = max(-(-total // max(1, WGS // b["kv"])), b["min"])
    assert longest <= fill or -(-total // fill) + item > cap
    return len(live), item


def batch(new, pre, heads, rows, split, least=4, spare=0):
    group, kv = heads
    pages = max(1, max((n + p + PAGE - 1) // PAGE for n, p in zip(new, pre))) + spare
    return dict(new=list(new), pre=list(pre), group=group, kv=kv, rows=rows, split=split, min=least, pages=pages,
                max_items=sum(new) * group // rows + len(new))


def test_parts_cover_random_batches_once(driver):
    rng = random.Random(3)
    batches = []
    while len(batches) < 1000:
        n = rng.randint(1, rng.choice([1, 3, 20, 60]))
        new = [rng.choice([0, 1, rng.randint(1, 64), rng.randint(1, 300)]) for _ in range(n)]
        pre = [rng.choice([0, rng.randint(0, 4096), rng.randint(0, 20000)]) for _ in range(n)]
        b = batch(new, pre, rng.choice([(5, 8), (7, 4), (2, 2), (1, 8)]), rng.choice([64, 128, 256]), rng.randint(2, 32),
                  rng.choice([1, 4]), rng.choice([0, 7]))
        if sum(new) and b["max_items"] < 256:
            batches.append(b)
    batches[0]["pages"] = 1                 # prefixes that the table cannot hold
    seen = [check(b, v) for b, v in zip(batches, driver(batches))]
    assert sum(p > i for p, i in seen) > 500 and sum(p == i for p, i in seen) > 20


@pytest.mark.parametrize("new,pre,split", [([1], [0], 2), ([1], [1 << 20], 2), ([1] * 255, [4000] * 255, 2), ([0, 0, 5], [9, 9, 63], 8)])
def test_parts_at_the_edges(driver, new, pre, split):
    b = batch(new, pre, (1, 8), 64, split)
    b["max_items"] = min(b["max_items"], 255)
    check(b, driver([b])[0])
