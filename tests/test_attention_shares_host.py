"""The device code that shares out a batch's attention (laps_dev_attn_sched, laps_dev_attn_bounds), run on the CPU over
random batches: the shares, walked as the attention kernel walks them, cover every key tile of every (kv head, query-row
block) once; a cut lies where every row of its block sees a key and no partial result is written twice; and the parts
that the merge kernel would add up are exactly the parts of each cut block, in key order."""
import os
import random
import subprocess

import pytest

KT, ROWS, PAGE = 64, 256, 16


@pytest.fixture(scope="module")
def driver(tmp_path_factory, repo_root):
    exe = str(tmp_path_factory.mktemp("shares") / "attn_shares")
    build = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            os.path.join(repo_root, "tests", "attn_shares_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr

    def run(batches):
        lines = []
        for b in batches:
            head = [b["wgs"], b["kv"], b["group"], b["pages"], ROWS, b["max_items"], len(b["new"])]
            lines.append(" ".join(map(str, head + b["new"] + b["pre"])))
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out = []
        for b, line in zip(batches, r.stdout.splitlines(), strict=True):
            v, n = list(map(int, line.split())), len(b["new"])
            flat = v[n + 1 + b["max_items"]:]
            out.append((v[:n + 1], v[n + 1:n + 1 + b["max_items"]], [tuple(flat[i:i + 3]) for i in range(0, len(flat), 3)]))
        return out

    return run


def blocks_of(b):
    """(visible keys, first key that every row sees last) of every query-row block, sequence by sequence."""
    out = []
    for new, pre in zip(b["new"], b["pre"]):
        h = max(0, min(pre, b["pages"] * PAGE - new))
        for r0 in range(0, new * b["group"], ROWS):
            last = min(r0 + ROWS, new * b["group"]) - 1
            out.append((h + last // b["group"] + 1, h + r0 // b["group"]))
    return out


def check(b, tile_start, item_seq, bounds):
    """Walks the shares; returns the number of cut blocks and of workgroups with work."""
    blocks, kv = blocks_of(b), b["kv"]
    counts = [-(-n * b["group"] // ROWS) for n in b["new"]]
    assert tile_start == [sum(counts[:i]) for i in range(len(counts) + 1)]
    assert item_seq[:len(blocks)] == [s for s, c in enumerate(counts) for _ in range(c)]
    assert all(x <= y for x, y in zip(bounds, bounds[1:])) and bounds[0] == ((0, 0, 0) if blocks else (kv, 0, 0)) and bounds[-1] == (kv, 0, 0)
    parts, slots, busy = {}, set(), 0
    for w in range(b["wgs"]):
        (head, item, t), end, slot, any_work = bounds[w], bounds[w + 1], 2 * w, False
        while head < kv and (head != end[0] or item != end[1] or t < end[2]):
            last = (head, item) == end[:2]
            keys, sees = blocks[item]
            begin, stop = t * KT, min(end[2] * KT if last else keys, keys)
            assert begin < stop and begin <= sees
            whole = begin == 0 and stop == keys
            parts.setdefault((head, item), []).append((begin, stop, None if whole else slot))
            assert whole or slot not in slots
            slots.add(None if whole else slot)
            any_work = True
            if last:
                break
            t, slot, item = 0, 2 * w + 1, item + 1
            if item >= len(blocks):
                item, head = 0, head + 1
        busy += any_work
    assert sorted(parts) == [(h, i) for h in range(kv) for i in range(len(blocks))]
    merged = {}
    for w in range(1, b["wgs"]):          # the merge kernel's workgroups
        here, before = bounds[w], bounds[w - 1]
        if here[2] == 0 or here[0] >= kv or (before[:2] == here[:2] and before[2] > 0):
            continue
        add = [2 * (w - 1) + (0 if before[:2] == here[:2] else 1)]
        for v in range(w, b["wgs"]):
            if bounds[v][:2] != here[:2]:
                break
            if bounds[v + 1] != bounds[v]:
                add.append(2 * v)
        assert here[:2] not in merged
        merged[here[:2]] = add
    for key, p in parts.items():
        p.sort()
        assert p[0][0] == 0 and p[-1][1] == blocks[key[1]][0] and all(x[1] == y[0] for x, y in zip(p, p[1:]))
        assert (len(p) == 1 and p[0][2] is None and key not in merged) or merged[key] == [x[2] for x in p]
    return len(merged), busy


def batch(new, pre, heads, wgs, spare_pages=0):
    group, kv = heads
    pages = max(1, max((n + p + PAGE - 1) // PAGE for n, p in zip(new, pre))) + spare_pages
    return dict(new=list(new), pre=list(pre), group=group, kv=kv, wgs=wgs, pages=pages, max_items=sum(new) * group // ROWS + len(new))


def test_shares_cover_random_batches_once(driver):
    rng = random.Random(1)
    batches = []
    while len(batches) < 1200:
        n = rng.randint(1, rng.choice([1, 3, 20, 70, 300]))
        new = [rng.choice([rng.randint(0, 64), rng.randint(0, 300), rng.randint(1, 2100) if n < 40 else 1]) for _ in range(n)]
        pre = [rng.choice([0, rng.randint(0, 4096), rng.randint(0, 8200)]) for _ in range(n)]
        if sum(new):
            batches.append(batch(new, pre, rng.choice([(5, 8), (7, 4), (2, 2), (1, 8)]), rng.choice([64, 128, 192, 256]), rng.choice([0, 7])))
    batches[0]["pages"] = 1                 # prefixes that the table cannot hold
    seen = [check(b, *got) for b, got in zip(batches, driver(batches))]
    assert sum(c > 0 for c, _ in seen) > 300 and sum(c == 0 for c, _ in seen) > 100


@pytest.mark.parametrize("new,pre,heads,cut", [
    ([1000], [0], (5, 8), False), ([1500], [600], (5, 8), False), ([500] * 2, [600, 700], (5, 8), False),
    ([40] * 16, [0] * 16, (5, 8), False), ([1000], [6000], (5, 8), True), ([1847], [6144], (5, 8), True), ([2048], [0], (5, 8), True),
    ([40] * 12, [4000] + [0] * 11, (5, 8), True)])
def test_blocks_are_cut_only_where_the_longest_one_would_decide(driver, new, pre, heads, cut):
    b = batch(new, pre, heads, 256)
    merged, busy = check(b, *driver([b])[0])
    units = len(blocks_of(b)) * heads[1]
    assert (merged > 0) == cut and (cut or busy == units)


def test_few_shares_are_spread_over_the_compute_units(driver):
    """Workgroup w of 256 runs on XCD w / 32: a batch with work for a quarter of them keeps all eight busy."""
    for b in (batch([40] * 8, [0] * 8, (5, 8), 256), batch([140] * 70 + [600], [0] * 70 + [50], (2, 2), 256)):
        _, _, bounds = driver([b])[0]
        per_xcd = [sum(bounds[w] != bounds[w + 1] for w in range(32 * x, 32 * x + 32)) for x in range(8)]
        assert max(per_xcd) - min(per_xcd) <= 2, per_xcd
