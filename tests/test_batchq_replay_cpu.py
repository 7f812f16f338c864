"""Host replay of the default batched selection's work (no GPU): the order of the arrays, their
parts and regions, the search for an item's slot and the predicates of the route it takes
(csrc/batch_queue.h, the kernels' own code), on batches with every kind of bad descriptor (also of
shared sizes, where an array's several items meet it) and with a pool too small for some regions.

What the kernels then do with an item is: its first part writes a bad descriptor's record or
lists an array that is left unread (too large, or shared without a region); one item selects an
array that is not shared; the last part to arrive selects a shared one.  So every array must
be answered exactly once and listed at most once, and every part must come up exactly once."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
BADARG, REDO, SMALL, LARGE, SHARED = range(5)
SHARE = {4: 1 << 18, 8: 1 << 16}
MAX_N = 1 << 31
BASE = 0x7F0000000000


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    exe = tmp_path_factory.mktemp("replay") / "batchq_replay"
    src = os.path.join(HERE, "cpp", "batchq_replay_main.cpp")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-o", str(exe), src], check=True)
    return exe


def run(replay, tmp_path, esize, grid, pool, addrs, sizes, ks):
    f = tmp_path / "batch.txt"
    with open(f, "w") as fh:
        fh.write(f"{esize} {grid} {pool} {len(sizes)}\n")
        fh.writelines(f"{a} {n} {k}\n" for a, n, k in zip(addrs, sizes, ks))
    out = subprocess.run([str(replay), str(f)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, (out.returncode, out.stderr[-2000:])
    lines = [ln.split() for ln in out.stdout.splitlines()]
    head = {lines[0][i]: int(lines[0][i + 1]) for i in (0, 2, 4)}
    slots = [tuple(int(v) for v in ln[2:]) for ln in lines if ln[0] == "slot"]
    items = [tuple(int(v) for v in ln[1:]) for ln in lines if ln[0] == "item"]
    return head, slots, items


def valid(esize, a, n, k):
    return a != 0 and a % esize == 0 and n >= 1 and 1 <= k <= n


def check(esize, pool, addrs, sizes, ks, head, slots, items):
    count = len(sizes)
    shared = [SHARE[esize] <= n <= MAX_N for n in sizes]
    assert sorted(s[0] for s in slots) == list(range(count))
    # the shared arrays first, by their sizes' classes (an eighth of a power of two), what is too
    # large for both last with the smallest
    assert [shared[s[0]] for s in slots] == sorted((shared[s[0]] for s in slots), reverse=True)
    assert head["shared"] == sum(shared)
    big = [sizes[s[0]] for s in slots if shared[s[0]]]
    assert all(b <= a * 1.125 for a, b in zip(big, big[1:]))
    # regions: disjoint, inside the pool, room for a sixteenth and the parts' bins, whole units
    end = 0
    for index, first, parts, region in slots:
        if region < 0:
            continue
        assert shared[index] and region % 64 == 0 and region >= end
        end = region + -(-(sizes[index] // 16) // 64) * 64 + parts * 8192 // esize
        assert end <= pool
    # items: consecutive, each slot's parts in turn
    assert [q for q, *_ in items] == list(range(head["items"]))
    want = [(i, p) for i, s in enumerate(slots) for p in range(s[2])]
    assert [(s, p) for _, s, p, _ in items] == want
    assert head["items_of_shared"] == sum(s[2] for s in slots if shared[s[0]])
    answered, listed = np.zeros(count, int), np.zeros(count, int)
    arrived = np.zeros(count, int)
    for _, s, part, route in items:
        index, first, parts, region = slots[s]
        n = sizes[index]
        assert (route == BADARG) == (not valid(esize, addrs[index], n, ks[index]))
        if route == BADARG:
            answered[index] += part == 0
        elif route == REDO:
            assert n > MAX_N and parts == 1
            listed[index] += 1
        elif route == SHARED:
            assert shared[index]
            if region < 0:
                listed[index] += part == 0
            else:
                arrived[index] += 1
                answered[index] += arrived[index] == parts
        else:
            assert parts == 1 and not shared[index] and n <= MAX_N
            assert (route == SMALL) == (n <= (16384 if esize == 4 else 8192))
            answered[index] += 1
    assert (answered + listed == 1).all()
    return listed


def batch(esize, count, seed, top):
    r = np.random.default_rng([seed, esize])
    sizes = [int(v) for v in 2.0 ** r.uniform(0, top, count)]
    edges = [1, 2, 7, 8, 9, 8192, 8193, 16384, 16385, SHARE[esize] - 1, SHARE[esize],
             SHARE[esize] + 1, MAX_N - 1, MAX_N, MAX_N + 1, (1 << 40) + 3]
    sizes[: len(edges)] = edges
    ks = [int(r.integers(1, n + 1)) for n in sizes]
    addrs = [BASE + 4096 * i for i in range(count)]
    return addrs, sizes, ks


@pytest.mark.parametrize("esize", [4, 8])
@pytest.mark.parametrize("count,top", [(40, 24), (300, 27), (4096, 20)])
@pytest.mark.parametrize("pool", [0, 1 << 16, 5_000_000, 256 * ((1 << 18) + 4096), 1 << 33])
def test_every_array_once(replay, tmp_path, esize, count, top, pool):
    addrs, sizes, ks = batch(esize, count, 1, top)
    head, slots, items = run(replay, tmp_path, esize, 512, pool, addrs, sizes, ks)
    listed = check(esize, pool, addrs, sizes, ks, head, slots, items)
    shared = sum(SHARE[esize] <= n <= MAX_N for n in sizes)
    if pool == 0:
        assert listed.sum() == shared + 2  # (and the two too large)
    elif pool == 1 << 33:
        # every array but those of about 2^30 elements and more has a region
        assert listed.sum() == 2 + sum(n > 1 << 29 and n <= MAX_N for n in sizes)


@pytest.mark.parametrize("count,n", [(1024, 1 << 20), (512, 1 << 21), (256, 1 << 22), (64, 1 << 24)])
def test_float64_batch_that_fills_the_default_pool(replay, tmp_path, count, n):
    """2^30 float64 elements (1024 candidates' squares over 2^20 rows among them): every array of
    equal size has a region of the default pool, 256 workgroups' workspaces."""
    addrs, sizes, ks = [BASE + 4096 * i for i in range(count)], [n] * count, [n // 2] * count
    pool = 256 * ((1 << 18) + 4096)
    head, slots, items = run(replay, tmp_path, 8, 512, pool, addrs, sizes, ks)
    assert check(8, pool, addrs, sizes, ks, head, slots, items).sum() == 0


@pytest.mark.parametrize("esize", [4, 8])
@pytest.mark.parametrize("pool", [0, 3_000_000, 1 << 33])
def test_bad_descriptors(replay, tmp_path, esize, pool):
    addrs, sizes, ks = batch(esize, 120, 2, 26)
    sizes[20:60] = [SHARE[esize] * (i - 15) + i for i in range(20, 60)]
    ks[20:60] = [n // 2 for n in sizes[20:60]]
    bad = []
    for i in range(60, 110, 10):  # of every size the batch holds, and of shared ones
        for at, kind in ((i, "null"), (i + 1, "unaligned"), (i + 2, "k0"), (i + 3, "kbig"), (i + 4, "size0"),
                         (i + 5, "negative"), (i + 6, "lowest")):
            bad.append((at, kind))
    for at, kind in zip(range(20, 55, 5), ("null", "unaligned", "k0", "kbig", "negk", "null", "kbig")):
        bad.append((at, kind))
    bad += [(13, "null"), (14, "kbig"), (15, "unaligned")]  # 2^31, beyond it, and 2^40
    for at, kind in bad:
        if kind == "null":
            addrs[at] = 0
        elif kind == "unaligned":
            addrs[at] += esize // 2
        elif kind == "k0":
            ks[at] = 0
        elif kind == "kbig":
            ks[at] = sizes[at] + 1
        elif kind == "negk":
            ks[at] = -(1 << 62)
        elif kind == "size0":
            sizes[at] = 0
        elif kind == "negative":
            sizes[at] = -5
        else:
            sizes[at] = -(1 << 63)
    head, slots, items = run(replay, tmp_path, esize, 512, pool, addrs, sizes, ks)
    check(esize, pool, addrs, sizes, ks, head, slots, items)
    assert sum(not valid(esize, *d) for d in zip(addrs, sizes, ks)) == len(bad)
    several = {i for i, s in enumerate(slots) if s[2] > 1 and not valid(esize, addrs[s[0]], sizes[s[0]], ks[s[0]])}
    assert several, "no bad descriptor of an array in several parts"
