"""Which sequences' block tables a narrow item looks at (WorkItem::peers, under AddressSanitizer and
UndefinedBehaviorSanitizer): only entries that the header says are read, that is below ceil(len / 16) of a sequence that
attends in the call, and among decodes all of the sixteen before and the fifteen behind it that have the column.  And which items look at none:
those whose K/V other items of the launch read, and all of a launch whose decodes' K/V and chunks are small."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_17357_amd", "csrc")


@pytest.fixture(scope="module")
def plan_of(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("policy") / "policy_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "policy_check_main.cpp"), os.path.join(CSRC, "plan.cpp"),
                    "-o", exe], check=True)
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)  # the sanitizer runtime must come first in the library list

    def run(hq, hkv, d, cus, seqs, fp8=0):
        text = " ".join(map(str, [hq, hkv, d, fp8, cus, len(seqs)] + [x for s in seqs for x in s]))
        r = subprocess.run([exe], input=text + "\n", capture_output=True, text=True, env=env)
        assert r.returncode == 0, r.stderr[-3000:]
        lines = r.stdout.splitlines()
        items = np.array([ln.split() for ln in lines[1:]], dtype=np.int64).reshape(-1, 7)
        n_items, run.rows_past = map(int, lines[0].split())
        assert n_items == items.shape[0]
        return items
    return run


OFFSETS = list(range(-16, 0)) + list(range(1, 16))


def look(items, seqs):
    """(seq, column, sequences looked at) of every item that looks."""
    for seq, _, _, _, begin, end, peers in items.tolist():
        if peers >= 0:
            yield seq, (begin + (end - begin) // 4 * 3) // 16, {seq + OFFSETS[b] for b in range(31) if peers >> b & 1}


def test_only_entries_in_use_are_looked_at(plan_of):
    rng = np.random.default_rng(8)
    looked = 0
    for i in range(60):
        n = int(rng.integers(1, 60))
        hq, hkv, d = [(8, 2, 64), (32, 8, 128), (28, 4, 128), (64, 8, 128), (8, 8, 64)][i % 5]
        P = rng.integers(0, int(rng.choice([50, 3000, 20000])), n)
        C = np.where(rng.random(n) < 0.7, 1, rng.integers(0, int(rng.choice([3, 30, 700])), n))
        seqs = list(zip(P.tolist(), C.tolist()))
        for seq, col, others in look(plan_of(hq, hkv, d, int(rng.choice([1, 64, 256])), seqs), seqs):
            for o in others:
                assert 0 <= o < n and seqs[o][1] > 0 and 16 * col < sum(seqs[o]), (i, seq, col, o)
            looked += len(others)
    assert looked > 1000


@pytest.mark.parametrize("n, keys", [(1, 90000), (3, 40000), (20, 3000), (64, 4000), (257, 8000)])
def test_decodes_look_at_every_neighbour_that_has_the_column(plan_of, n, keys):
    rng = np.random.default_rng(n)
    seqs = [(int(p), 1) for p in rng.integers(keys // 100, keys, n)]
    items = plan_of(32, 8, 128, 256, seqs)
    assert len({tuple(x) for x in items[:, [0, 1, 4]].tolist()}) == len(items)
    for seq, col, others in look(items, seqs):
        assert others == {o for o in range(max(0, seq - 16), min(n, seq + 16)) if o != seq and 16 * col < sum(seqs[o])}
    assert (items[:, 6] >= 0).all()


def test_head_groups_that_share_a_kv_head_do_not_look(plan_of):
    assert (plan_of(64, 1, 128, 256, [(90000, 1)] * 5)[:, 6] < 0).all()


def test_the_tail_of_a_chunk_does_not_look(plan_of):
    """Its keys are those of the chunk's tiles; a short chunk that is one item does look."""
    for heads, seqs in (((32, 8, 128), [(6000, 516), (25000, 1), (50, 7)]), ((28, 4, 128), [(0, 36 * 5 + 3)] * 4 + [(50000, 1)]), ((8, 2, 64), [(300, 65), (180000, 1)])):
        items = plan_of(*heads, 256, seqs)
        tails = items[:, 3] < np.array([seqs[s][1] for s in items[:, 0]])
        assert tails.any() and (items[tails, 6] < 0).all() and (items[~tails, 6] >= 0).all()


@pytest.mark.parametrize("fp8, heads, below", [(0, (32, 8, 128), 21972), (0, (8, 2, 64), 175781), (0, (28, 4, 128), 43945), (1, (64, 8, 128), 43945), (1, (8, 1, 64), 703125)])
def test_small_launches_keep_their_kv_in_the_caches(plan_of, fp8, heads, below):
    """`below` keys of decodes are the most that take 90 MB or less."""
    row = 2 * heads[1] * heads[2] * (1 if fp8 else 2)
    assert below * row <= 90e6 < (below + 1) * row
    for chunks in ([], [(70, 300), (0, 200)]):  # whose keys do not count
        for keys in (below - (below * row == 90e6), below + 1):
            n = keys // 3
            peers = plan_of(*heads, 256, [(n - 1, 1), (n - 1, 1)] + chunks + [(keys - 2 * n - 1, 1)], fp8)
            decodes = peers[peers[:, 3] == 1]
            assert len(decodes) and ((decodes[:, 6] >= 0) == (keys > below)).all(), keys


# (heads, fp8, sequences, whether the rows are stored past the caches): 6 TB/s of streaming, 1.2 PFLOP/s of products
ROWS = [((32, 8, 128), 0, [(9763, 1), (9764, 1), (9766, 1)], 0),      # 29 296 keys, 19.9994 us
        ((32, 8, 128), 0, [(9764, 1), (9764, 1), (9766, 1)], 1),      # 29 297, 20.00009
        ((64, 8, 128), 1, [(58592, 1)], 0), ((64, 8, 128), 1, [(58593, 1)], 1),
        ((8, 8, 64), 0, [(58592, 1)], 0), ((8, 8, 64), 0, [(58593, 1)], 1),
        # products of 1024 tokens: 4 x 32 x 128 x (1024 P + 1024 x 1025 / 2) / 1.2e9 = 19.9998 and 20.014 us, streaming of 58 594 keys 40.0002
        ((32, 8, 128), 0, [(58593, 1), (918, 1024)], 1), ((32, 8, 128), 0, [(58593, 1), (919, 1024)], 0),
        ((32, 8, 128), 0, [(58593, 1), (918, 1024), (5000, 0)], 1),   # a skipped sequence does not count
        ((32, 8, 128), 0, [(40000, 8)], 1), ((32, 8, 128), 0, [(40000, 9)], 0),  # 32 rows stream, 36 are a tile
        ((64, 1, 128), 0, [(300000, 1)], 1), ((32, 8, 128), 0, [(100, 700), (0, 40)], 0), ((32, 8, 128), 0, [(100, 0)], 0)]


@pytest.mark.parametrize("case", range(len(ROWS)))
def test_which_iterations_place_their_rows_past_the_caches(plan_of, case):
    heads, fp8, seqs, past = ROWS[case]
    plan_of(*heads, 256, seqs, fp8)
    assert plan_of.rows_past == past


@pytest.mark.parametrize("heads, fp8, chunk", [((32, 8, 128), 0, (918, 1024)), ((64, 8, 128), 1, (918, 512)), ((8, 2, 64), 0, (2000, 3000))])
def test_decodes_next_to_long_products_keep_out_of_the_caches(plan_of, heads, fp8, chunk):
    """Products of 20 us at 1.2 PFLOP/s, with one decode of few keys next to them."""
    us = lambda P, C: 4 * heads[0] * heads[2] * (C * P + C * (C + 1) / 2) / 1.2e9
    P, C = chunk
    while us(P, C) < 20:
        P += 1
    while us(P - 1, C) >= 20:
        P -= 1
    for p, past in ((P - 1, False), (P, True)):
        items = plan_of(*heads, 256, [(500, 1), (p, C)], fp8)
        assert ((items[items[:, 3] == 1][:, 6] >= 0) == past).all(), p
