"""The compact form of the work list, which the entry point for callers that cannot allocate
uploads: for every batch it accepts, each reference must expand to the record of the ordinary
list, bit for bit (under AddressSanitizer and UndefinedBehaviorSanitizer).  Batches: decodes
unsplit and split, chunks with narrow tails, tiles cut into spans, half tiles, more than 32
heads per KV head, one KV head, more references than 16 bits hold, empty chunks, a launch with
more rows to cut than merge groups; and lists that the compact form cannot express, which must
be refused, not mangled: more than 255 head groups, a row whose first partial slot is beyond 16
bits, and merge groups that run out between the KV heads of a tile."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_17357_amd", "csrc")


def _cases():
    rng = np.random.default_rng(60)
    cases = [
        ("decodes", 32, 8, 128, 256, [(int(p), 1) for p in rng.integers(100, 4000, 64)]),
        ("split decodes", 32, 8, 128, 256, [(int(p), 1) for p in rng.integers(3000, 30000, 9)]),
        ("one decode", 8, 1, 64, 256, [(33000, 1)]),
        ("tile spans and tails", 28, 4, 128, 256, [(9000, 163), (2000, 1), (0, 0), (5, 37)]),
        ("half tiles", 32, 8, 128, 256, [(300, 500), (20, 1)]),
        ("two head groups", 64, 1, 64, 64, [(200, 70), (9000, 1), (3, 33)]),
        ("many tiles", 32, 8, 128, 304, [(0, 7000), (100, 9000)]),
        ("many sequences", 4, 2, 64, 256, [(int(p), int(c)) for p, c in zip(rng.integers(0, 900, 9000), rng.integers(0, 3, 9000))]),
        ("no merge groups left", 8, 8, 64, 4096, [(int(p), 1) for p in rng.integers(5000, 9000, 600)]),
        ("refused: 257 head groups", 8224, 1, 64, 256, [(300, 1), (40, 3)]),
        ("refused: partial slots beyond 16 bits", 32, 8, 128, 256, [(400000, 1)] * 100),
        ("refused: groups end between KV heads", 3, 3, 64, 8400, [(20000, 256)] * 1400),
    ]
    for i in range(40):
        n = int(rng.integers(1, 60))
        hq, hkv, d = [(8, 2, 64), (32, 8, 128), (28, 4, 128), (64, 8, 128), (40, 1, 64)][i % 5]
        P = rng.integers(0, int(rng.choice([50, 3000, 20000])), n)
        C = np.where(rng.random(n) < 0.6, 1, rng.integers(0, int(rng.choice([30, 700])), n))
        cases.append((f"random {i}", hq, hkv, d, int(rng.choice([1, 64, 256])), list(zip(P.tolist(), C.tolist()))))
    return cases


def test_every_accepted_list_expands_to_the_records(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "compact_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "compact_check_main.cpp"), os.path.join(CSRC, "plan.cpp"),
                    "-o", exe], check=True)
    cases = _cases()
    text = "\n".join(" ".join(map(str, [hq, hkv, d, cus, len(seqs)] + [x for s in seqs for x in s]))
                     for _, hq, hkv, d, cus, seqs in cases)
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)  # the sanitizer runtime must come first in the library list
    r = subprocess.run([exe], input=text + "\n", capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stderr[-3000:]
    replies = [tuple(map(int, ln.split())) for ln in r.stdout.splitlines()]
    assert len(replies) == len(cases)
    for (name, *_), (accepted, items, nbytes, bad) in zip(cases, replies):
        assert bad == 0, name
        assert not accepted or nbytes <= 64 * items, name
    by_name = {c[0]: rep for c, rep in zip(cases, replies)}
    for name in ("decodes", "split decodes", "one decode", "tile spans and tails", "half tiles", "two head groups",
                 "many tiles", "many sequences", "no merge groups left"):
        assert by_name[name][0] == 1, name
    for name in by_name:
        assert not (name.startswith("refused") and by_name[name][0]), name
    assert by_name["decodes"][2] <= 3840  # one launch's arguments
