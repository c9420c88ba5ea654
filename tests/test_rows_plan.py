"""Workgroups of the row form (csrc/swr_rows_plan.h, host code): every task of a
list is in one workgroup of its own form, and the waves are full wherever
enough tasks have the form -- also where every problem has its own potential and
so every task its own factor record."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_02564_amd", "csrc")
# rows per task, record in LDS, waves per workgroup: kRowsKind
KINDS = [(4, False, 1), (1, False, 1), (1, True, 2), (2, False, 1), (2, True, 2)]

CASES = [   # (potential per problem, problems, subdomains, cells from, to)
    (1, 20, 150, 40, 127), (1, 30, 100, 40, 240), (1, 32, 64, 130, 250), (0, 20, 150, 40, 127),
    (0, 32, 200, 40, 500), (0, 64, 100, 150, 220), (1, 3, 7, 1, 500), (0, 1, 40, 500, 700),
]


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("plan") / "rows_plan_check")
    r = subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC,
                        os.path.join(ROOT, "tests", "rows_plan_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("vpp,B,N,lo,hi", CASES)
def test_workgroups_are_whole_and_full(check, vpp, B, N, lo, hi):
    J = np.random.default_rng(1).integers(lo, hi + 1, N)
    r = subprocess.run([check], input=f"{vpp} {B} {N} " + " ".join(map(str, J)), capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.endswith("end\n")
    lines = [x.split() for x in r.stdout.splitlines()[:-1]]
    for q in (0, 1):
        tasks = [tuple(map(int, x[2:])) for x in lines if x[0] == "t" and int(x[1]) == q]
        assert len(tasks) == B * N + (0 if q else (B if vpp else 1) * (2 * N - 2))
        seen, waves = set(), {}
        for x in lines:
            if x[0] != "w" or int(x[1]) != q:
                continue
            kind, first, count, P = map(int, x[2:])
            rw, lds, nw = KINDS[kind]
            mine = tasks[first:first + count]
            assert 1 <= count <= nw * (4 // rw) and len(mine) == count
            assert {t[2] for t in mine} == {P + 32 * rw} and (P >= 9) == lds
            if lds:
                assert len({t[1] for t in mine}) == 1
            assert not seen & set(range(first, first + count))
            seen |= set(range(first, first + count))
            key = (P + 32 * rw, mine[0][1] if lds else -1)
            waves.setdefault(key, [0, 0, nw * (4 // rw)])
            waves[key][0] += 1
            waves[key][1] += count
        assert seen == {i for i, t in enumerate(tasks) if t[2]}
        for key, (n, count, cap) in waves.items():
            assert n == math.ceil(count / cap), key
