"""The direct family's LDS layout (direct_layout.cpp, built with the undefined-behaviour
sanitizer): every valid schedule of layers of each filter path stays inside its LDS."""
import os
import re
import subprocess

import pytest

import direct_paths as DP
from paper_2008_03602_amd import _lib as L, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_03602_amd", "csrc")


def _f32(name, n, c, h, w, k, r, s, stride, pad, dil=(1, 1)):
    return W.Op(name, n, c, h, w, k, r, s, stride, stride, pad[0], pad[1], dil[0], dil[1], 1, 0, 0)


OPS = W.resnet18() + [
    _f32("pw_odd", 2, 37, 27, 29, 50, 1, 1, 1, (0, 0)),
    _f32("pw_s2_odd", 1, 18, 9, 11, 20, 1, 1, 2, (0, 0)),
    _f32("c13", 1, 13, 6, 30, 10, 3, 3, 2, (1, 1)),
    _f32("f5", 2, 24, 28, 28, 48, 5, 5, 1, (2, 2)),
    _f32("f5s2", 1, 6, 31, 35, 18, 5, 5, 2, (2, 1)),
    _f32("f7", 1, 16, 28, 28, 32, 7, 7, 1, (3, 3)),
    _f32("rect3x7s2", 2, 12, 29, 40, 32, 3, 7, 2, (0, 4)),
    _f32("dilh5", 1, 8, 34, 30, 16, 3, 5, 1, (2, 2), (4, 1)),
    _f32("f4", 1, 32, 28, 28, 64, 4, 4, 1, (1, 1)),
    _f32("dil", 1, 64, 28, 28, 64, 3, 3, 1, (2, 2), (2, 2)),
]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("direct_layout")
    exe = str(tmp / "direct_layout")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "direct_layout.cpp"),
           os.path.join(CSRC, "schedule.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(ops, *args):
        listing = tmp / "ops.txt"
        listing.write_text("".join(" ".join(str(v) for v in o.as_tuple()) + "\n" for o in ops))
        p = subprocess.run([exe, str(listing)] + list(args), stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                           text=True, timeout=300)
        assert p.returncode == 0, p.stdout[-3000:]
        return p.stdout.splitlines()
    return run


def test_every_lds_schedule_stays_inside_its_lds(driver):
    lines = driver(OPS)
    rows = [[int(v) for v in re.findall(r"\d+", l)] for l in lines if l.startswith("op ")]
    assert len(rows) == len(OPS) and all(r[1] > 0 for r in rows)
    # each way a chunk can go is taken
    assert all(sum(r[i] for r in rows) > 1000 for i in (2, 3, 4))


@pytest.mark.parametrize("op", OPS[::3] + OPS[-2:], ids=lambda o: o.name)
def test_the_ways_that_the_gpu_tests_pick_by_are_the_librarys(driver, op):
    n = 0
    for line in driver([op], "list"):
        f = line.split()
        if f[0].isdigit():
            n += 1
            if n % 7 == 0:  # names are asked for one by one
                s = L.make_schedule(W.FAM_DIRECT_F32, [int(v) for v in f[:9]])
                assert DP.lds_way(op, s) == (f[9],) + tuple(int(v) for v in f[10:]), line
    assert n > 100
