"""The direct family's LDS layout (direct_layout.cpp, built with the undefined-behaviour
sanitizer): every valid schedule of layers of each filter path stays inside its LDS."""
import os
import re
import subprocess

from paper_2008_03602_amd import workloads as W

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


def test_every_lds_schedule_stays_inside_its_lds(tmp_path):
    exe = str(tmp_path / "direct_layout")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "direct_layout.cpp"),
           os.path.join(CSRC, "schedule.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    listing = tmp_path / "ops.txt"
    listing.write_text("".join(" ".join(str(v) for v in o.as_tuple()) + "\n" for o in OPS))
    p = subprocess.run([exe, str(listing)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert p.returncode == 0, p.stdout[-3000:]
    rows = [[int(v) for v in re.findall(r"\d+", l)] for l in p.stdout.splitlines() if l.startswith("op ")]
    assert len(rows) == len(OPS) and all(r[1] > 0 for r in rows)
    # each way a chunk can go is taken
    assert all(sum(r[i] for r in rows) > 1000 for i in (2, 3, 4))
