"""Byte offsets of the kernels' buffer accesses: an offset may be a sum of parts of which
each is outside the image on its own, and a multi-word access goes on past one. Such sums
exceed the largest int and have to be made unsigned. Constant evaluation refuses a
signed overflow, which makes the compiler the check (a syntax check of the host side)."""
import os
import subprocess

from paper_2008_03602_amd import build as B

UNIT = r"""
#include "k_util.h"
// a dead thread, a row outside and a column outside at once, plus the immediate
constexpr auto three = ct::part_sum(ct::kPartOob + ct::kPartOob, ct::kPartOob);
static_assert(three == 0xBFFFFFD0 && three + 4095 > three, "three parts outside stay below 2^32");
// a row and a column outside, and the later words of a window that starts outside
constexpr auto two = ct::kOob + ct::kOob;
static_assert(two == 0xFFFFFFF8, "");
// past the largest tensor, which holds fewer than 2^31 bytes in whole words
static_assert(ct::kOob >= 0x7FFFFFFF / 4 * 4 && ct::kOob % 4 == 0, "");
static_assert(ct::kOobQuad >= 0x7FFFFFFF / 4 * 4 && ct::kOobQuad % 16 == 0, "");
constexpr auto window = ct::kOob + 16 + 16 + 4;
static_assert(window > ct::kOob, "");
// one part outside sends any sum with parts inside past the largest buffer, in any order
constexpr int last = ct::kPartOob - 4;
static_assert(ct::part_sum(ct::kPartOob + 0, 0) >= ct::kPartOob, "");
static_assert(ct::part_sum(last + ct::kPartOob, last) >= ct::kPartOob, "");
static_assert(ct::part_sum(last + last, ct::kPartOob) >= ct::kPartOob, "");
"""


def test_sums_of_offset_parts_are_unsigned(tmp_path):
    src = tmp_path / "offsets.hip"
    src.write_text(UNIT)
    cmd = [B._hipcc()] + B.HIP_FLAGS + ["--offload-host-only", "-fsyntax-only", str(src)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]
