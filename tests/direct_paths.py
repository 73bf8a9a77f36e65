"""Which way a direct schedule reads its operands, from the facts of the schedule: the
library's rules for the LDS layout and what an instance's registers hold, restated
(compared with them for every schedule by test_host_direct_layout.py)."""
from __future__ import annotations

import re

from paper_2008_03602_amd import _lib as L

TOH, TOW, TK, MK, MW, LDS, CT, SPLIT, UNROLL = range(9)


def _up(a, b):
    return -(-a // b)


def kernel(op, s):
    """(specialisation, variant) of the schedule's kernel, by its name."""
    m = re.match(r"direct_f32_kernel<\d, \d, (?:true|false), (\d), \d, (true|false)>", L.ct_kernel_name(op, s))
    return int(m.group(1)), m.group(2) == "true"


def held(mk, mw, spec):
    """(staged words per thread, copies planned) beside the accumulators and the ring."""
    cols = {0: 0, 1: 1, 2: 1, 3: 3, 4: 3, 5: 5, 6: 5, 7: 7, 8: 7}[spec]
    stride = 0 if spec == 0 else (1 if spec % 2 else 2)
    limit = 256 if mk * mw >= 16 else 128
    unit = 4 * (mw + mk) if cols == 1 else (((mw - 1) * stride + cols + cols * mk) if cols else 2)
    clocks = 16 * mk * mw if cols == 1 else 4 * cols * mk * mw
    want = 2 if clocks >= 160 else (3 if clocks >= 48 or cols == 1 else 4)
    ring = max(1, min(want, (limit - mk * mw - 72) // unit))
    left = limit - mk * mw - (ring * unit if cols else 24)
    words = (left - (60 if cols == 1 else 44)) // 2
    staged = 24 if words >= 24 and limit == 256 else next((n for n in (16, 12, 8) if words >= n), 6)
    return staged, max(4, min(12, (left - 56) // 2))


def lds_way(op, s):
    """How a chunk of a schedule with LDS gets there: ("staged", words per thread) through
    registers, ("plan",) by copies whose offsets are kept, ("deep", ...) by 16-byte filter
    copies without a plan, ("copied", ...) word by word; the flags say whether planes, and
    groups' slices, are copied one by one."""
    k = s.knob
    spec, alt = kernel(op, s)
    mk, mw, ct, groups = k[MK], k[MW], k[CT], k[TK] // k[MK]
    threads = groups * k[TOH] * (k[TOW] // mw)
    ih = (k[TOH] - 1) * op.stride_h + (op.r - 1) * op.dil_h + 1
    iw = (k[TOW] - 1) * op.stride_w + (op.s - 1) * op.dil_w + 1
    wpc = ct * op.r * op.s
    pitch, ks = iw, wpc * mk
    if spec:
        step = mw * op.stride_w
        unit = 1 if spec == 2 else (4 if step % 4 == 0 else (2 if step % 2 == 0 else 1))
        pitch = _up(iw, unit) * unit
        wa = 4 if mk > 1 or wpc % 4 == 0 else 1
        ks = (_up(ks, wa) | 1) * wa
    plane = ih * pitch
    staged, plan = held(mk, mw, spec)

    def rows(words):
        return _up(words, threads)

    def fills(words):
        return int(2 * words > rows(words) * threads)

    if spec and alt:
        if max(rows(groups * ks // 4), rows(ct * plane)) <= plan:
            return ("plan",)
        return ("deep", fills(plane), fills(ks // 4), fills(ks))
    nst = rows(groups * ks) + rows(ct * plane)
    return ("staged", nst) if nst <= staged else ("copied", fills(plane), fills(ks))
