"""The kernel names that the C ABI reports (traces and counter runs are searched by them)
against the kernels the library holds: every instance that a schedule names exists, with
all its template arguments."""
import random
import re
import subprocess

import pytest

from paper_2008_03602_amd import _lib as L, workloads as W


def _f32(name, c, h, k, r, s, stride, pad, groups=1, n=1, w=None, dil=1):
    return W.Op(name, n, c, h, w or h, k, r, s, stride, stride, pad, pad, dil, dil, groups, 0, 0)


OPS = W.resnet18() + W.mobilenet_v2_depthwise(16) + W.mobilenet_v2_pointwise(16) + [
    _f32("f5", 24, 28, 48, 5, 5, 1, 2),
    _f32("f5s2", 24, 28, 48, 5, 5, 2, 2),
    _f32("f7s1", 16, 28, 32, 7, 7, 1, 3),
    _f32("f4", 32, 28, 64, 4, 4, 1, 1),
    _f32("f2", 32, 28, 64, 2, 2, 1, 0),
    _f32("dil", 32, 28, 64, 3, 3, 1, 2, dil=2),
    _f32("dw5", 32, 28, 32, 5, 5, 1, 2, groups=32),
    # blocks whose planes span more than 2^30 bytes, fixed filters and another one
    _f32("wide3", 2, 8200, 2, 3, 3, 1, 1, groups=2, w=16400),
    _f32("wide3s2", 2, 8200, 2, 3, 3, 2, 1, groups=2, w=16400),
    _f32("wide5", 2, 8200, 2, 5, 5, 1, 2, groups=2, w=16400),
    W.Op("pw960", 16, 960, 7, 7, 320, 1, 1, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
    W.Op("pw1024", 1, 1024, 14, 14, 1024, 1, 1, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
]


@pytest.fixture(scope="module")
def kernels():
    out = subprocess.run(["nm", "-C", L.LIB_PATH], stdout=subprocess.PIPE, text=True, check=True).stdout
    names = set(re.findall(r"\bct::((?:direct|depthwise|igemm)_\w*kernel<[^>]*>)", out))
    assert names
    return names


@pytest.mark.parametrize("op", OPS, ids=lambda o: o.name)
def test_reported_kernel_names_are_the_librarys(op, kernels):
    space = L.ct_valid_space(op)
    assert space
    for s in random.Random(4).sample(space, min(1500, len(space))):
        assert L.ct_kernel_name(op, s) in kernels, (op.name, L.schedule_tuple(s))


def test_wide_depthwise_blocks_are_named_as_such(kernels):
    wide = next(o for o in OPS if o.name == "wide3")
    s = L.make_schedule(W.FAM_DEPTHWISE_F32, (2, 8, 64, 2, 2, 0, 1, 0, 0))
    assert L.ct_kernel_name(wide, s).endswith(", true>")
    small = _f32("small", 2, 64, 2, 3, 3, 1, 1, groups=2, w=64)
    assert L.ct_kernel_name(small, s) == "depthwise_f32_kernel<2, 2, false, 3, false>"
    # fixed filters keep their path without LDS
    assert L.ct_kernel_name(wide, s) == "depthwise_f32_kernel<2, 2, false, 3, true>"
    # what counts is what one block reaches: here 16 planes of 8 MB of an image of 1 GB, or
    # the same channels of two images
    hd = _f32("hd", 128, 1088, 128, 3, 3, 1, 1, groups=128, n=2, w=1920)
    for nb, ending in ((1, "false>"), (2, "true>")):
        t = L.make_schedule(W.FAM_DEPTHWISE_F32, (16, 8, 16, 2, 2, 0, nb, 0, 0))
        assert L.ct_validate(hd, t) == L.S_OK
        assert L.ct_kernel_name(hd, t).endswith(ending)
    # the kernel of 4 consecutive columns addresses planes of any size
    q4 = L.make_schedule(W.FAM_DEPTHWISE_F32, (2, 8, 64, 4, 2, 0, 1, 0, 1))
    assert L.ct_kernel_name(wide, q4) == "depthwise_q4_kernel<1, 2>"
