"""GPU parity at the edges of the kernels' own choices of path: sizes where an index, a
load width or an address range changes, against the fp64 oracle (or, for tensors too large
for it, against shifted sums in torch)."""
import random

import numpy as np
import pytest
import torch

from paper_2008_03602_amd import _lib as L, workloads as W
from gpu_util import check_close, device_ready, make_inputs, note, reference, sched_str, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    device_ready()
    yield


def _dw(name, n, c, h, w, r, s, stride, pad):
    return W.Op(name, n, c, h, w, c, r, s, stride, stride, pad[0], pad[1], 1, 1, c, 0, 0)


# one-row and one-column maps, channel and image groups that run past the tensor, a
# rectangular filter and a stride the fixed paths do not take
DW_EDGES = [
    _dw("row", 3, 5, 1, 9, 3, 3, 1, (1, 1)),
    _dw("column", 2, 17, 9, 1, 3, 3, 2, (1, 1)),
    _dw("wide33", 5, 6, 6, 33, 3, 3, 1, (1, 1)),
    _dw("s2_31", 3, 3, 31, 30, 3, 3, 2, (1, 1)),
    _dw("rect1x5", 2, 9, 8, 13, 1, 5, 1, (0, 2)),
    _dw("stride3", 1, 4, 16, 16, 3, 3, 3, (1, 1)),
]


@pytest.mark.parametrize("op", DW_EDGES, ids=lambda o: o.name)
def test_depthwise_edges_match_oracle(op):
    x, w = make_inputs(op, "uniform", seed=41)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    space = L.ct_valid_space(op)
    for s in random.Random(6).sample(space, min(48, len(space))):
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, tag)


def _f32(name, n, c, h, w, k, r, s, stride, pad):
    return W.Op(name, n, c, h, w, k, r, s, stride, stride, pad[0], pad[1], 1, 1, 1, 0, 0)


# direct family: channel counts below and off the ring's depth, windows wider than the
# image, both strides of the 5- and 7-column paths with uneven padding and rectangular
# filters, and shapes that stay on the generic path, with rows of fewer than four taps and
# of one, two and more groups of them
DIRECT_EDGES = [
    _f32("c1", 2, 1, 5, 6, 9, 3, 3, 1, (1, 1)),
    _f32("c13", 1, 13, 6, 3, 10, 3, 3, 2, (1, 1)),
    _f32("pw_c7", 2, 7, 5, 9, 12, 1, 1, 1, (0, 0)),
    _f32("pw_s2_c18", 1, 18, 9, 11, 20, 1, 1, 2, (0, 0)),
    _f32("f5", 2, 3, 9, 13, 10, 5, 5, 1, (2, 2)),
    _f32("f5s2", 1, 6, 11, 15, 18, 5, 5, 2, (2, 1)),
    _f32("f7", 1, 4, 8, 5, 6, 7, 7, 1, (3, 3)),
    _f32("f7s2", 1, 3, 21, 18, 20, 7, 7, 2, (3, 3)),
    _f32("rect2x5", 1, 9, 7, 12, 8, 2, 5, 1, (1, 0)),
    _f32("rect3x7s2", 2, 5, 9, 16, 8, 3, 7, 2, (0, 4)),
    _f32("f4", 1, 5, 9, 10, 8, 4, 4, 1, (1, 1)),
    _f32("f6s2", 2, 3, 15, 13, 12, 6, 6, 2, (2, 2)),
    _f32("row9", 1, 4, 7, 17, 9, 2, 9, 1, (0, 4)),
    W.Op("dil2x11", 1, 3, 9, 34, 8, 3, 11, 1, 1, 1, 10, 1, 2, 1, 0, 0),
    W.Op("dilh5", 1, 4, 14, 10, 8, 3, 5, 1, 1, 2, 2, 2, 1, 1, 0, 0),
]


@pytest.mark.parametrize("op", DIRECT_EDGES, ids=lambda o: o.name)
def test_direct_edges_match_oracle(op):
    x, w = make_inputs(op, "uniform", seed=43)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    space = [s for s in L.ct_valid_space(op) if s.family == W.FAM_DIRECT_F32]
    # one schedule of every kernel, then a sample
    by = {}
    for s in random.Random(8).sample(space, len(space)):
        by.setdefault(L.ct_kernel_name(op, s), s)
    for s in list(by.values()) + random.Random(9).sample(space, min(40, len(space))):
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, tag, split=4)


def test_direct_tiles_whose_padded_layout_exceeds_the_lds_run_generic():
    op = W.conv("b3x3s2", 1, 64, 30, 64, 3, 2)
    x, w = make_inputs(op, "uniform", seed=44)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    for knobs in ((14, 16, 32, 2, 4, 1, 32, 1, 1), (14, 16, 32, 2, 4, 1, 32, 2, 2), (14, 16, 32, 2, 4, 1, 16, 1, 1)):
        s = L.make_schedule(W.FAM_DIRECT_F32, knobs)
        assert L.ct_validate(op, s) == L.S_OK
        generic = ", 0, " in L.ct_kernel_name(op, s)
        assert generic == (knobs[6] == 32)
        note("b3x3s2 " + sched_str(s))
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, sched_str(s), split=4)


# two planes of 512 MB and more (a block's planes span more than 2^30 bytes) with each filter
# path, and 128 planes of 8 MB, of which a block's 16 do not
@pytest.mark.parametrize("op,tc,wide", [
    (_dw("huge", 1, 2, 8200, 16400, 3, 3, 1, (1, 1)), 2, True),
    (_dw("huge_s2", 1, 2, 8200, 16400, 3, 3, 2, (1, 1)), 2, True),
    (_dw("huge_5x3", 1, 2, 8200, 16400, 5, 3, 1, (2, 1)), 2, True),
    (_dw("hd", 1, 128, 1088, 1920, 3, 3, 1, (1, 1)), 16, False),
], ids=lambda v: getattr(v, "name", None))
def test_depthwise_planes_around_the_32_bit_part_offsets(op, tc, wide):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    xd = torch.rand(op.x_shape(), generator=gen, device="cuda") * 2 - 1
    wd = torch.rand(op.w_shape(), generator=gen, device="cuda") * 2 - 1
    ref = torch.zeros(op.y_shape(), device="cuda")
    p = torch.nn.functional.pad(xd, (op.pad_w, op.pad_w, op.pad_h, op.pad_h))
    st = op.stride_h
    for r in range(op.r):
        for s in range(op.s):
            part = p[:, :, r:r + (op.oh - 1) * st + 1:st, s:s + (op.ow - 1) * st + 1:st]
            ref += part * wd[:, :, r, s].reshape(1, -1, 1, 1)
    del p
    yd = torch.empty(op.y_shape(), device="cuda")
    n = op.r * op.s
    for lds in (0, 1):
        s = L.make_schedule(W.FAM_DEPTHWISE_F32, (tc, 8, 64 if tc == 2 else 16, 2, 2, lds, 1, 0, 0))
        assert L.ct_validate(op, s) == L.S_OK
        assert L.ct_kernel_name(op, s).endswith("true>" if wide else "false>")
        note(op.name + " " + sched_str(s))
        yd.fill_(float("nan"))
        torch.cuda.synchronize()
        L.conv2d_run(op, s, xd, wd, yd)
        # n products of at most 1: both sums err by at most n roundings of at most n * 2^-24
        assert float((yd - ref).abs().max()) <= 2 * n * n * 2.0 ** -24


# Infinities and NaN reach the outputs whose taps read them and no others: a window is read
# past an image's edge into the neighbouring row or plane, tiles and chunks past the tensor.
SPECIAL_OPS = [
    _f32("sv3", 2, 5, 6, 7, 9, 3, 3, 1, (1, 1)),
    _f32("sv3s2", 1, 6, 9, 11, 10, 3, 3, 2, (1, 1)),
    _f32("sv1", 1, 7, 5, 9, 12, 1, 1, 1, (0, 0)),
    _f32("sv1s2", 1, 9, 7, 9, 12, 1, 1, 2, (0, 0)),
    _f32("sv5", 1, 3, 7, 9, 6, 5, 5, 1, (2, 2)),
    _f32("sv7s2", 1, 3, 13, 11, 6, 7, 7, 2, (3, 3)),
    _f32("sv4", 1, 3, 7, 10, 6, 4, 4, 1, (1, 1)),
    _dw("svdw", 2, 5, 6, 9, 3, 3, 1, (1, 1)),
    _dw("svdw_s2", 1, 5, 9, 12, 3, 3, 2, (1, 1)),
    W.Op("svbf", 1, 24, 5, 7, 17, 1, 1, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
]


@pytest.mark.parametrize("op", SPECIAL_OPS, ids=lambda o: o.name)
def test_special_values_stay_where_they_are_read(op):
    bf16 = op.dtype == W.DT_BF16
    x, w = make_inputs(op, "uniform", seed=48)
    img = x if not bf16 else x.transpose(0, 3, 1, 2)  # a view: NCHW
    # the last column of the first row (the next row follows it), the first pixel of a
    # channel (the row before it ends the plane before), the last pixel of the last channel
    img[0, 0, 0, -1] = np.nan
    img[0, 1, 0, 0] = np.inf
    img[-1, -1, -1, -1] = -np.inf
    # which taps an output reads: the same layer over marks; a zero weight on a special
    # value counts (0 * inf is NaN), and there is none
    assert (w != 0).all()
    marks = np.zeros_like(x)
    marks[~np.isfinite(x)] = 1
    touched, _ = reference(op, marks, np.ones_like(w))
    ref, a = reference(op, np.where(np.isfinite(x), x, 0).astype(x.dtype), w)
    nans = np.zeros_like(x)
    nans[np.isnan(x)] = 1
    nan_at, _ = reference(op, nans, np.ones_like(w))
    xd, wd, yd = to_device(op, x, w)
    space = [s for s in L.ct_valid_space(op) if s.family != W.FAM_IGEMM_F32]
    by = {}  # one schedule of every kernel, then a sample
    for s in random.Random(14).sample(space, len(space)):
        by.setdefault(L.ct_kernel_name(op, s), s)
    for s in list(by.values()) + random.Random(15).sample(space, min(30, len(space))):
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        y = yd.cpu().numpy()
        assert np.array_equal(np.isfinite(y), touched == 0), tag
        assert np.isnan(y[nan_at > 0]).all(), tag
        check_close(op, np.where(touched == 0, y, 0), np.where(touched == 0, ref, 0), np.where(touched == 0, a, 1), tag,
                    split=4)


def test_padding_of_an_image_that_ends_just_before_2_gib():
    # x of 2^29 - 2 words: what lies outside the image must not read its last words, the only
    # ones that are not 0
    op = _f32("end", 1, 2, 18705, 14351, 1, 3, 3, 1, (1, 1))
    xd = torch.zeros(op.x_shape(), device="cuda")
    assert xd.numel() == 2 ** 29 - 2
    xd.view(-1)[-2:] = 1e6
    wd = torch.ones(op.w_shape(), device="cuda")
    yd = torch.empty(op.y_shape(), device="cuda")
    ref = torch.zeros(op.y_shape(), device="cuda")
    ref[0, 0, -2:, -3] = 1e6
    ref[0, 0, -2:, -2:] = 2e6
    for fam, knobs in ((W.FAM_DIRECT_F32, (8, 32, 4, 4, 4, 1, 2, 1, 1)),
                       (W.FAM_DIRECT_F32, (8, 32, 4, 4, 4, 0, 2, 1, 1)),
                       (W.FAM_DIRECT_F32, (14, 16, 4, 1, 1, 1, 1, 1, 1)),
                       (W.FAM_IGEMM_F32, (16, 1, 4, 1, 4, 1, 64, 2, 1, 1))):
        s = L.make_schedule(fam, knobs)
        assert L.ct_validate(op, s) == L.S_OK
        note("end " + sched_str(s))
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        assert torch.equal(yd, ref), sched_str(s)


def _pw(name, n, c, h, w, k, stride=1):
    return W.Op(name, n, c, h, w, k, 1, 1, stride, stride, 0, 0, 1, 1, 1, W.DT_BF16, W.LAYOUT_NHWC)


# reductions of one group of 8, off every chunk and step length, and longer than the steps
# in flight; channel and pixel counts off every tile; a stride
BF16_EDGES = [
    _pw("c8k1", 1, 8, 5, 7, 1),
    _pw("c24k17", 3, 24, 5, 5, 17),
    _pw("c40k30", 2, 40, 9, 7, 30),
    _pw("c136k65s2", 2, 136, 9, 11, 65, 2),
    _pw("c328k130", 1, 328, 11, 13, 130),
    _pw("c648k48", 1, 648, 7, 9, 48),
]


@pytest.mark.parametrize("op", BF16_EDGES, ids=lambda o: o.name)
def test_bf16_edges_match_oracle(op):
    x, w = make_inputs(op, "uniform", seed=45)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    space = L.ct_valid_space(op)
    # one schedule of every kernel, then a sample
    by = {}
    for s in random.Random(10).sample(space, len(space)):
        by.setdefault(L.ct_kernel_name(op, s), s)
    for s in list(by.values()) + random.Random(11).sample(space, min(40, len(space))):
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, tag, split=4)


def _shifted(t, shift):
    """The same values `shift` elements past an allocation's start."""
    u = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)
    u[shift:] = t.reshape(-1)
    return u[shift:].reshape(t.shape)


# one chunk and a part of one, and more chunks than LDS holds at once
@pytest.mark.parametrize("op", [_pw("off72", 2, 72, 9, 7, 40), _pw("off648", 1, 648, 11, 13, 130)],
                         ids=lambda o: o.name)
@pytest.mark.parametrize("shift", [1, 2, 4])
def test_bf16_tensors_off_16_byte_addresses(op, shift):
    x, w = make_inputs(op, "uniform", seed=46)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    space = L.ct_valid_space(op)
    by = {}  # one schedule of every kernel that uses LDS, then a sample
    for s in random.Random(13).sample(space, len(space)):
        if s.knob[6]:
            by.setdefault(L.ct_kernel_name(op, s), s)
    for xs, ws in ((_shifted(xd, shift), wd), (xd, _shifted(wd, shift)), (_shifted(xd, shift), _shifted(wd, shift))):
        for s in list(by.values()) + random.Random(12).sample(space, 16):
            tag = "%s by %d %s" % (op.name, shift, sched_str(s))
            note(tag)
            yd.fill_(float("nan"))
            L.conv2d_run(op, s, xs, ws, yd)
            check_close(op, yd.cpu().numpy(), ref, a, tag, split=4)


def test_bf16_tensors_off_16_byte_addresses_are_still_staged_once():
    # a block reads a tensor off 16-byte addresses once into LDS, as it does others: its
    # loads straddle lines and go through registers, but not once per wave that needs them
    # (3.5 to 4 times as long on these schedules)
    op = _pw("deep", 1, 1024, 14, 14, 1024)
    xd = (torch.rand(op.x_shape(), device="cuda") * 2 - 1).to(torch.bfloat16)
    wd = (torch.rand(op.w_shape(), device="cuda") * 2 - 1).to(torch.bfloat16)
    yd = torch.empty(op.y_shape(), device="cuda")
    scheds = [L.make_schedule(W.FAM_IGEMM_BF16, k) for k in ((32, 1, 1, 2, 4, 128, 1, 2, 1), (32, 1, 1, 4, 2, 64, 1, 2, 0),
                                                             (16, 4, 4, 4, 2, 32, 1, 2, 1))]
    assert all(L.ct_validate(op, s) == L.S_OK for s in scheds)
    opts = L.make_opts(3, 11, 10, 3)
    lat, st = L.measure_candidates(op, scheds, 1.0, opts, xd, wd, yd)
    off, st2 = L.measure_candidates(op, scheds, 1.0, opts, _shifted(xd, 1), _shifted(wd, 1), yd)
    assert (st == 0).all() and (st2 == 0).all()
    print("aligned", lat, "off", off)
    assert (off < 2.5 * lat).all(), (lat, off)


def test_bf16_operand_beyond_2_gib():
    # x of 3.3 GB: byte offsets past 2^31, and the last pixels' reads end near the buffer's
    op = _pw("huge", 1, 960, 1280, 1343, 16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    xd = torch.empty(op.x_shape(), dtype=torch.bfloat16, device="cuda")
    for r in range(0, op.h, 128):
        xd[:, r:r + 128] = torch.rand(xd[:, r:r + 128].shape, generator=gen, device="cuda") * 2 - 1
    wd = (torch.rand(op.w_shape(), generator=gen, device="cuda") * 2 - 1).to(torch.bfloat16)
    yd = torch.empty(op.y_shape(), device="cuda")
    wt = wd.reshape(op.k, op.c).double().t().contiguous()
    for lds in (0, 1):
        s = L.make_schedule(W.FAM_IGEMM_BF16, (16, 2, 1, 2, 1, 128 if lds else 32, lds, 1, 0))
        assert L.ct_validate(op, s) == L.S_OK
        note("huge " + sched_str(s))
        yd.fill_(float("nan"))
        torch.cuda.synchronize()
        L.conv2d_run(op, s, xd, wd, yd)
        for r in (0, 640, 1216):  # the start, the 2 GiB boundary and past it
            d = yd[0, r:r + 64].reshape(-1, op.k).double() - xd[0, r:r + 64].reshape(-1, op.c).double() @ wt
            # 960 exact products of at most 1, and as many roundings
            assert float(d.abs().max()) <= 962 * 960 * 2.0 ** -24
