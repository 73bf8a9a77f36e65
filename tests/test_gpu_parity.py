"""GPU parity of every kernel family against the fp64 oracle, through the C ABI.

Shapes are small enough for the oracle to finish in seconds but span several
tiles with ragged tails (H, W, K and C not multiples of the tile sizes, C = 3,
stride 2, 7x7 filters). Each case runs a seeded sample of schedules from the
op's valid candidate space.
"""
import random

import numpy as np
import pytest
import torch

import direct_paths as DP
from paper_2008_03602_amd import _lib as L, workloads as W
from gpu_util import check_close, device_ready, make_inputs, note, reference, sched_str, to_device

pytestmark = pytest.mark.gpu

F32_OPS = [
    W.conv("odd3x3", 1, 5, 13, 11, 3, 1),
    W.conv("odd3x3s2", 2, 6, 15, 9, 3, 2),
    W.conv("stem7x7", 1, 3, 29, 10, 7, 2, 3),
    W.conv("pw_odd", 2, 19, 9, 21, 1, 1, 0),
    W.conv("pw_s2", 1, 24, 14, 40, 1, 2, 0),
    W.Op("rect5x3", 1, 7, 12, 17, 12, 5, 3, 1, 2, 2, 1, 1, 1, 1, 0, 0),
    W.Op("dilated", 1, 4, 11, 11, 6, 3, 3, 1, 1, 2, 2, 2, 2, 1, 0, 0),
]
DW_OPS = [
    W.conv("dw_odd", 2, 13, 15, 13, 3, 1, 1, groups=13),
    W.conv("dw_s2", 3, 24, 17, 24, 3, 2, 1, groups=24),
    W.Op("dw5x5", 1, 8, 10, 10, 8, 5, 5, 1, 1, 2, 2, 1, 1, 8, 0, 0),
]
# shapes where IGEMM_F32 copies 16 bytes per lane (W a multiple of 4), with ragged tiles
VEC_OPS = [
    W.conv("vec3x3", 1, 24, 20, 40, 3, 1),
    W.conv("vec3x3s2", 1, 16, 28, 24, 3, 2),
    W.conv("vec1x1", 2, 32, 12, 20, 1, 1, 0),
    W.Op("vec_rect", 2, 12, 9, 24, 20, 3, 3, 1, 1, 1, 1, 1, 1, 1, 0, 0),
]
BF_OPS = [
    W.conv("pwbf_odd", 2, 24, 9, 40, 1, 1, 0, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
    W.conv("pwbf_c96", 1, 96, 11, 24, 1, 1, 0, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
    W.conv("pwbf_s2", 1, 40, 13, 72, 1, 2, 0, dtype=W.DT_BF16, layout=W.LAYOUT_NHWC),
]


@pytest.fixture(scope="module", autouse=True)
def _device():
    device_ready()
    yield


def _run_sample(op, n_sched, seed, dist="uniform", int_range=2, exact=False, family=None):
    x, w = make_inputs(op, dist, seed=seed, int_range=int_range)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    if family is None:
        scheds = L.ct_sample(op, seed, 99, 0, n_sched)
    else:  # a seeded sample of one family's valid schedules
        space = [s for s in L.ct_valid_space(op) if s.family == family]
        scheds = random.Random(seed).sample(space, min(n_sched, len(space)))
    assert len(scheds) > 0
    fams = set()
    for s in scheds:
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        y = yd.cpu().numpy()
        split = W.split_of(s)
        if exact:
            assert np.array_equal(y.astype(np.float64), ref), tag + ": not bit-exact on integer inputs"
        else:
            check_close(op, y, ref, a, tag, split=4 if split > 1 else 1)
        fams.add(s.family)
    return fams


@pytest.mark.parametrize("op", F32_OPS, ids=lambda o: o.name)
def test_fp32_families_match_oracle(op):
    fams = _run_sample(op, 24, seed=11)
    assert fams <= {W.FAM_DIRECT_F32, W.FAM_IGEMM_F32}


@pytest.mark.parametrize("op", F32_OPS + VEC_OPS, ids=lambda o: o.name)
def test_fp32_mfma_schedules_match_oracle(op):
    # 24 schedules of the MFMA family alone: both staging depths, 1- and
    # 16-byte copies, register double buffering, reduction groups and splits
    assert _run_sample(op, 24, seed=14, family=W.FAM_IGEMM_F32) == {W.FAM_IGEMM_F32}


def test_misaligned_tensors_are_refused_by_16_byte_schedules():
    op = VEC_OPS[0]
    x, w = make_inputs(op, "uniform", seed=3)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    buf = torch.empty(xd.numel() + 4, dtype=torch.float32, device=xd.device)
    xm = buf[1:1 + xd.numel()].view(op.x_shape())  # 4 bytes past a 16-byte boundary
    xm.copy_(xd)
    space = L.ct_valid_space(op)
    vec = next(s for s in space if s.family == W.FAM_IGEMM_F32)
    direct = next(s for s in space if s.family == W.FAM_DIRECT_F32)
    note("misaligned x: " + sched_str(vec))
    with pytest.raises(L.CtError) as e:
        L.conv2d_run(op, vec, xm, wd, yd)
    assert e.value.code == L.CT_E_ARG and "aligned" in str(e.value)
    lat, st = L.measure_candidates_mask(op, [vec, direct], L.ct_cu_mask(1.0, 0), L.make_opts(1, 1, 2, 2),
                                        xm, wd, yd)
    assert list(st) == [L.S_LAUNCH, L.S_OK]
    yd.fill_(float("nan"))
    L.conv2d_run(op, direct, xm, wd, yd)
    check_close(op, yd.cpu().numpy(), ref, a, "misaligned x, direct schedule")


@pytest.mark.parametrize("op", DW_OPS, ids=lambda o: o.name)
def test_depthwise_matches_oracle(op):
    _run_sample(op, 24, seed=12)


# 3x3 pad-1 depthwise shapes for the 4-columns-per-thread variant: 16-byte
# loads and stores (W a multiple of 4, W = stride * OW, OW a multiple of 4),
# and the word-by-word fallback (odd widths, W != 2 OW), with ragged tiles
Q4_OPS = [
    W.conv("dwq_s1", 2, 12, 20, 12, 3, 1, 1, groups=12),
    W.conv("dwq_s2", 3, 8, 24, 8, 3, 2, 1, groups=8),
    W.conv("dwq_odd", 2, 13, 15, 13, 3, 1, 1, groups=13),
    W.conv("dwq_s2odd", 1, 6, 17, 6, 3, 2, 1, groups=6),
    W.conv("dwq_s2w14", 2, 10, 14, 10, 3, 2, 1, groups=10),
]


def _q4_sample(op, n, seed):
    space = [s for s in L.ct_valid_space(op) if s.family == W.FAM_DEPTHWISE_F32 and s.knob[8] == 1]
    assert space, op.name
    return random.Random(seed).sample(space, min(n, len(space)))


@pytest.mark.parametrize("op", Q4_OPS, ids=lambda o: o.name)
def test_depthwise_q4_matches_oracle_and_is_exact_on_integers(op):
    x, w = make_inputs(op, "uniform", seed=31)
    ref, a = reference(op, x, w)
    xi, wi = make_inputs(op, "int", seed=32)
    refi, _ = reference(op, xi, wi)
    xd, wd, yd = to_device(op, x, w)
    xid, wid, yid = to_device(op, xi, wi)
    for s in _q4_sample(op, 16, seed=33):
        tag = "%s %s" % (op.name, sched_str(s))
        note(tag)
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, tag)
        yid.fill_(float("nan"))
        L.conv2d_run(op, s, xid, wid, yid)
        assert np.array_equal(yid.cpu().numpy().astype(np.float64), refi), tag + ": not bit-exact on integers"


@pytest.mark.parametrize("op", BF_OPS, ids=lambda o: o.name)
def test_bf16_pointwise_matches_oracle(op):
    _run_sample(op, 24, seed=13)


@pytest.mark.parametrize("op", [F32_OPS[0], F32_OPS[3], DW_OPS[0]], ids=lambda o: o.name)
def test_integer_inputs_bit_exact_fp32(op):
    _run_sample(op, 16, seed=21, dist="int", int_range=2, exact=True)


@pytest.mark.parametrize("op", [BF_OPS[0], BF_OPS[1]], ids=lambda o: o.name)
def test_integer_inputs_bit_exact_bf16(op):
    _run_sample(op, 16, seed=22, dist="int", int_range=8, exact=True)


def test_every_family_covered_on_config1_shape():
    op = W.config(1).ops[0]
    x, w = make_inputs(op, "uniform", seed=0, config_id=1)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    scheds = L.ct_sample(op, 0, 1, 0, 64)
    for s in scheds:
        note("config1 " + sched_str(s))
        yd.fill_(float("nan"))
        L.conv2d_run(op, s, xd, wd, yd)
        check_close(op, yd.cpu().numpy(), ref, a, "config1 " + sched_str(s), split=4)


def _direct_class(op, s):
    """Which operand path a direct schedule takes: its kernel's specialisation and variant,
    and with LDS the way its chunks go there (staged words by the lengths that have loops
    of their own)."""
    spec, alt = DP.kernel(op, s)
    if not s.knob[DP.LDS]:
        return "regs spec %d%s" % (spec, " scalar-w" if alt else "")
    way = DP.lds_way(op, s)
    if way[0] == "staged":
        return "lds spec %d staged-%d" % (spec, next(n for n in (2, 4, 6, 8, 12, 16, 24) if way[1] <= n))
    return "lds spec %d " % spec + " ".join(str(v) for v in way)


STAGING_OPS = [W.conv("deep3x3", 1, 48, 9, 72, 3, 1), F32_OPS[1], F32_OPS[4], F32_OPS[5],
               W.conv("pw52", 1, 52, 13, 36, 1, 1, 0), W.conv("pw52s2", 1, 52, 17, 36, 1, 2, 0),
               W.conv("f5c20", 1, 20, 13, 24, 5, 1, 2), W.conv("f7c12s2", 1, 12, 21, 20, 7, 2, 3)]


@pytest.mark.parametrize("op", STAGING_OPS, ids=lambda o: o.name)
def test_direct_staging_paths_match_oracle(op):
    # every way the direct family reads its operands: registers with vector or scalar
    # filter loads; LDS chunks staged through registers by each loop length, copied by a
    # plan, by 16 bytes without one or word by word, plane by plane or flat (a last chunk
    # shorter than CT where C is not a multiple of it, split channel ranges). The copies by
    # 16 bytes need w at a 16-byte address: those schedules run with w one float off as
    # well, where its copies go word by word
    x, w = make_inputs(op, "uniform", seed=31)
    ref, a = reference(op, x, w)
    xd, wd, yd = to_device(op, x, w)
    w_off = torch.empty(wd.numel() + 1, dtype=wd.dtype, device=wd.device)
    w_off[1:] = wd.reshape(-1)
    w_off = w_off[1:].reshape(wd.shape)
    by = {}
    for s in L.ct_valid_space(op):
        if s.family == W.FAM_DIRECT_F32:
            by.setdefault(_direct_class(op, s), []).append(s)
    rng = random.Random(5)
    ragged = off = 0
    for cls in sorted(by):
        pool = by[cls]
        # schedules whose channel chunks do not divide C, and split ones, among them
        pick = rng.sample(pool, min(2, len(pool)))
        odd = [s for s in pool if op.c % s.knob[DP.CT] and s not in pick]
        spl = [s for s in pool if s.knob[DP.SPLIT] > 1 and s not in pick]
        pick += rng.sample(odd, min(2, len(odd))) + rng.sample(spl, min(1, len(spl)))
        aligned_copies = "plan" in cls or "deep" in cls
        for s in pick:
            for wt in (wd, w_off) if aligned_copies else (wd,):
                tag = "%s %s [%s%s]" % (op.name, sched_str(s), cls, ", w off" if wt is w_off else "")
                note(tag)
                yd.fill_(float("nan"))
                L.conv2d_run(op, s, xd, wt, yd)
                check_close(op, yd.cpu().numpy(), ref, a, tag, split=4 if W.split_of(s) > 1 else 1)
                off += wt is w_off
            ragged += bool(op.c % s.knob[DP.CT])
    ways = {" ".join(c.split()[3:]) for c in by if c.startswith("lds")}
    print(op.name, "paths:", sorted(by), "ragged chunks:", ragged, "with w off:", off)
    if op.name == "deep3x3":
        assert {"regs spec 3", "regs spec 3 scalar-w", "lds spec 3 plan"} <= set(by)
        assert {"staged-%d" % n for n in (2, 4, 6, 8, 12, 16, 24)} <= ways and ragged > 0
        assert {"deep %d %d 1" % (i, j) for i in (0, 1) for j in (0, 1)} <= ways and off > 10
        assert {"copied 0 1", "copied 1 1"} <= ways
    if op.name == "pw52s2":  # slices that do not fill the rows of threads they take
        assert {"deep 0 0 0", "deep 1 0 0", "copied 1 0"} <= ways and off > 10


# Degenerate shapes: a one-pixel image (only the centre tap of a padded 3x3
# filter sees data), a filter as large as the image (one output pixel),
# one input and one output channel, a stride larger than the filter, a batch
# of three, and a one-row bf16 image.
DEGENERATE_OPS = [
    W.conv("one_pixel", 1, 8, 1, 8, 3, 1),
    W.Op("filter_covers_image", 1, 5, 7, 7, 6, 7, 7, 1, 1, 0, 0, 1, 1, 1, 0, 0),
    W.conv("one_channel", 2, 1, 9, 1, 3, 1),
    W.conv("stride3_1x1", 1, 12, 10, 8, 1, 3, 0),
    W.conv("batch3", 3, 16, 6, 16, 3, 1),
    W.Op("pwbf_one_row", 2, 16, 1, 9, 24, 1, 1, 1, 1, 0, 0, 1, 1, 1, W.DT_BF16, W.LAYOUT_NHWC),
]


@pytest.mark.parametrize("op", DEGENERATE_OPS, ids=lambda o: o.name)
def test_degenerate_shapes_match_oracle(op):
    fams = _run_sample(op, 12, seed=11)
    assert fams, op.name
    # every family that has a schedule for the shape, including the MFMA ones
    space_fams = {s.family for s in L.ct_valid_space(op)}
    for fam in sorted(space_fams - fams):
        _run_sample(op, 4, seed=12, family=fam)


@pytest.mark.parametrize("op", DEGENERATE_OPS, ids=lambda o: o.name)
def test_degenerate_shapes_bit_exact_on_integers(op):
    bf16 = op.dtype == W.DT_BF16
    _run_sample(op, 8, seed=13, dist="int", int_range=8 if bf16 else 2, exact=True)
