"""Edges of the kernels' tiles, lanes and dispatch rules against the oracle, bit for bit.

Everything compared is a whole number or a byte, so the tolerance is zero.
"""

import numpy as np
import pytest

import oracle
import synth
from mtb_decode import bitmaps, gray_levels, histograms, medians, stack_workspace

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


@pytest.fixture(scope="module")
def mtb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2007_06483_amd as m

    m.lib()
    return m


def _view(img, extra, offset):
    """Device view of img whose rows are 3W + extra bytes apart, starting offset bytes in."""
    h, w, _ = img.shape
    stride = 3 * w + extra
    buf = np.full(offset + stride * h, 201, np.uint8)
    rows = buf[offset:].reshape(h, stride)
    rows[:, :3 * w] = img.reshape(h, 3 * w)
    return torch.as_strided(torch.from_numpy(buf).to(DEV), (h, w, 3), (stride, 3, 1), offset)


def _check_pyramid(mtb, d_img, img, L):
    h, w, _ = img.shape
    lay = mtb.mtb_get_layout(w, h, L)
    pyr = mtb.mtb_build_pyramid(d_img, L)
    bm = mtb.mtb_bitmaps(pyr, w, h, L)
    torch.cuda.synchronize()
    pyr_h, bm_h = pyr.cpu().numpy(), bm.cpu().numpy()
    want = oracle.pyramid(img, L)
    for l, g in enumerate(gray_levels(pyr_h, lay)):
        assert np.array_equal(g, want.gray(l)), f"gray level {l}"
    assert np.array_equal(histograms(pyr_h, lay), want.hist)
    assert np.array_equal(medians(bm_h, lay), want.median)
    for l, (t, e, tp, ep) in enumerate(bitmaps(bm_h, lay)):
        assert np.array_equal(t, want.tb(l)) and np.array_equal(e, want.eb(l)), f"bitmaps level {l}"
        assert not tp.any() and not ep.any(), f"padding bits set at level {l}"


# A lane takes 16 pixels of a row: widths around its multiples, and the widths
# at which the last lane holds 1, 2 or 3 pixels (3 to 9 bytes).
@pytest.mark.parametrize("w", [1, 2, 3, 4, 5, 15, 16, 17, 18, 21, 31, 33, 255, 257, 262, 271])
@pytest.mark.parametrize("extra,offset", [(0, 0), (1, 0), (0, 1), (3, 2), (16, 15)])
def test_pyramid_row_ends_at_every_alignment(mtb, w, extra, offset):
    img = np.random.default_rng(1000 * w + 10 * extra + offset).integers(0, 256, (67, w, 3), dtype=np.uint8)
    L = min(7, mtb.mtb_max_levels(w, 67))
    _check_pyramid(mtb, _view(img, extra, offset), img, L)


# k_apply writes 16-byte chunks at aligned output addresses in runs of whole
# wavefronts: rows around a chunk (5, 6 pixels), around 1, 4 and 5 KiB, and
# shifts that leave no, some and every source column inside, with input and
# output rows at every kind of alignment.
@pytest.mark.parametrize("w", [1, 5, 6, 11, 341, 342, 1365, 1706, 1707, 1712])
@pytest.mark.parametrize("extra,offset,out_extra,out_offset", [(0, 0, 0, 0), (1, 3, 0, 5), (4, 4, 7, 0), (16, 1, 13, 2)])
def test_apply_rows_at_every_alignment(mtb, w, extra, offset, out_extra, out_offset):
    h = 9
    rng = np.random.default_rng(w * 100 + extra)
    imgs = [rng.integers(0, 256, (h, w, 3), dtype=np.uint8) for _ in range(6)]
    shifts = [(0, 0), (1, -1), (-w, 0), (w - 1, 8), (-5, -9), (2, 2)]
    sh = torch.tensor(shifts, dtype=torch.int32, device=DEV)
    for fill in (mtb.MTB_FILL_ZERO, mtb.MTB_FILL_EDGE):
        d = [_view(im, extra, offset) for im in imgs]
        outs = [_view(np.zeros_like(im), out_extra, out_offset) for im in imgs]
        mtb.mtb_apply_shifts(d, sh, fill, out=outs)
        torch.cuda.synchronize()
        for im, o, (dx, dy) in zip(imgs, outs, shifts):
            assert np.array_equal(o.cpu().numpy(), oracle.apply_shift(im, dx, dy, fill)), (fill, dx, dy)
            if out_extra:  # row padding stays as it was
                pad = o.as_strided((h - 1, out_extra), (o.stride(0), 1), o.storage_offset() + 3 * w)
                assert (pad == 201).all()


# Beyond two tiles a workgroup, k_pyramid's workgroups claim tiles (in groups of
# 1, 2 or 4 by launch shape, or 2 by rule between one and two tiles a slot); every
# tile must be counted exactly once, merged
# histograms or not, also where every pixel falls into one bin.
@pytest.mark.parametrize("n,w,h,pct,group", [(3, 4096, 3072, 25, 4), (3, 4096, 3072, 25, 2), (3, 4096, 3072, 25, 1),
                                             (2, 4001, 3003, 25, 1), (1, 6000, 4200, 100, 1), (5, 3000, 2000, 50, 2),
                                             (3, 3000, 2000, 100, 1), (5, 2449, 1633, 100, 1), (4, 2560, 1440, 50, 1)])
def test_pyramid_claimed_tiles(mtb, n, w, h, pct, group):
    L = 7
    rng = np.random.default_rng(w + n)
    imgs = [rng.integers(0, 256, (h, w, 3), dtype=np.uint8)]
    imgs += [np.full((h, w, 3), 255, np.uint8), imgs[0] // 32, imgs[0] // 2, imgs[0]][:n - 1]
    stride = 3 * w
    mtb.mtb_set_shape(n, w, h, stride, L, {"pyramid_slots_pct": pct, "pyramid_tile_group": group})
    try:
        d = [_view(im, 0, 0) for im in imgs]
        lay = mtb.mtb_get_layout(w, h, L)
        for _ in range(3):  # the claims start from zero on every call
            got = mtb.mtb_align_stack(d, L)
            torch.cuda.synchronize()
            pyrs, bms = stack_workspace(mtb, got["workspace"], n, lay)
            for im, p, b in zip(imgs, pyrs, bms):
                want = oracle.pyramid(im, L)
                assert np.array_equal(histograms(p, lay), want.hist)
                assert np.array_equal(medians(b, lay), want.median)
                for l, g in enumerate(gray_levels(p, lay)):
                    assert np.array_equal(g, want.gray(l)), f"gray level {l}"
    finally:
        mtb.mtb_tune_reset()


# A fine level is searched one word a lane, 1, 2 or 4 rows each, while that
# takes at most one workgroup a compute unit (65536 lanes), else in row
# streams: sizes whose levels 0 to 2 fall on every side of those limits, rows
# of 1 to 40 words, heights that are no multiple of the rows, many pairs, and
# shifts that move words across the row's ends; rows of 134 two-word columns take
# streams that pad them by a fifth.
@pytest.mark.parametrize("n,w,h,L", [(2, 1300, 1250, 5), (2, 2000, 1030, 6), (2, 2049, 2051, 6), (3, 700, 2901, 6),
                                     (9, 640, 403, 5), (5, 1111, 777, 6), (2, 129, 4000, 5), (32, 300, 331, 4),
                                     (5, 8485, 300, 4)])
def test_fine_levels_one_word_a_lane(mtb, n, w, h, L):
    imgs, _, _ = synth.make_stack(w, h, n, 12, 500 + w + n, min(1 << (L - 1), min(w, h) // 4), sat_frac=0.05)
    d = [_view(im, 0, 0) for im in imgs]
    mtb.mtb_tune_reset()
    mtb.mtb_set_shape(n, w, h, 3 * w, L, {"small_search": 0, "coarse_levels": 0})
    try:
        alt = mtb.mtb_align_stack(d, L, trace=True)
    finally:
        mtb.mtb_tune_reset()
    got = mtb.mtb_align_stack(d, L, trace=True)
    torch.cuda.synchronize()
    want = oracle.align_stack(imgs, L, threads=4, keep=False)
    for r in (got, alt):
        assert np.array_equal(r["shifts"].cpu().numpy(), want["shifts"])
        assert np.array_equal(r["errs"].cpu().numpy().astype(np.int64), want["errs"])
        assert np.array_equal(r["trace"].cpu().numpy(), got["trace"].cpu().numpy())


# The quadrant flag and the chained sums are formed by the search's last
# workgroup where one launch sees every pair's level 0, else by a launch of
# their own: quadrants that share one launch set, that do not (odd sizes), and
# that one workgroup searches; stacks with all levels searched exhaustively.
@pytest.mark.parametrize("w,h,L,extra_shift", [(1600, 1200, 6, 0), (1600, 1200, 6, 9), (1601, 1203, 5, 9), (1600, 1201, 6, 0),
                                               (400, 300, 4, 9), (1600, 1200, 3, 9)])
def test_quadrant_flag_of_the_search(mtb, w, h, L, extra_shift):
    base = synth.expose(synth.rect_field(w, h, 60, np.random.default_rng(w + h + extra_shift)), 0.0)
    mov = synth.translate(base, 3, -2)
    mov[:h // 2, w // 2:] = synth.translate(base, 3 + extra_shift, -2)[:h // 2, w // 2:]
    for tol in (0, 1, 60):
        want = oracle.align_quadrants(base, mov, L, tolerance=tol)
        got = mtb.mtb_align_quadrants(_view(base, 0, 0), _view(mov, 0, 0), L, tolerance=tol)
        torch.cuda.synchronize()
        assert np.array_equal(got["shifts"].cpu().numpy(), want["shifts"])
        assert np.array_equal(got["errs"].cpu().numpy().astype(np.int64), want["errs"])
        assert int(got["flag"].cpu()[0]) == want["flag"]


@pytest.mark.parametrize("n,w,h,L", [(5, 640, 480, 3), (5, 640, 480, 2), (2, 900, 700, 5), (7, 901, 703, 6)])
@pytest.mark.parametrize("ref", [0, 1])
def test_chained_sums_of_the_search(mtb, n, w, h, L, ref):
    imgs, _, _ = synth.make_stack(w, h, n, 30, 800 + n + L, 5, sat_frac=0.05)
    want = oracle.align_stack_chained(imgs, L, ref_index=ref, threads=4)
    got = mtb.mtb_align_stack_chained([_view(im, 0, 0) for im in imgs], L, ref_index=ref)
    torch.cuda.synchronize()
    assert np.array_equal(got["shifts"].cpu().numpy(), want["shifts"])
    assert np.array_equal(got["errs"].cpu().numpy().astype(np.int64), want["errs"])


# The coarse levels are searched from the gray levels inside the bitmaps launch
# while their rows hold at most 64 words and their workgroups are few, else by
# a launch of their own: sizes on both sides, level widths that end inside a
# word (the gray behind them is whatever the workspace held), every number of
# coarse levels, one to many slabs.
@pytest.mark.parametrize("n,w,h,L,coarse", [(3, 1000, 700, 5, -1), (3, 1000, 700, 5, 1), (3, 1000, 700, 5, 2),
                                            (2, 1200, 3900, 6, -1), (2, 2301, 1700, 6, -1), (2, 3990, 531, 4, -1),
                                            (2, 9000, 90, 4, -1), (2, 2040, 1031, 4, 3), (32, 1200, 900, 6, -1),
                                            (32, 2000, 1500, 6, -1),
                                            (2, 700, 1500, 10, -1), (3, 1000, 700, 5, 4), (2, 640, 480, 3, -1)])
def test_coarse_levels_inside_the_bitmaps_launch(mtb, n, w, h, L, coarse):
    imgs, _, _ = synth.make_stack(w, h, n, 12, 300 + w + L, min(1 << (min(L, 6) - 1), h // 8), sat_frac=0.05)
    d = [_view(im, 0, 0) for im in imgs]
    ws = torch.full((mtb.mtb_stack_workspace_bytes(n, w, h, L),), 173, dtype=torch.uint8, device=DEV)
    mtb.mtb_tune_reset()
    if coarse >= 0:
        mtb.mtb_set_shape(n, w, h, 3 * w, L, {"coarse_levels": coarse, "small_search": 0})
    try:
        got = mtb.mtb_align_stack(d, L, workspace=ws, trace=True)
        mtb.mtb_set_shape(n, w, h, 3 * w, L, {"coarse_levels": 0, "small_search": 0})
        alt = mtb.mtb_align_stack(d, L, trace=True)
    finally:
        mtb.mtb_tune_reset()
    torch.cuda.synchronize()
    want = oracle.align_stack(imgs, L, threads=4, keep=False)
    assert np.array_equal(got["shifts"].cpu().numpy(), want["shifts"])
    assert np.array_equal(got["errs"].cpu().numpy().astype(np.int64), want["errs"])
    assert np.array_equal(got["trace"].cpu().numpy(), alt["trace"].cpu().numpy())


def _check_traces(got, imgs, L):
    want = oracle.align_stack(imgs, L, threads=4)
    assert np.array_equal(got["shifts"].cpu().numpy(), want["shifts"])
    assert np.array_equal(got["errs"].cpu().numpy().astype(np.int64), want["errs"])
    trace = got["trace"].cpu().numpy().astype(np.int64)
    for k, pair in want["pairs"].items():
        assert np.array_equal(trace[k], pair["trace"]), f"trace of image {k}"


# With few levels the coarse levels reach down to level 1, whose gray is not in
# the workspace where its bitmaps come from level 0: the workspace's old bytes
# must not be searched instead.
@pytest.mark.parametrize("n,w,h,L", [(2, 640, 480, 2), (2, 800, 600, 2), (2, 640, 480, 3), (2, 900, 700, 3),
                                     (2, 1024, 768, 3), (2, 1024, 768, 4), (2, 1100, 700, 4), (3, 1000, 700, 4),
                                     (3, 1000, 700, 5)])
@pytest.mark.parametrize("l1", [0, 1])
def test_coarse_levels_where_level_1_comes_from_level_0(mtb, n, w, h, L, l1):
    imgs, _, _ = synth.make_stack(w, h, n, 12, 900 + w + L, 1 << (L - 1), sat_frac=0.05)
    ws = torch.full((mtb.mtb_stack_workspace_bytes(n, w, h, L),), 173, dtype=torch.uint8, device=DEV)
    mtb.mtb_tune_reset()
    mtb.mtb_set_shape(n, w, h, 3 * w, L, {"small_search": 0, "level1_from_level0": l1})
    try:
        got = mtb.mtb_align_stack([_view(im, 0, 0) for im in imgs], L, workspace=ws, trace=True)
    finally:
        mtb.mtb_tune_reset()
    torch.cuda.synchronize()
    _check_traces(got, imgs, L)


# Rows whose bytes pass 2^31 and 2^32: every pixel's gray and both levels'
# histograms, against the same integers formed by torch.
@pytest.mark.parametrize("w,h,L", [(715_827_899, 2, 2), (800_000_003, 1, 1), (1_431_655_783, 1, 1), (2**31 - 200, 1, 1),
                                   (2**31 - 1, 1, 1)])
def test_pyramid_of_very_long_rows(mtb, w, h, L):
    torch.manual_seed(w)
    img = torch.randint(0, 256, (h, w, 3), dtype=torch.uint8, device=DEV)
    lay = mtb.mtb_get_layout(w, h, L)
    pyr = torch.full((mtb.mtb_pyramid_bytes(w, h, L),), 173, dtype=torch.uint8, device=DEV)
    mtb.mtb_build_pyramid(img, L, pyramid=pyr)
    weights = torch.tensor([54, 183, 19], dtype=torch.int32, device=DEV)
    hist = torch.zeros((L, 256), dtype=torch.int64, device=DEV)
    step = 1 << 25
    for x in range(0, w, step):
        gray = (img[:, x:x + step].to(torch.int32) * weights).sum(2, dtype=torch.int32) >> 8
        for l in range(L):
            if l:
                gray = gray[:, :gray.shape[1] // 2 * 2].reshape(gray.shape[0] // 2, 2, -1, 2).sum((1, 3)) >> 2
            p, x_l = lay.gray_pitch[l], x >> l
            for y in range(gray.shape[0]):
                o = lay.gray_offset[l] + y * p + x_l
                assert torch.equal(pyr[o:o + gray.shape[1]], gray[y].to(torch.uint8)), f"level {l} from column {x_l}"
            hist[l] += torch.bincount(gray.reshape(-1), minlength=256)
    got = pyr[lay.hist_offset:lay.hist_offset + 1024 * L].view(torch.int32).view(L, 256)
    assert torch.equal(got.to(torch.int64), hist)


# The same levels' traces (every candidate's error, not the winners' alone)
# against the oracle: by the built-in rule, and in row streams of given rows,
# which k_search_fine takes at every level.
@pytest.mark.parametrize("n,w,h,L", [(2, 1300, 1250, 5), (2, 2000, 1030, 6), (2, 2049, 2051, 6), (3, 700, 2901, 6),
                                     (9, 640, 403, 5), (5, 1111, 777, 6), (2, 129, 4000, 5), (32, 300, 331, 4),
                                     (5, 8485, 300, 4)])
@pytest.mark.parametrize("rows", [0, 4, 24])
@pytest.mark.parametrize("coarse", [-1, 0])
def test_fine_levels_traces(mtb, n, w, h, L, rows, coarse):
    imgs, _, _ = synth.make_stack(w, h, n, 12, 500 + w + n, min(1 << (L - 1), min(w, h) // 4), sat_frac=0.05)
    mtb.mtb_tune_reset()
    mtb.mtb_set_shape(n, w, h, 3 * w, L, {"small_search": 0, "coarse_levels": coarse, "search_rows": [rows] * 16})
    try:
        got = mtb.mtb_align_stack([_view(im, 0, 0) for im in imgs], L, trace=True)
    finally:
        mtb.mtb_tune_reset()
    torch.cuda.synchronize()
    _check_traces(got, imgs, L)
