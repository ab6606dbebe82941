"""The alignment workloads whose speed is tracked, over the sizes users bring.

Each case is one call (or, for the per-step path, one sequence of calls) of the
public Python entry points on images that are already in device memory.  The
images are synthetic exposures of Gaussian-blob scenes with sensor noise, two
stops apart for pairs and one stop apart for stacks, translated by integer
shifts within the search's reach, as in the repository's own workloads.

`listed()` gives the fixed cases, `draw(rng)` one more of the same ranges,
`prepare` a case's inputs and kept buffers, `run` one pass, `work` the bytes and
operations a pass cannot do without, `exact` the results by plain integer torch
operations that share nothing with the library.
"""

import math

import numpy as np
import torch

import paper_2007_06483_amd as mtb

EXCLUDE = 4          # half-width of the excluded band around the median
SERVED_WIDTH = 8704  # row length of the resident frames that served requests are cut from


def listed():
    return [
        # The smallest call: one thumbnail pair, a few launches' latency.
        {"name": "pair_512x384", "kind": "stack", "n": 2, "width": 512, "height": 384, "levels": 5,
         "crop": False, "trace": False},
        # An ordinary camera pair, 12.6 MP each.
        {"name": "pair_4096x3072", "kind": "stack", "n": 2, "width": 4096, "height": 3072, "levels": 6,
         "crop": False, "trace": False},
        # The repository's headline: a seven-exposure bracket at 24 MP.
        {"name": "stack7_6000x4000", "kind": "stack", "n": 7, "width": 6000, "height": 4000, "levels": 7,
         "crop": False, "trace": False},
        # A served request of middling size: views into resident frames at odd columns.
        {"name": "served5_2449x1633", "kind": "stack", "n": 5, "width": 2449, "height": 1633, "levels": 6,
         "crop": True, "trace": False},
        # The largest served request: nine exposures of 48 MP, again views.
        {"name": "served9_8485x5657", "kind": "stack", "n": 9, "width": 8485, "height": 5657, "levels": 7,
         "crop": True, "trace": False},
        # The chained mode with its trace, on packed images of odd size.
        {"name": "chained7_3001x1999", "kind": "chained", "n": 7, "width": 3001, "height": 1999, "levels": 6,
         "crop": False, "trace": True},
        # The per-step path of a caller that keeps pyramids and bitmaps (video size).
        {"name": "steps_1920x1080", "kind": "steps", "n": 2, "width": 1920, "height": 1080, "levels": 6,
         "crop": False, "trace": True},
        # An offline batch of pairs of uneven sizes (the repository's four size classes).
        {"name": "batch16_uneven", "kind": "batch", "crop": False,
         "items": "640x480x5:4 1920x1080x6:4 4000x3000x7:4 6000x4000x7:4"},
        # A batch of small exposure stacks, odd sizes, cut from larger frames.
        {"name": "stacks8_small", "kind": "stacks", "crop": True,
         "items": "1225x817x5:3 1225x817x5:5 1000x667x5:4 1731x1154x6:7 1000x667x5:9 1731x1154x6:3 1100x733x5:5 "
                  "1225x817x5:9"},
        # Writing the aligned images of the headline stack.
        {"name": "apply7_6000x4000", "kind": "apply", "n": 7, "width": 6000, "height": 4000, "crop": False,
         "edge": False},
        # The same on packed images of odd size (rows at every alignment), edge fill.
        {"name": "apply5_3001x1999", "kind": "apply", "n": 5, "width": 3001, "height": 1999, "crop": False,
         "edge": True},
        # The rotation check of one 24 MP pair: four quadrant pairs.
        {"name": "quadrants_6000x4000", "kind": "quadrants", "n": 2, "width": 6000, "height": 4000, "levels": 7,
         "crop": False},
    ]


def _levels(width, height):
    """Levels of a served request: a coarsest level of at least 32 rows, at most seven."""
    m, levels = min(width, height), 1
    while levels < 7 and (32 << levels) <= m:
        levels += 1
    return levels


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_size(rng, lo_mp, hi_mp):
    """An image size of lo_mp .. hi_mp megapixels; half of them multiples of 16, half odd."""
    aspect = rng.choice([1.0, 4 / 3, 1.5, 16 / 9])
    mp = _log_uniform(rng, lo_mp, hi_mp)
    width = int(round(math.sqrt(mp * 1e6 * aspect)))
    height = int(round(width / aspect))
    if rng.random() < 0.5:
        width, height = max(16, width // 16 * 16), max(16, height // 16 * 16)
    else:
        width, height = width | 1, height | 1
    return width, height


def draw(rng):
    kind = rng.choice(["stack", "stack", "stack", "chained", "steps", "batch", "stacks", "apply", "quadrants"])
    if kind in ("stack", "chained"):
        n = rng.randint(2, 9)
        w, h = _draw_size(rng, 0.2, 40.0)
        return {"kind": kind, "n": n, "width": w, "height": h, "levels": _levels(w, h),
                "crop": rng.random() < 0.5, "trace": rng.random() < 0.3}
    if kind == "steps":
        w, h = _draw_size(rng, 0.2, 24.0)
        return {"kind": kind, "n": 2, "width": w, "height": h, "levels": _levels(w, h),
                "crop": rng.random() < 0.5, "trace": True}
    if kind in ("batch", "stacks"):
        items = []
        for _ in range(rng.randint(2, 6)):
            w, h = _draw_size(rng, 0.2, 12.0 if kind == "batch" else 4.0)
            items.append(f"{w}x{h}x{_levels(w, h)}:{rng.randint(1, 4) if kind == 'batch' else rng.randint(2, 9)}")
        return {"kind": kind, "crop": rng.random() < 0.5, "items": " ".join(items)}
    if kind == "apply":
        w, h = _draw_size(rng, 0.2, 24.0)
        return {"kind": kind, "n": rng.randint(2, 9), "width": w, "height": h, "crop": rng.random() < 0.5,
                "edge": rng.random() < 0.5}
    w, h = _draw_size(rng, 1.0, 24.0)
    return {"kind": kind, "n": 2, "width": w, "height": h, "levels": _levels(w // 2, h // 2),
            "crop": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs

def _radiance(width, height, rng, gen):
    """float32 radiance (3, height, width): Gaussian blobs plus noise of sd 0.01."""
    rad = torch.empty((3, height, width), dtype=torch.float32, device="cuda")
    rad.normal_(0.0, 0.01, generator=gen)
    blobs = 400 if width * height >= 1_000_000 else 40
    for cx, cy, s, a in zip(rng.uniform(0, width, blobs), rng.uniform(0, height, blobs), rng.uniform(5, 60, blobs),
                            rng.uniform(0.1, 1.0, (blobs, 3))):
        x0, x1 = max(0, math.ceil(cx - 4 * s)), min(width - 1, math.floor(cx + 4 * s))
        y0, y1 = max(0, math.ceil(cy - 4 * s)), min(height - 1, math.floor(cy + 4 * s))
        if x0 > x1 or y0 > y1:
            continue
        gx = np.exp(-((np.arange(x0, x1 + 1) - cx) ** 2) / (2 * s * s))
        gy = np.exp(-((np.arange(y0, y1 + 1) - cy) ** 2) / (2 * s * s))
        g = torch.from_numpy(np.concatenate([gx, gy, a]).astype(np.float32)).cuda()
        gx, gy, a = g[:gx.size], g[gx.size:gx.size + gy.size], g[gx.size + gy.size:]
        rad[:, y0:y1 + 1, x0:x1 + 1] += a[:, None, None] * (gy[:, None] * gx[None, :])
    return rad


def _gain(rad, evs):
    """Gain at which about five per cent of the pixels pooled over the exposures saturate."""
    peak = rad[:, ::8, ::8].amax(0).flatten()
    pooled = torch.cat([peak * 2.0 ** e for e in evs])
    return (1.0 / torch.kthvalue(pooled, max(1, int(0.95 * pooled.numel()))).values.clamp_min(1e-3)).item()


def _expose(rad, scale):
    """8-bit gamma-1/2.2 image (height, width, 3) of the radiance at the given scale."""
    out = torch.empty((rad.shape[1], rad.shape[2], 3), dtype=torch.uint8, device="cuda")
    for c in range(3):
        out[:, :, c] = ((rad[c] * scale).clamp_(0.0, 1.0).pow_(1 / 2.2).mul_(255.0).add_(0.5)).to(torch.uint8)
    return out


def _stack(seed, n, width, height, levels, crop):
    """n exposures of one scene; image n // 2 is the unshifted reference, the others
    are translated by up to 2^(levels-1) pixels per axis.  With `crop` they are
    views at odd columns of wider frames, otherwise packed images."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 62)))
    reach = 1 << (levels - 1)
    margin = reach + 1
    frame_w = width + 2 * margin
    if crop:
        frame_w = SERVED_WIDTH if frame_w <= SERVED_WIDTH and width > 2000 else (frame_w + 63) // 64 * 64
    frame_h = height + 2 * margin
    rad = _radiance(frame_w, frame_h, rng, gen)
    evs = [0.0, -2.0] if n == 2 else [float(i - n // 2) for i in range(n)]
    gain = 1.0 if n == 2 else _gain(rad, evs)
    ref = 0 if n == 2 else n // 2
    x0 = int(rng.integers(margin, frame_w - width - margin + 1)) | 1 if crop else margin
    x0 = min(x0, frame_w - width - reach)
    images = []
    for i in range(n):
        tx, ty = (0, 0) if i == ref else (int(v) for v in rng.integers(-reach, reach + 1, 2))
        frame = _expose(rad, gain * 2.0 ** evs[i])
        view = frame[margin + ty:margin + ty + height, x0 + tx:x0 + tx + width]
        images.append(view if crop else view.contiguous())
    return images


def _items(case):
    """[(width, height, levels, count), ...] of a batch case."""
    out = []
    for word in case["items"].split():
        size, count = word.split(":")
        w, h, levels = (int(v) for v in size.split("x"))
        out.append((w, h, levels, int(count)))
    return out


def _ref_index(n):
    return 0 if n == 2 else n // 2


def _batch_inputs(case, seed):
    """Pairs [(ref, mov, levels), ...] or stacks [(images, levels), ...] of a batch case."""
    out = []
    for k, (w, h, levels, count) in enumerate(_items(case)):
        if case["kind"] == "stacks":
            out.append((_stack(seed * 64 + k, count, w, h, levels, case["crop"]), levels, _ref_index(count)))
            continue
        for j in range(count):
            ref, mov = _stack(seed * 1024 + 16 * k + j, 2, w, h, levels, case["crop"])
            out.append((ref, mov, levels))
    return out


def _apply_shifts(seed, n):
    rng = np.random.default_rng(seed + 7)
    sh = rng.integers(-100, 101, (n, 2)).astype(np.int32)
    sh[n // 2] = 0
    return torch.from_numpy(sh)


def _level_views(layout, pyramid, bitmaps):
    """Every defined part of one image's two buffers: gray, T and E per level, histograms, medians."""
    views = {}
    for l in range(layout.levels):
        w, h, wpr = layout.level_width[l], layout.level_height[l], layout.words_per_row[l]
        pitch = layout.gray_pitch[l]
        off = layout.gray_offset[l]
        views[f"gray{l}"] = pyramid[off:off + pitch * h].view(h, pitch)[:, :w]
        for name, o in (("t", layout.tb_offset[l]), ("e", layout.eb_offset[l])):
            views[f"{name}{l}"] = bitmaps[o:o + 8 * wpr * h].view(h, 8 * wpr)
    o = layout.hist_offset
    views["hist"] = pyramid[o:o + 1024 * layout.levels].view(torch.int32).view(layout.levels, 256)
    o = layout.median_offset
    views["median"] = bitmaps[o:o + 4 * layout.levels].view(torch.int32)
    return views


def prepare(case, seed):
    kind = case["kind"]
    dev = "cuda"
    state = {"case": case}
    if kind in ("batch", "stacks"):
        items = _batch_inputs(case, seed)
        if kind == "batch":
            need, rows = mtb.mtb_batch_workspace_bytes(items), len(items)
        else:
            need, rows = mtb.mtb_batch_stacks_workspace_bytes(items), sum(len(it[0]) for it in items)
        state.update(items=items, workspace=torch.empty(need, dtype=torch.uint8, device=dev),
                     shifts=torch.empty((rows, 2), dtype=torch.int32, device=dev),
                     errs=torch.empty(rows, dtype=torch.int32, device=dev))
        return state
    n, w, h = case["n"], case["width"], case["height"]
    levels = case.get("levels", 7)
    images = _stack(seed, n, w, h, min(levels, mtb.mtb_max_levels(w, h)), case["crop"])
    state["images"] = images
    if kind == "apply":
        state["shifts"] = _apply_shifts(seed, n).to(dev)
        state["out"] = [torch.empty((h, w, 3), dtype=torch.uint8, device=dev) for _ in range(n)]
    elif kind == "steps":
        layout = mtb.mtb_get_layout(w, h, levels)
        state["pyr"] = [torch.empty(layout.pyramid_bytes, dtype=torch.uint8, device=dev) for _ in images]
        state["bm"] = [torch.empty(layout.bitmaps_bytes, dtype=torch.uint8, device=dev) for _ in images]
        state["workspace"] = torch.empty(mtb.mtb_pair_workspace_bytes(levels), dtype=torch.uint8, device=dev)
        state["views"] = [_level_views(layout, p, b) for p, b in zip(state["pyr"], state["bm"])]
        state["shift"] = torch.empty(2, dtype=torch.int32, device=dev)
        state["err"] = torch.empty(1, dtype=torch.int32, device=dev)
    elif kind == "quadrants":
        need = mtb.mtb_quadrant_workspace_bytes(w, h, images[0].stride(0), levels)
        state["workspace"] = torch.empty(need, dtype=torch.uint8, device=dev)
    else:
        need = mtb.mtb_stack_workspace_bytes(n, w, h, levels)
        state.update(workspace=torch.empty(need, dtype=torch.uint8, device=dev),
                     shifts=torch.empty((n, 2), dtype=torch.int32, device=dev),
                     errs=torch.empty(n, dtype=torch.int32, device=dev))
    return state


# ------------------------------------------------------------------ one pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("stack", "chained"):
        call = mtb.mtb_align_stack if kind == "stack" else mtb.mtb_align_stack_chained
        r = call(state["images"], case["levels"], EXCLUDE, _ref_index(case["n"]), workspace=state["workspace"],
                 trace=case["trace"], shifts=state["shifts"], errs=state["errs"])
        out = {"shifts": r["shifts"], "errs": r["errs"]}
        if case["trace"]:
            out["trace"] = r["trace"]
        return out
    if kind == "steps":
        w, h, levels = case["width"], case["height"], case["levels"]
        for im, p, b in zip(state["images"], state["pyr"], state["bm"]):
            mtb.mtb_build_pyramid(im, levels, pyramid=p)
            mtb.mtb_bitmaps(p, w, h, levels, EXCLUDE, bitmaps=b)
        r = mtb.mtb_align_pair(state["bm"][0], state["bm"][1], w, h, levels, workspace=state["workspace"], trace=True,
                               level_shifts=True, shift=state["shift"], err=state["err"])
        return {"images": state["views"], "shift": r["shift"], "err": r["err"], "trace": r["trace"],
                "level_shifts": r["level_shifts"]}
    if kind in ("batch", "stacks"):
        call = mtb.mtb_align_batch if kind == "batch" else mtb.mtb_align_batch_stacks
        r = call(state["items"], EXCLUDE, workspace=state["workspace"], shifts=state["shifts"], errs=state["errs"])
        return {"shifts": r["shifts"], "errs": r["errs"]}
    if kind == "apply":
        return mtb.mtb_apply_shifts(state["images"], state["shifts"],
                                    mtb.MTB_FILL_EDGE if case["edge"] else mtb.MTB_FILL_ZERO, out=state["out"])
    ref, mov = state["images"]
    return mtb.mtb_align_quadrants(ref, mov, case["levels"], EXCLUDE, 1, workspace=state["workspace"])


# ------------------------------------------------------------------ what a pass cannot do without

def _stack_work(n, pairs, w, h, levels):
    """Every image's RGB read once, the results written; operations of the method's steps."""
    px = sum((w >> l) * (h >> l) for l in range(levels))
    # gray 6 per pixel, 4 per coarser pixel, histogram 1, two bit tests 3; 9 candidates of 4 per 64-pixel word
    ops = n * (6 * w * h + 4 * (px - w * h) + 4 * px) + pairs * 9 * 4 * px / 64
    return 3 * w * h * n + 12 * n, ops


def work(case):
    kind = case["kind"]
    if kind in ("batch", "stacks"):
        nbytes = flops = 0
        for w, h, levels, count in _items(case):
            n, pairs = (2 * count, count) if kind == "batch" else (count, count - 1)
            b, f = _stack_work(n, pairs, w, h, levels)
            nbytes, flops = nbytes + b, flops + f
        return {"bytes": nbytes, "flops": flops}
    n, w, h = case["n"], case["width"], case["height"]
    if kind == "apply":
        return {"bytes": 6 * w * h * n, "flops": 0}
    nbytes, flops = _stack_work(n, n - 1, w, h, case["levels"])
    if kind == "steps":
        # The steps' own results are outputs here: gray and bitmaps written, then read by the next step.
        px = sum((w >> l) * (h >> l) for l in range(case["levels"]))
        nbytes += n * (2 * px + 2 * 2 * px // 8)
    elif case.get("trace"):
        nbytes += 36 * n * case["levels"]
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ results by plain integer torch

def _exact_maps(img, levels):
    """Per level: gray, histogram, median, T and E of one image."""
    out = []
    rgb = img.to(torch.int64)
    g = (54 * rgb[..., 0] + 183 * rgb[..., 1] + 19 * rgb[..., 2]) >> 8
    del rgb
    for l in range(levels):
        if l:
            h, w = g.shape[0] // 2 * 2, g.shape[1] // 2 * 2
            g = g[:h, :w]
            g = (g[0::2, 0::2] + g[0::2, 1::2] + g[1::2, 0::2] + g[1::2, 1::2]) >> 2
        hist = torch.stack([(g == v).sum() for v in range(256)])
        need = (g.numel() + 1) // 2
        m = int((hist.cumsum(0) < need).sum())
        out.append({"gray": g.to(torch.uint8), "hist": hist, "median": m, "t": g > m, "e": (g - m).abs() > EXCLUDE})
    return out


def _exact_error(ref, mov, cx, cy):
    """#{(T_ref ^ S T_mov) & E_ref & S E_mov} for the shift (cx, cy)."""
    h, w = ref["t"].shape
    ys, ye, xs, xe = max(0, cy), min(h, h + cy), max(0, cx), min(w, w + cx)
    if ys >= ye or xs >= xe:
        return 0
    r, s = (slice(ys, ye), slice(xs, xe)), (slice(ys - cy, ye - cy), slice(xs - cx, xe - cx))
    return int(((ref["t"][r] ^ mov["t"][s]) & ref["e"][r] & mov["e"][s]).sum())


def _exact_pair(ref, mov, levels):
    """(shift, error, trace[levels][9], level shifts) of the coarse-to-fine search."""
    trace, shifts = [None] * levels, [None] * levels
    bx = by = err = 0
    for l in range(levels - 1, -1, -1):
        c = [_exact_error(ref[l], mov[l], bx + dx, by + dy) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
        best = c.index(min(c))
        sx, sy = bx + best % 3 - 1, by + best // 3 - 1
        trace[l], shifts[l], err = c, (sx, sy), c[best]
        bx, by = 2 * sx, 2 * sy
    return shifts[0], err, trace, shifts


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _exact_stack(images, levels, ref, chained=False):
    n = len(images)
    shifts, errs = [(0, 0)] * n, [0] * n
    traces = [[[0] * 9 for _ in range(levels)] for _ in range(n)]
    order = list(range(ref - 1, -1, -1)) + list(range(ref + 1, n))
    base = _exact_maps(images[ref], levels)
    near = base
    for i in order:
        if chained and i == ref + 1:
            near = base
        maps = _exact_maps(images[i], levels)
        s, errs[i], traces[i], _ = _exact_pair(near if chained else base, maps, levels)
        if chained:
            prev = shifts[i + 1] if i < ref else shifts[i - 1]
            s = (s[0] + prev[0], s[1] + prev[1])
            near = maps
        shifts[i] = s
    return shifts, errs, traces


def _packed(bits, words):
    """Rows of bits packed least significant first into 8 * words bytes."""
    h, w = bits.shape
    p = torch.zeros((h, 64 * words), dtype=torch.int64, device=bits.device)
    p[:, :w] = bits
    return (p.view(h, 8 * words, 8) << torch.arange(8, device=bits.device)).sum(-1).to(torch.uint8)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "stacks"):
        shifts, errs = [], []
        for it in _batch_inputs(case, seed):
            images, levels, ref = ([it[0], it[1]], it[2], 0) if kind == "batch" else it
            s, e, _ = _exact_stack(images, levels, ref)
            shifts += s[1:] if kind == "batch" else s
            errs += e[1:] if kind == "batch" else e
        return {"shifts": _i32(shifts), "errs": _i32(errs)}
    n, w, h = case["n"], case["width"], case["height"]
    levels = case.get("levels", 7)
    images = _stack(seed, n, w, h, min(levels, mtb.mtb_max_levels(w, h)), case["crop"])
    if kind in ("stack", "chained"):
        s, e, t = _exact_stack(images, levels, _ref_index(n), kind == "chained")
        out = {"shifts": _i32(s), "errs": _i32(e)}
        if case["trace"]:
            out["trace"] = _i32(t)
        return out
    if kind == "steps":
        maps = [_exact_maps(im, levels) for im in images]
        views = []
        for m in maps:
            v = {}
            for l in range(levels):
                words = 2 * ((m[l]["t"].shape[1] + 127) // 128)
                v[f"gray{l}"] = m[l]["gray"]
                v[f"t{l}"] = _packed(m[l]["t"], words)
                v[f"e{l}"] = _packed(m[l]["e"], words)
            v["hist"] = torch.stack([m[l]["hist"] for l in range(levels)]).to(torch.int32)
            v["median"] = _i32([m[l]["median"] for l in range(levels)])
            views.append(v)
        s, e, t, ls = _exact_pair(maps[0], maps[1], levels)
        return {"images": views, "shift": _i32(s), "err": _i32([e]), "trace": _i32(t), "level_shifts": _i32(ls)}
    if kind == "apply":
        out = []
        for im, (dx, dy) in zip(images, _apply_shifts(seed, n).tolist()):
            y = torch.arange(h, device="cuda") - dy
            x = torch.arange(w, device="cuda") - dx
            o = im[y.clamp(0, h - 1)][:, x.clamp(0, w - 1)]
            if not case["edge"]:
                o = o * ((y >= 0) & (y < h))[:, None, None] * ((x >= 0) & (x < w))[None, :, None]
            out.append(o)
        return out
    ref, mov = images
    w0, h0 = w // 2, h // 2
    shifts, errs = [], []
    for q in range(4):
        part = (slice(h0, h) if q & 2 else slice(0, h0), slice(w0, w) if q & 1 else slice(0, w0))
        s, e, _, _ = _exact_pair(_exact_maps(ref[part], levels), _exact_maps(mov[part], levels), levels)
        shifts.append(s)
        errs.append(e)
    flag = any(abs(a[c] - b[c]) > 1 for a in shifts for b in shifts for c in (0, 1))
    return {"shifts": _i32(shifts), "errs": _i32(errs), "flag": _i32([int(flag)])}
