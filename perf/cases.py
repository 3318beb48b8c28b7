"""Timed cases: what a program that removes objects from images has this library do.

Five kinds of work, each through the public binding or the serving loop:

  query     one exemplar search (findBestPatch) on a live context, with or without the
            allocation-free entry point: the smallest call there is
  removal   one whole removal from host buffers: context, fill loop, the image and the
            fill log back on the host
  resume    a checkpoint of a half-done removal imported, some iterations run, the new
            checkpoint exported (interactive editing)
  batch     several uneven images removed together by one kept Batch
  serve     the continuous-batching server on a queue of jobs of several patch sizes

Images and masks are drawn by the seeded generators of ``synth``; the sizes are those of
its workloads (128x96 to 2048x1536 pixels, patches of 5 to 17 pixels, holes of 1% to 10%).
"""
import math

import numpy as np

from paper_1403_4238_amd import binding as B
from paper_1403_4238_amd import serve, synth

PATHS = {"auto": B.PATH_AUTO, "simt": B.PATH_SIMT, "mfma": B.PATH_MFMA}
ALPHA_FULL = 0          # alpha_den of a full search
SERVE_BUDGET = 4 << 30  # device bytes the server may admit
LOG_WHOLE = ("target_index", "source_index", "ssd", "known_k", "n_filled", "remaining")
LOG_REAL = ("priority", "confidence", "data_term")


def _image(kind, name, width, height, patch, content, hole, blobs=1, **more):
    case = {"kind": kind, "name": name, "width": width, "height": height, "patch": patch, "content": content,
            "hole": hole, "blobs": blobs, "alpha_num": 0, "alpha_den": ALPHA_FULL, "path": "auto", "form": "plain",
            "check": 16, "current": False, "intersect": False}
    case.update(more)
    return case


def listed():
    return [
        # A single search on a live context made with the default parameters: what a
        # tool that proposes one patch per click waits for.
        _image("query", "query_vga_p9", 640, 480, 9, "noise", 0.08, targets=1, static=False),
        # A few searches with a large patch on a full-HD frame through the call that
        # allocates nothing, as a loop that may not allocate makes them.
        _image("query", "query_hd_p13_static", 1920, 1080, 13, "voronoi", 0.05, path="mfma", targets=4, static=True),
        # The first call of a new user: default parameters, a thumbnail.  Context
        # creation, launches and host checks count here.
        _image("removal", "removal_small_default", 128, 96, 9, "gradient", 0.031),
        # The same defaults on a VGA image.
        _image("removal", "removal_vga_default", 640, 480, 9, "noise", 0.08),
        # A portrait photograph of the paper's River size, its largest patch, a search
        # window around the object: the size where the matrix path is not offered.
        _image("removal", "removal_portrait_p17_window", 480, 639, 17, "noise", 0.018, alpha_num=1, alpha_den=2,
               form="persistent", check=1024),
        # The headline removal: full HD, 9x9 patch, full search, the fastest form.
        _image("removal", "removal_hd_p9", 1920, 1080, 9, "voronoi", 0.05, path="mfma", form="persistent", check=1024),
        # The same frame with the paper's larger patch and its alpha = 1 window.
        _image("removal", "removal_hd_p13_window", 1920, 1080, 13, "voronoi", 0.05, alpha_num=1, alpha_den=1,
               path="mfma", form="persistent", check=1024),
        # More search tiles than work-groups fit on the device: a large serving job alone.
        _image("removal", "removal_big_p7", 1992, 1221, 7, "voronoi", 0.03, blobs=2, path="mfma", form="persistent",
               check=1024),
        # The paper's literal reading of its domain: filled pixels become sources and
        # overlapping candidates are scored on the intersection.
        _image("removal", "domains_vga_p9", 640, 480, 9, "noise", 0.08, form="stream", check=128, current=True,
               intersect=True),
        # Interactive editing: a checkpoint in, 256 iterations, the next checkpoint out.
        _image("resume", "resume_hd_p9", 1920, 1080, 9, "voronoi", 0.05, path="mfma", form="persistent", check=1024,
               before=1500, iterations=256),
        # A folder of uneven images in one kept batch.
        {"kind": "batch", "name": "batch_12_uneven", "images": 12, "patch": 9, "max_width": 1280, "max_height": 720,
         "graph_iters": 64},
        # The server, saturated: jobs of three patch sizes waiting when it starts.
        {"kind": "serve", "name": "serve_8_mixed", "images": 8, "max_width": 1600, "max_height": 1200, "capacity": 8,
         "graph_iters": 128},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = max(listed(), key=lambda c: work(c)["flops"])
    most = work(largest)["flops"]
    while True:
        kind = rng.choice(["query", "query", "removal", "removal", "removal", "removal", "removal", "resume", "batch",
                           "serve"])
        if kind == "batch":
            case = {"kind": kind, "images": rng.randint(3, 12), "patch": rng.choice([7, 9, 11]),
                    "max_width": _spread(rng, 400, 1280), "max_height": _spread(rng, 300, 720),
                    "graph_iters": rng.choice([16, 64, 128])}
        elif kind == "serve":
            case = {"kind": kind, "images": rng.randint(3, 8), "max_width": _spread(rng, 400, 1600),
                    "max_height": _spread(rng, 300, 1200), "capacity": rng.randint(2, 8),
                    "graph_iters": rng.choice([64, 128])}
        else:
            path = rng.choice(["auto", "simt", "mfma", "mfma"])
            patch = rng.choice([5, 7, 9, 11, 13] if path == "mfma" else [5, 7, 9, 11, 13, 17])
            case = _image(kind, "", _spread(rng, 128, 2048), _spread(rng, 96, 1536), patch,
                          rng.choice(["noise", "voronoi", "gradient"]), round(rng.uniform(0.01, 0.10), 4),
                          rng.randint(1, 3), path=path)
            del case["name"]
            if kind != "query" and rng.random() < 0.3:
                case["alpha_num"], case["alpha_den"] = rng.choice([(1, 2), (1, 1), (2, 1)])
            if kind == "query":
                case["targets"], case["static"] = rng.randint(1, 8), rng.random() < 0.5
            else:
                case["form"] = rng.choice(["plain", "stream", "graph", "persistent", "persistent", "persistent"])
                case["check"] = {"plain": 16, "stream": 128, "graph": 16, "persistent": 1024}[case["form"]]
            if kind == "removal" and path == "auto" and rng.random() < 0.3:
                case["current"], case["intersect"] = rng.choice([(True, False), (False, True), (True, True)])
            if kind == "resume":
                case["before"], case["iterations"] = _spread(rng, 4, 400), _spread(rng, 1, 256)
        # no costlier than the largest listed case: its work, its iterations, and its launches
        slow = case.get("form") != "persistent" and kind in ("removal", "resume")
        if work(case)["flops"] <= most and _iterations(case) <= (2500 if slow else 5000):
            return case


# ------------------------------------------------------------------ inputs

def _content(name, width, height, rng):
    if name == "noise":
        return synth.content_noise_edges(width, height, rng)
    if name == "voronoi":
        return synth.content_voronoi_textures(width, height, rng)
    return synth.content_gradient_rects(width, height, rng)


def _picture(case, seed):
    content, hole = [np.random.default_rng(s) for s in np.random.SeedSequence(seed).spawn(2)]
    width, height, patch = case["width"], case["height"], case["patch"]
    small = min(width, height)
    rgb = _content(case["content"], width, height, content)
    mask = synth.mask_blobs(width, height, hole, case["hole"], case["blobs"], max(3, small // 54), max(6, small // 18),
                            patch)
    return rgb, mask


def _context(case, rgb, mask):
    search = B.SEARCH_FULL if case["alpha_den"] == ALPHA_FULL else B.SEARCH_ALPHA
    alpha = (0, 1) if search == B.SEARCH_FULL else (case["alpha_num"], case["alpha_den"])
    return B.Inpainter(rgb, mask, case["patch"] // 2, search_mode=search, alpha=alpha, path=PATHS[case["path"]],
                       form=case["form"], iters_per_check=case["check"],
                       source_policy=B.SOURCE_CURRENT if case["current"] else B.SOURCE_ORIGINAL,
                       scoring=B.SCORE_INTERSECT if case["intersect"] else B.SCORE_WHOLE)


def _targets(case, mask, seed):
    """Hole-border pixels, where a removal's targets lie."""
    hole = mask != 0
    known = np.zeros_like(hole)
    known[1:] |= ~hole[:-1]
    known[:-1] |= ~hole[1:]
    known[:, 1:] |= ~hole[:, :-1]
    known[:, :-1] |= ~hole[:, 1:]
    ys, xs = np.nonzero(hole & known)
    pick = np.random.default_rng(seed).integers(0, len(xs), size=case["targets"])
    return [(int(xs[i]), int(ys[i])) for i in pick]


def _members(case):
    """The images of a batch or a queue: sizes from half the largest width and height up."""
    sizes = np.random.default_rng((case["images"], case["max_width"], case["max_height"]))
    for i in range(case["images"]):
        yield {"kind": "removal", "patch": case["patch"] if "patch" in case else (7, 9, 11)[i % 3],
               "width": int(sizes.integers(case["max_width"] // 2, case["max_width"] + 1)),
               "height": int(sizes.integers(case["max_height"] // 2, case["max_height"] + 1)),
               "hole": float(sizes.uniform(0.02, 0.06)), "blobs": int(sizes.integers(1, 4)),
               "content": "voronoi" if i % 2 else "gradient", "alpha_den": ALPHA_FULL, "intersect": False}


def _jobs(case, seed):
    jobs = []
    for i, one in enumerate(_members(case)):
        rgb, mask = _picture(one, (seed, i))
        jobs.append(synth.Job("job%d" % i, rgb, mask, one["patch"] // 2))
    return jobs


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "batch":
        state["jobs"] = _jobs(case, seed)
        state["batch"] = B.Batch(case["images"], case["graph_iters"])
        return state
    if kind == "serve":
        state["jobs"] = _jobs(case, seed)
        state["engine"] = serve.GpuEngine(case["capacity"], case["graph_iters"])
        return state
    rgb, mask = _picture(case, seed)
    if kind == "removal":
        state["rgb"], state["mask"] = rgb, mask
        return state
    state["context"] = _context(case, rgb, mask)
    if kind == "query":
        state["targets"] = _targets(case, mask, seed)
    else:
        state["context"].run(max_iters=case["before"])
        state["checkpoint"] = state["context"].export_state()
    return state


# -------------------------------------------------------------------- passes

def _log(case, log):
    """The fill log as one array of whole numbers and one of reals; a removal's length depends
    on its mask, so both end with rows of zeros."""
    rows = 6 * _iterations(case) + 64
    if len(log) > rows:
        raise ValueError("the removal took %d iterations" % len(log))
    whole, real = np.zeros((rows, len(LOG_WHOLE)), np.int64), np.zeros((rows, len(LOG_REAL)))
    for i, f in enumerate(LOG_WHOLE):
        whole[:len(log), i] = log[f]
    for i, f in enumerate(LOG_REAL):
        real[:len(log), i] = log[f]
    return [whole, real]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "query":
        find = state["context"].find_exemplar_static if case["static"] else state["context"].find_exemplar
        return np.array([find(x, y) for x, y in state["targets"]], dtype=np.int64)
    if kind == "removal":
        mask = state["mask"]
        job = _context(case, state["rgb"], mask)
        _, _, log = job.run(log_cap=int(np.count_nonzero(mask)))
        image = job.read_image()
        job.close()
        return [image] + _log(case, log)
    if kind == "resume":
        job = state["context"]
        job.import_state(*state["checkpoint"])
        job.run(max_iters=case["iterations"])
        return list(job.export_state())
    if kind == "batch":
        batch = state["batch"]
        jobs = [B.Inpainter(j.rgb, j.mask, j.patch_radius, path=B.PATH_MFMA) for j in state["jobs"]]
        for j in jobs:
            batch.attach(j)
        while batch.step():
            pass
        out = []
        for one, j in zip(_members(case), jobs):
            batch.detach(j)
            out += [j.read_image()] + _log(one, j.read_log(0, j.progress()[0]))
            j.close()
        return out
    server = serve.Server(state["engine"], SERVE_BUDGET, case["capacity"], case["graph_iters"], workers=1)
    out = []
    for one, rec in zip(_members(case), server.run(state["jobs"])):
        out += [rec.result["image"]] + _log(one, rec.result["log"])
    return out


# ----------------------------------------------------------------- the least

def _patch_iterations(width, height, hole, patch):
    """A fill copies about a third of a patch."""
    return max(1, int(width * height * hole / (0.33 * patch * patch)))


def _iterations(case):
    kind = case["kind"]
    if kind == "query":
        return case["targets"]
    if kind in ("batch", "serve"):
        return sum(_iterations(one) for one in _members(case))
    if kind == "resume":
        return case["iterations"]
    n = _patch_iterations(case["width"], case["height"], case["hole"], case["patch"])
    return 2 * n if case["intersect"] else n


def work(case):
    """Host buffers in and out once; two operations for each product of Eq. 4, over every
    centre of the search and the known two thirds of each target patch."""
    if case["kind"] in ("batch", "serve"):
        each = [work(one) for one in _members(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    patch, pixels = case["patch"], case["width"] * case["height"]
    centres = pixels
    if case["alpha_den"] != ALPHA_FULL:
        side = 1 + 2 * case["alpha_num"] / case["alpha_den"]
        centres = min(pixels, 3 * case["hole"] * pixels * side * side)
    iterations = _iterations(case)
    flops = 2.0 * iterations * centres * 3 * 0.65 * patch * patch
    if case["kind"] == "query":
        return {"bytes": float(7 * centres + 16 * iterations), "flops": flops}
    moved = (3 + 1 + 3) * pixels + 64 * iterations
    if case["kind"] == "resume":
        moved = 2 * (3 + 1 + 8) * pixels
    return {"bytes": float(moved), "flops": flops}


# --------------------------------------------------------------------- exact

def _shifted(a, dx, dy, fill):
    """out[y, x] = a[y + dy, x + dx], `fill` outside."""
    height, width = a.shape[:2]
    out = np.full_like(a, fill)
    y0, y1, x0, x1 = max(0, -dy), min(height, height - dy), max(0, -dx), min(width, width - dx)
    if y1 > y0 and x1 > x0:
        out[y0:y1, x0:x1] = a[y0 + dy:y1 + dy, x0 + dx:x1 + dx]
    return out


def _valid(mask, r):
    """Centres whose whole window lies in the image and outside the original hole."""
    bad = mask != 0
    out = np.ones(bad.shape, dtype=bool)
    for d in range(-r, r + 1):
        out &= ~_shifted(bad, d, 0, True)
    rows = out.copy()
    for d in range(-r, r + 1):
        out &= _shifted(rows, 0, d, False)
    return out


def _best_patch(image, hole, valid, x, y, r):
    """(centre, SSD, known pixels) of the best exemplar, ties to the lowest raster index."""
    height, width = hole.shape
    ssd = np.zeros((height, width), dtype=np.int64)
    known = 0
    for dy in range(-r, r + 1):
        for dx in range(-r, r + 1):
            if not (0 <= x + dx < width and 0 <= y + dy < height) or hole[y + dy, x + dx]:
                continue
            known += 1
            diff = _shifted(image, dx, dy, 0) - image[y + dy, x + dx]
            ssd += (diff.astype(np.int64) ** 2).sum(axis=2)
    ssd[~valid] = np.iinfo(np.int64).max
    best = int(ssd.argmin())
    return best, int(ssd.flat[best]), known


def _exact_removal(rgb, mask, r):
    """The fill loop in plain numpy and binary64."""
    height, width = mask.shape
    patch = 2 * r + 1
    hole = mask != 0
    image = rgb.astype(np.int32)
    image[hole] = 0
    conf = np.where(hole, 0.0, 1.0)
    valid = _valid(mask, r)
    rows = []
    while hole.any():
        gray = (299 * image[..., 0] + 587 * image[..., 1] + 114 * image[..., 2] + 500) // 1000
        known = ~hole
        near = [_shifted(known, dx, dy, False) for dx, dy in ((1, 0), (-1, 0), (0, 1), (0, -1))]
        inner = known & near[0] & near[1] & near[2] & near[3]
        gx = _shifted(gray, 1, 0, 0) - _shifted(gray, -1, 0, 0)
        gy = _shifted(gray, 0, 1, 0) - _shifted(gray, 0, -1, 0)
        size = np.where(inner, gx * gx + gy * gy, -1)
        nx = (~near[0]).astype(np.int64) - (~near[1])
        ny = (~near[2]).astype(np.int64) - (~near[3])
        top = None
        for y, x in zip(*np.nonzero(hole & (near[0] | near[1] | near[2] | near[3]))):
            box = (slice(max(y - r, 0), y + r + 1), slice(max(x - r, 0), x + r + 1))
            c = 0.0
            for v in conf[box][known[box]].tolist():
                c += v
            c /= float(patch * patch)
            sizes = size[box]
            at = np.unravel_index(int(sizes.argmax()), sizes.shape)
            n2 = int(nx[y, x] ** 2 + ny[y, x] ** 2)
            d = 0.0
            if n2 and sizes[at] >= 0:
                along = abs(int(gx[box][at]) * int(ny[y, x]) - int(gy[box][at]) * int(nx[y, x]))
                d = 0.5 * float(along) / (255.0 if n2 == 1 else math.sqrt(2.0) * 255.0)
            if top is None or c * d > top[0]:
                top = (c * d, c, d, int(x), int(y))
        p, c, d, x, y = top
        q, ssd, k = _best_patch(image, hole, valid, x, y, r)
        qx, qy = q % width, q // width
        filled = 0
        for dy in range(-r, r + 1):
            for dx in range(-r, r + 1):
                if 0 <= x + dx < width and 0 <= y + dy < height and hole[y + dy, x + dx]:
                    hole[y + dy, x + dx] = False
                    image[y + dy, x + dx] = image[qy + dy, qx + dx]
                    conf[y + dy, x + dx] = c
                    filled += 1
        rows.append((y * width + x, q, ssd, k, filled, int(hole.sum()), p, c, d))
    log = np.zeros(len(rows), dtype=[(f, "i8") for f in LOG_WHOLE] + [(f, "f8") for f in LOG_REAL])
    log[:] = rows
    return image.astype(np.uint8), log


def exact(case, seed):
    if case["kind"] == "query":
        r = case["patch"] // 2
        if case["width"] * case["height"] * case["targets"] * case["patch"] ** 2 > 6e8:
            return None
        rgb, mask = _picture(case, seed)
        image, hole = rgb.astype(np.int32), mask != 0
        valid = _valid(mask, r)
        return np.array([_best_patch(image, hole, valid, x, y, r)[:2] for x, y in _targets(case, mask, seed)],
                        dtype=np.int64)
    plain = case["kind"] == "removal" and case["alpha_den"] == ALPHA_FULL
    if not plain or case["current"] or case["intersect"]:
        return None
    if case["width"] * case["height"] * case["width"] * case["height"] * case["hole"] > 1.5e8:
        return None
    image, log = _exact_removal(*_picture(case, seed), case["patch"] // 2)
    return [image] + _log(case, log)
