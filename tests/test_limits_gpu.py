"""Calls at the limits of what the library accepts."""
import numpy as np
import pytest

import oracle
from paper_1403_4238_amd import synth

from test_parity_gpu import B, _built, _full_run_parity  # noqa: F401

pytestmark = pytest.mark.gpu


def _noise(W, H, seed):
    return np.random.default_rng(seed).integers(0, 256, size=(H, W, 3)).astype(np.uint8)


def test_static_query_of_as_many_tiles_as_the_scratch_holds():
    # 32768 SIMT tiles in one row; the aligned MFMA tiling has one more
    W, H, r = 2097167, 9, 4
    rgb = _noise(W, H, 1)
    mask = np.zeros((H, W), np.uint8)
    mask[3:6, 1000:1004] = 1
    g = B.Inpainter(rgb, mask, r)
    rect = (11, 0, W, H)
    want = g.find_exemplar(1000, 4, r, rect)
    assert g.find_exemplar_static(1000, 4, r, rect) == want
    with pytest.raises(B.InpaintError) as e:
        g.find_exemplar_static(1000, 4, r, (10, 0, W, H))
    assert e.value.status == B.INVALID_ARGUMENT
    g.close()


# The last record of a dispatch that empties the hole follows its iteration
# with no barrier of the next one between; here it is also the first record.
@pytest.mark.parametrize("r", range(1, 9))
@pytest.mark.parametrize("path", ["auto", "simt"])
def test_record_of_an_iteration_that_empties_the_hole(r, path):
    import torch
    mask = np.zeros((70, 90), np.uint8)
    mask[30:30 + min(r + 1, 6), 40] = 1   # within the patch of its every pixel
    job = synth.Job("one", _noise(90, 70, r), mask, r)
    for iters in (1, 64):
        stale = torch.full((4 << 20,), 0xAB, dtype=torch.uint8, device="cuda")   # the workspace's block
        del stale
        log = _full_run_parity(job, "one iteration r=%d" % r, path={"auto": B.PATH_AUTO, "simt": B.PATH_SIMT}[path],
                               form="persistent", iters_per_check=iters)
        assert len(log) == 1


# More rows of 64 x 16 tiles of the padded planes than a grid's second dimension
# takes; the search rect keeps the oracle's search small.
def test_very_tall_image():
    W, H, r = 17, 1_100_000, 2
    rgb = _noise(W, H, 3)
    mask = np.zeros((H, W), np.uint8)
    mask[H - 9:H - 5, 8:13] = 1
    job = synth.Job("tall", rgb, mask, r, search_mode=synth.SEARCH_RECT, rect=(0, H - 300, W, H))
    _full_run_parity(job, "tall", form="persistent", iters_per_check=8)


# More AUTO images than the MFMA dispatch has committers for (256 of 512
# work-groups), of one radius and of the radii that share the mixed dispatch:
# the persistent form takes them on the SIMT search, and goes over to the
# matrix cores once enough are done.
@pytest.mark.parametrize("radii", [(2,), (1, 2, 3, 4, 5)])
def test_more_auto_images_than_mfma_committers(radii):
    n, W, H = 300, 48, 40
    batch = B.Batch(n, 2, form="persistent")
    jobs = []
    for i in range(n):
        mask = np.zeros((H, W), np.uint8)
        mask[12:14 + 3 * (i % 4), 15 + i % 9:22 + i % 9] = 1
        jobs.append((_noise(W, H, i), mask, radii[i % len(radii)]))
    ctxs = [B.Inpainter(*j) for j in jobs]
    for i, c in enumerate(ctxs):
        assert batch.room(c, 64), i
        batch.attach(c)
    left = n
    for _ in range(100):
        left = batch.step()
        assert batch.last_form() == "persistent"
        if not left:
            break
    assert left == 0
    for i in range(0, n, 23):
        alone = B.Inpainter(*jobs[i], path=B.PATH_SIMT)
        k = alone.run(log_cap=400)[1]
        assert ctxs[i].progress()[0] == k
        assert ctxs[i].read_log(0, k).tobytes() == alone.read_log(0, k).tobytes(), i
        assert (ctxs[i].read_image() == alone.read_image()).all()
        alone.close()
    for c in ctxs:
        batch.detach(c)
        c.close()
    batch.close()


# As many SIMT tiles in one row as the persistent form takes (8192); the aligned
# MFMA tiling has one more, so AUTO keeps the form on the SIMT search.
@pytest.mark.parametrize("x0,form", [(2, "persistent"), (1, "stream")])
def test_auto_persistent_at_its_most_tiles(x0, form):
    W, H, r = 64 * 8192 + 3, 9, 1
    rgb = _noise(W, H, 5)
    mask = np.zeros((H, W), np.uint8)
    mask[4, 300000:300004] = 1
    job = synth.Job("wide", rgb, mask, r, search_mode=synth.SEARCH_RECT, rect=(x0, 0, W, H))
    g = B.Inpainter(rgb, mask, r, B.SEARCH_RECT, rect=job.rect, form="persistent", iters_per_check=8)
    assert g.run_form() == form
    g.close()
    _full_run_parity(job, "wide", form="persistent", iters_per_check=8)


# The image read back whole: packed on the host up to 2^17 pixels, above on the
# device in pieces that end within rows; with the caller's rows packed or padded.
@pytest.mark.parametrize("W,H", [(40, 30), (362, 362), (363, 362), (701, 433), (1031, 777)])
@pytest.mark.parametrize("pad", [0, 13])
def test_read_image_rows(W, H, pad):
    rgb = _noise(W, H, W)
    mask = np.zeros((H, W), np.uint8)
    mask[5:9, 7:12] = 1
    g = B.Inpainter(rgb, mask, 2)
    out = np.full((H, 3 * W + pad), 0x5A, np.uint8)
    for _ in range(2):
        assert B.lib().inpaint_read_image(g.ctx, out.ctypes.data, 3 * W + pad) == B.OK
        want = rgb * (mask == 0)[..., None]
        assert (out[:, :3 * W].reshape(H, W, 3) == want).all()
        assert (out[:, 3 * W:] == 0x5A).all()
    assert B.lib().inpaint_read_image(g.ctx, out.ctypes.data, 3 * W - 1) == B.INVALID_ARGUMENT
    g.close()


# The read-back works in planes that hold nothing between calls: a removal that
# is read back part of the way goes on as one that is not.
@pytest.mark.parametrize("kw", [dict(form="persistent"), dict(form="graph"), dict(form="stream", path=B.PATH_SIMT),
                                dict(form="stream", source_policy=B.SOURCE_CURRENT),
                                dict(form="stream", source_policy=B.SOURCE_CURRENT, scoring=B.SCORE_INTERSECT)])
def test_read_image_between_runs_changes_nothing(kw):
    job = synth.vga()
    a, b = [B.Inpainter(job.rgb, job.mask, 4, iters_per_check=8, **kw) for _ in range(2)]
    for _ in range(4):
        a.run(max_iters=24)
        a.read_image()
        a.find_exemplar_static(300, 200)
    b.run(max_iters=96)
    assert a.read_log(0, 96).tobytes() == b.read_log(0, 96).tobytes()
    assert (a.read_image() == b.read_image()).all()
    ck = a.export_state()
    a.import_state(*ck)
    a.read_image()
    assert a.run(max_iters=24)[1] == b.run(max_iters=24)[1]
    assert a.read_log(96, 24).tobytes() == b.read_log(96, 24).tobytes()
    for g in (a, b):
        g.close()


# The stream form's commit reduces one minimum per tile, eight per thread and
# round: counts on either side of its rounds of 2048.
@pytest.mark.parametrize("tiles", [2047, 2048, 2049, 4097, 9000])
def test_minima_of_many_tiles(tiles):
    W, H, r = 64 * tiles + 2, 9, 1
    rgb = _noise(W, H, tiles)
    mask = np.zeros((H, W), np.uint8)
    mask[3:6, 90:97] = 1
    mask[3:6, W - 90:W - 81] = 1
    log = _full_run_parity(synth.Job("wide", rgb, mask, r), "%d tiles" % tiles, path=B.PATH_SIMT, form="stream",
                           iters_per_check=4)
    assert len(np.unique(log["source_index"] % W // 64)) > 4


# 8200 SIMT tiles and 4100 MFMA tiles: AUTO runs the persistent form where the
# SIMT tiling does, so it takes the stream form here; results are the same.
@pytest.mark.parametrize("r", [1, 2])
def test_auto_persistent_goes_by_the_simt_tiles(r):
    W, H = 64 * 99 + 40 + 2 * r, 32 * 81 + 20 + 2 * r
    rgb = _noise(W, H, r)
    mask = np.zeros((H, W), np.uint8)
    mask[700:712, 3000:3020] = 1
    logs = []
    for path, form in ((B.PATH_AUTO, "stream"), (B.PATH_MFMA, "persistent"), (B.PATH_SIMT, "stream")):
        g = B.Inpainter(rgb, mask, r, path=path, form="persistent", iters_per_check=32)
        assert g.run_form() == form
        st, n, log = g.run(log_cap=400)
        assert st == B.DONE
        logs.append(log.tobytes())
        g.close()
    assert logs[0] == logs[1] == logs[2]


# The MFMA tile of radius 1 at the edges of its tiles (AUTO's queries of that
# radius run the SIMT search).
@pytest.mark.parametrize("cw,ch", [(1, 40), (64, 64), (65, 63), (67, 130)])
def test_mfma_tile_edges_radius_1(cw, ch):
    W, H, r = cw + 2, ch + 2, 1
    rgb = _noise(W, H, cw)
    rgb[: H // 3] = np.where(rgb[: H // 3, :, :1] > 127, 255, 0)
    mask = np.zeros((H, W), np.uint8)
    mask[0, 0] = 1
    o = oracle.Oracle(rgb, mask, r)
    for path in (B.PATH_MFMA, B.PATH_AUTO):
        g = B.Inpainter(rgb, mask, r, path=path)
        for x, y in ((W - 1, H - 1), (0, H // 2), (W // 2, H // 2), (W // 2, 0)):
            assert g.find_exemplar(x, y, r) == o.find_exemplar(x, y, r, (0, 0, W, H))[:2], (x, y)
            assert g.find_exemplar_static(x, y, r) == g.find_exemplar(x, y, r)
        g.close()
