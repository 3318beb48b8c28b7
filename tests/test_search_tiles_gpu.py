"""Edges of the MFMA search tile, the AUTO dispatch and the superblock maxima,
against the CPU oracle (integers and bit patterns: no tolerance)."""
import numpy as np
import pytest

import oracle
from paper_1403_4238_amd import synth

from _util import assert_logs_equal
from test_parity_gpu import B, _built, _full_run_parity, _pair  # noqa: F401

pytestmark = pytest.mark.gpu


# Candidate grids (W - 2r) x (H - 2r) of one pixel, one tile, a tile and a
# pixel, and ragged ones, at every radius; AUTO runs the MFMA search here.
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("cw,ch", [(1, 40), (64, 64), (65, 63), (67, 130)])
def test_tile_edges_match_oracle(r, cw, ch):
    W, H = cw + 2 * r, ch + 2 * r
    rng = np.random.default_rng(100 * r + cw)
    rgb = rng.integers(0, 256, size=(H, W, 3)).astype(np.uint8)
    rgb[: H // 3] = (rng.integers(0, 2, size=(H // 3, W, 1)) * 255).astype(np.uint8)   # the extreme values
    mask = np.zeros((H, W), np.uint8)
    mask[H - 1, W - 1] = 1
    job = synth.Job("edge", rgb, mask, r)
    if cw == 1:
        mask[H - 1, W - 1], mask[0, 0] = 0, 1
    o, g = _pair(job)
    for x, y in ((W - 1, H - 1), (0, H // 2), (W // 2, H // 2), (W // 2, 0)):
        assert g.find_exemplar(x, y, r) == o.find_exemplar(x, y, r, (0, 0, W, H))[:2], (x, y)
        assert g.find_exemplar_static(x, y, r) == g.find_exemplar(x, y, r)


@pytest.mark.parametrize("r", [7, 8])
@pytest.mark.parametrize("form", ["plain", "stream", "graph", "persistent"])
def test_auto_large_radii_full_run(r, form):
    job = synth.small()
    job.patch_radius = r
    _full_run_parity(job, f"auto r={r} {form}", form=form, iters_per_check=3)


@pytest.mark.parametrize("path", [B.PATH_AUTO, B.PATH_SIMT])
def test_auto_equals_simt_with_current_sources(path):
    job = synth.small()
    o = oracle.Oracle(job.rgb, job.mask, 4, source_policy=1)
    g = B.Inpainter(job.rgb, job.mask, 4, path=path, source_policy=B.SOURCE_CURRENT)
    want = o.run()
    st, n, got = g.run(log_cap=len(want) + 8)
    assert st == B.DONE and n == len(want)
    for f in ("target_index", "source_index", "ssd", "remaining"):
        assert (got[f] == want[f]).all(), f
    assert (g.read_image() == o.read()[0]).all()


# Two holes far apart: the priority range needs superblocks of more than
# 8 x 8 blocks, and the far target is the usual one.
@pytest.mark.parametrize("form,path", [("persistent", B.PATH_AUTO), ("stream", B.PATH_AUTO), ("persistent", B.PATH_SIMT)])
def test_large_superblocks(form, path):
    W, H, r = 1700, 1500, 2
    rng = np.random.default_rng(9)
    rgb = rng.integers(0, 256, size=(H, W, 3)).astype(np.uint8)
    mask = np.zeros((H, W), np.uint8)
    mask[20:32, 25:39] = 1
    mask[H - 40:H - 29, W - 45:W - 30] = 1
    job = synth.Job("far", rgb, mask, r, search_mode=synth.SEARCH_RECT, rect=(700, 700, 780, 770))
    _full_run_parity(job, f"far holes {form}", form=form, path=path, iters_per_check=16)


# More tiles than resident groups at the radius whose group holds one tile per
# CU and three in LDS, and at radius 7 (one in LDS): tiles take turns.
@pytest.mark.parametrize("r", [7, 8])
def test_large_radii_several_tiles_per_group(r):
    W, H = 2600, 1400
    rng = np.random.default_rng(r)
    rgb = synth.content_voronoi_textures(W, H, rng)
    mask = np.zeros((H, W), np.uint8)
    mask[600:640, 1000:1050] = 1
    a = B.Inpainter(rgb, mask, r, form="persistent", iters_per_check=64)
    b = B.Inpainter(rgb, mask, r, path=B.PATH_SIMT, form="stream", iters_per_check=16)
    na, nb = a.run(log_cap=4096), b.run(log_cap=4096)
    assert a.run_form() == "persistent" and na[1] == nb[1] > 0
    for f in na[2].dtype.names:
        assert na[2][f].tobytes() == nb[2][f].tobytes(), f
    assert (a.read_image() == b.read_image()).all()


@pytest.mark.parametrize("path,n,radii,first", [("auto", 32, (4,), "persistent"), ("mfma", 64, (4,), "graph"),
                                                 ("simt", 32, (4,), "graph"), ("auto", 32, (1, 3, 5), "persistent")])
def test_auto_batch_form_by_items_per_group(path, n, radii, first):
    # Either side of AUTO's line between the batch forms (12 MFMA items per
    # search work-group, 16 with several radii, 4 SIMT ones): the form of the
    # first step, and each log's head against the image stepped alone.
    jobs = synth.batch()[:n]
    pid = {"auto": B.PATH_AUTO, "mfma": B.PATH_MFMA, "simt": B.PATH_SIMT}[path]
    rs = [radii[i % len(radii)] for i in range(n)]
    batch = B.Batch(capacity=n, graph_iters=6, autotune=False, form="auto")
    ctxs = [B.Inpainter(j.rgb, j.mask, r, path=pid) for j, r in zip(jobs, rs)]
    for c in ctxs:
        batch.attach(c)
    batch.step()
    assert batch.last_form() == first
    batch.step()
    for i in range(0, n, 5):
        alone = B.Inpainter(jobs[i].rgb, jobs[i].mask, rs[i], path=B.PATH_SIMT)
        alone.run(max_iters=12)
        assert_logs_equal(ctxs[i].read_log(0, 12), alone.read_log(0, 12), jobs[i].name)
        alone.close()
    for c in ctxs:
        batch.detach(c)
        c.close()
    batch.close()
