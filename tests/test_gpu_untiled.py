"""Untiled batches, whose points go to the visibility buffer one by one behind an early-depth read: one read in flight or
four, by the image's size and by whether the frame's batches are cut, against the oracle; and the number of atomics they
issue where batches overlap."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_vb_equal, gpu_build, gpu_render, oracle_stats_match, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    import paper_2204_01287_amd as pr

    assert torch.cuda.is_available()
    c = pr.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", [10, 20, 30])
@pytest.mark.parametrize("nb,S", [(255, 1028), (256, 2564), (300, 1280)])
def test_reads_in_flight(ctx, nb, S, precision):
    """Images on both sides of 2^20 pixels, batches just below and above the number of workgroups (one per CU), odd numbers
    of groups of 256 points and ragged tails, cameras outside (every point inside the image) and within the points."""
    import torch
    import paper_2204_01287_amd as pr

    xyz, rgba = synth.primitives(5, nb * S - 3)
    o = np.random.default_rng(S).permutation(len(xyz))
    xyz, rgba = np.ascontiguousarray(xyz[o]), np.ascontiguousarray(rgba[o])  # every batch spans the image
    dc, B = gpu_build(ctx, xyz, rgba, S, 0), oracle.build_cloud(xyz, rgba, S, morton=0)
    cams = [synth.camera((50.0, -120.0, 90.0), (50, 50, 50), (0, 0, 1), 60.0, 1024, 1024, 0.5, 5000.0),
            synth.camera((50.0, -120.0, 90.0), (50, 50, 50), (0, 0, 1), 60.0, 1025, 1024, 0.5, 5000.0),
            synth.camera((50.0, 40.0, 50.0), (50, 90, 40), (0, 0, 1), 90.0, 1361, 911, 0.05, 5000.0)]
    pr.pr_set_tuning(ctx.handle, wg_per_cu=1)
    refs = []
    for c in cams:
        say(f"untiled nb={nb} S={S} precision={precision} {c.width}x{c.height}")
        vb, _, st = gpu_render(ctx, dc, c.view, c.proj, c.width, c.height, precision=precision)
        ref, st_ref = oracle.render(B, c.view, c.proj, c.width, c.height, oracle.opts(precision=precision))
        assert_vb_equal(vb, ref, c.width)
        oracle_stats_match(st, st_ref)
        refs.append(ref)
    vbs = [torch.empty((c.width * c.height + 1) // 2 * 2, dtype=torch.int64, device="cuda") for c in cams]
    need = pr.pr_views_work_bytes(dc.handle, len(cams))
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    say(f"untiled nb={nb} S={S} precision={precision} views")
    pr.pr_render_views(ctx.handle, dc.handle, [(c.view, c.proj, c.width, c.height, vb) for c, vb in zip(cams, vbs)],
                       pr.RenderOpts.make(precision=precision), work, need)
    pr.pr_sync(ctx.handle)
    pr.pr_set_tuning(ctx.handle)
    for c, vb, ref in zip(cams, vbs, refs):
        assert_vb_equal(vb.cpu().numpy().view(np.uint64)[:c.width * c.height], ref, c.width)


@pytest.mark.parametrize("nb", [700, 1000])
def test_overlapping_batches_write_little(ctx, nb):
    """Batches that cover each other: a point that an earlier one hides must mostly be dropped by its early-depth read. The
    two render kernels work the same batches in as many workgroups; the runs of one differ by up to 20 %."""
    import torch
    import paper_2204_01287_amd as pr

    w, h = 1280, 720
    xyz, rgba = synth.primitives(3, nb * 10240 - 7)
    dc = gpu_build(ctx, xyz, rgba, 10240, 0)
    c = synth.camera((50.0, -90.0, 120.0), (50, 50, 50), (0, 0, 1), 60.0, w, h, 0.5, 1000.0)
    vb = torch.empty(w * h, dtype=torch.int64, device="cuda")
    need = pr.pr_views_work_bytes(dc.handle, 1)
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    opts = pr.RenderOpts.make(precision=20, counters=1)
    atomics = [[], []]
    for i in range(5):
        say(f"overlapping batches nb={nb} run {i}")
        pr.pr_render(ctx.handle, dc.handle, c.view, c.proj, w, h, opts, vb)
        atomics[0].append(pr.pr_get_stats(ctx.handle)["atomics"])
        pr.pr_render_views(ctx.handle, dc.handle, [(c.view, c.proj, w, h, vb)], opts, work, need)
        atomics[1].append(pr.pr_get_stats(ctx.handle)["atomics"])
    one, views = np.median(atomics[0]), np.median(atomics[1])
    assert one < 1.3 * views, atomics
