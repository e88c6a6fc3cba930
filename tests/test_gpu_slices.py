"""Frames of few batches, whose batches the render and shading kernels cut into slices, against the oracle.

Point counts around the edges of the slicing (one group of 256 points, a ragged tail, one batch more or less, as many
batches as there are workgroups to fill), in tiled, banded and untiled batches (the camera's distance decides), single
views, several views in one launch and shading: bit for bit.
"""
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


def _cams(n):
    # far (the batches' rectangles fit a tile), middle (bands), near (untiled)
    return [synth.camera((50.0, -d, 60.0 + d / 4), (50, 50, 50), (0, 0, 1), 60.0, w, h, 0.5, 5000.0)
            for d, w, h in ((1500.0, 320, 200), (400.0, 641, 479), (90.0, 1023, 701))]


@pytest.mark.parametrize("n,S", [(1, 4), (255, 256), (257, 1024), (2560, 2560), (10239, 10240), (10241, 10240),
                                 (20011, 10240), (40003, 1024), (163841, 10240), (300007, 512)])
def test_few_batches(ctx, n, S):
    import torch
    import paper_2204_01287_amd as pr

    xyz, rgba = synth.primitives(3, n)
    say(f"slices: build n={n} S={S}")
    dc, B = gpu_build(ctx, xyz, rgba, S, 0), oracle.build_cloud(xyz, rgba, S, morton=0)
    cams = _cams(n)
    refs = []
    for c in cams:
        for bands in (0, 64):
            say(f"slices: n={n} S={S} {c.width}x{c.height} bands={bands}")
            pr.pr_set_tuning(ctx.handle, max_bands=bands)
            vb, fb, st = gpu_render(ctx, dc, c.view, c.proj, c.width, c.height)
            ref, st_ref = oracle.render(B, c.view, c.proj, c.width, c.height)
            assert_vb_equal(vb, ref, c.width)
            oracle_stats_match(st, st_ref)
        refs.append(ref)
    pr.pr_set_tuning(ctx.handle)
    vbs = [torch.empty(c.width * c.height, dtype=torch.int64, device="cuda") for c in cams]
    need = pr.pr_views_work_bytes(dc.handle, len(cams))
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    say(f"slices: n={n} S={S} views")
    pr.pr_render_views(ctx.handle, dc.handle, [(c.view, c.proj, c.width, c.height, vb) for c, vb in zip(cams, vbs)],
                       None, work, need)
    pr.pr_sync(ctx.handle)
    for c, vb, ref in zip(cams, vbs, refs):
        assert_vb_equal(vb.cpu().numpy().view(np.uint64), ref, c.width)
    for c, ref in zip(cams, refs):
        px = c.width * c.height
        vb = torch.empty(px, dtype=torch.int64, device="cuda")
        acc = torch.empty(2 * px + px % 2, dtype=torch.int64, device="cuda")
        fb = torch.empty(px, dtype=torch.int32, device="cuda")
        say(f"slices: n={n} S={S} {c.width}x{c.height} shading")
        pr.pr_render_hqs(ctx.handle, dc.handle, c.view, c.proj, c.width, c.height, None, 1.01, vb, acc, 7, fb)
        pr.pr_sync(ctx.handle)
        want = oracle.accumulate(B, c.view, c.proj, c.width, c.height, ref, 1.01)
        assert np.array_equal(acc.cpu().numpy().view(np.uint64)[:2 * px], want)
        assert np.array_equal(fb.cpu().numpy().view(np.uint32), oracle.resolve_hqs(want, 7))


@pytest.mark.parametrize("S", [1280, 2836, 4100])
@pytest.mark.parametrize("precision", [10, 20, 30])
def test_untiled_groups(ctx, S, precision):
    """Batches that span the image (points in no order), too many to be sliced: a wave's groups of 256 points in pairs,
    odd numbers of groups and ragged tails, at each precision, straight into the visibility buffer and the sums."""
    import torch
    import paper_2204_01287_amd as pr

    xyz, rgba = synth.primitives(5, 1100 * S)
    o = np.random.default_rng(S).permutation(len(xyz))
    xyz, rgba = np.ascontiguousarray(xyz[o]), np.ascontiguousarray(rgba[o])
    say(f"untiled groups: S={S} precision={precision}")
    dc, B = gpu_build(ctx, xyz, rgba, S, 0), oracle.build_cloud(xyz, rgba, S, morton=0)
    c = synth.camera((50.0, -90.0, 80.0), (50, 50, 50), (0, 0, 1), 60.0, 1023, 701, 0.5, 5000.0)
    px = c.width * c.height
    vb = torch.empty(px, dtype=torch.int64, device="cuda")
    acc = torch.empty(2 * px + px % 2, dtype=torch.int64, device="cuda")
    fb = torch.empty(px, dtype=torch.int32, device="cuda")
    pr.pr_render_hqs(ctx.handle, dc.handle, c.view, c.proj, c.width, c.height, pr.RenderOpts.make(precision=precision),
                     1.01, vb, acc, 7, fb)
    pr.pr_sync(ctx.handle)
    ref, _ = oracle.render(B, c.view, c.proj, c.width, c.height, oracle.opts(precision=precision))
    assert_vb_equal(vb.cpu().numpy().view(np.uint64), ref, c.width)
    want = oracle.accumulate(B, c.view, c.proj, c.width, c.height, ref, 1.01, oracle.opts(precision=precision))
    assert np.array_equal(acc.cpu().numpy().view(np.uint64)[:2 * px], want)
