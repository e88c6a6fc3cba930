"""Frames of 130 to 1,030 batches in rows across the image: banded and untiled batches together, the default band limit
(which grows where the batches leave workgroups idle) and the slices that it counts on, against the oracle; and the
default limit's time against a fixed one's."""
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


def _rows(n):
    """A hilly square kilometre, 10 m tile after tile, row by row."""
    rng = np.random.default_rng(n)
    t = np.arange(n) * 10000 // n
    x = np.empty((n, 3), np.float32)
    x[:, 0] = (t % 100 + rng.random(n)) * 10.0
    x[:, 1] = (t // 100 + rng.random(n)) * 10.0
    x[:, 2] = 15 * np.sin(x[:, 0] / 60) * np.cos(x[:, 1] / 80) + 8 * rng.random(n) * (rng.random(n) < 0.1)
    return x, rng.integers(0, 1 << 32, n, dtype=np.uint32)


def _cam(w, h, d=800.0):
    return synth.camera((500.0 + d * 0.6, 500.0 - d * 0.8, 450.0), (500, 500, 0), (0, 0, 1), 60.0, w, h, 0.5, 5000.0)


@pytest.mark.parametrize("nb,S,wg", [(130, 10240, 0), (205, 10240, 0), (300, 5120, 0), (257, 2052, 1), (255, 2052, 1),
                                     (1023, 1024, 0), (1025, 1024, 0)])
def test_mixed_frames(ctx, nb, S, wg):
    import torch
    import paper_2204_01287_amd as pr

    xyz, rgba = _rows(nb * S - 5)
    dc, B = gpu_build(ctx, xyz, rgba, S, 0), oracle.build_cloud(xyz, rgba, S, morton=0)
    cams = [_cam(1280, 720), _cam(2382, 1923), _cam(641, 479, 300.0)]
    refs = []
    for bands in (0, 16):
        pr.pr_set_tuning(ctx.handle, max_bands=bands, wg_per_cu=wg)
        refs = []
        for c in cams:
            say(f"mixed frame nb={nb} S={S} wg={wg} bands={bands} {c.width}x{c.height}")
            vb, _, st = gpu_render(ctx, dc, c.view, c.proj, c.width, c.height)
            ref, st_ref = oracle.render(B, c.view, c.proj, c.width, c.height)
            assert_vb_equal(vb, ref, c.width)
            oracle_stats_match(st, st_ref)
            refs.append(ref)
    pr.pr_set_tuning(ctx.handle, wg_per_cu=wg)
    vbs = [torch.empty((c.width * c.height + 1) // 2 * 2, dtype=torch.int64, device="cuda") for c in cams]
    need = pr.pr_views_work_bytes(dc.handle, len(cams))
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    say(f"mixed frame nb={nb} S={S} wg={wg} views")
    pr.pr_render_views(ctx.handle, dc.handle, [(c.view, c.proj, c.width, c.height, vb) for c, vb in zip(cams, vbs)], None,
                       work, need)
    pr.pr_sync(ctx.handle)
    for c, vb, ref in zip(cams, vbs, refs):
        assert_vb_equal(vb.cpu().numpy().view(np.uint64)[:c.width * c.height], ref, c.width)
    c, ref = cams[0], refs[0]
    px = c.width * c.height
    vb = torch.empty(px, dtype=torch.int64, device="cuda")
    acc = torch.empty(2 * px, dtype=torch.int64, device="cuda")
    fb = torch.empty(px, dtype=torch.int32, device="cuda")
    say(f"mixed frame nb={nb} S={S} wg={wg} shading")
    pr.pr_render_hqs(ctx.handle, dc.handle, c.view, c.proj, c.width, c.height, None, 1.01, vb, acc, 7, fb)
    pr.pr_sync(ctx.handle)
    pr.pr_set_tuning(ctx.handle)
    want = oracle.accumulate(B, c.view, c.proj, c.width, c.height, ref, 1.01)
    assert np.array_equal(acc.cpu().numpy().view(np.uint64), want)


@pytest.mark.parametrize("nb,w,h", [(130, 2382, 1923), (160, 1280, 720), (205, 1280, 720)])
def test_default_band_limit_is_no_loss(ctx, nb, w, h):
    """The default limit lies above 4 only where a batch's bands run side by side: its frames are at most as long as those
    of the fixed limit of 4, here with half as much again for the clock."""
    import torch
    import paper_2204_01287_amd as pr

    xyz, rgba = _rows(nb * 10240 - 5)
    dc = gpu_build(ctx, xyz, rgba, 10240, 0)
    c = _cam(w, h)
    vb = torch.empty((w * h + 1) // 2 * 2, dtype=torch.int64, device="cuda")
    took = {}
    for bands in (0, 4):
        pr.pr_set_tuning(ctx.handle, max_bands=bands)
        times = []
        for i in range(7):
            say(f"band limit {bands} nb={nb} {w}x{h} run {i}")
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            for _ in range(20):
                pr.pr_render(ctx.handle, dc.handle, c.view, c.proj, w, h, None, vb)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        took[bands] = min(times)
    pr.pr_set_tuning(ctx.handle)
    assert took[0] < 1.5 * took[4], took
