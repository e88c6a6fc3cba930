"""The build of every point order against the oracle on clouds that reach each branch of the sort and of the batch
kernel: counts around a sort tile (8,192) and a run tile (2,048), more leading-bit passes as the count grows, runs that
the leading bits leave equal (short, longer than the run limit, of equal points, out of order: sorted again in full), and
batch sizes around the ones that the whole-batch kernel takes (512 .. 20,480) and its workgroup sizes."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_build_equal, gpu_build, gpu_build_outputs, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    import paper_2204_01287_amd as pr

    assert torch.cuda.is_available()
    c = pr.Context(0)
    yield c
    c.close()


def _cloud(kind, n):
    rng = np.random.default_rng(n)
    if kind == "primitives":
        return synth.primitives(3, n)
    if kind == "terrain":
        return synth.terrain(3, n, order=0)
    x = rng.random((n, 3), dtype=np.float32)
    if kind == "equal":
        x[:] = 1.25
    elif kind == "outlier":  # one far point: all others agree in the leading bits, out of order
        x[n // 2] = 1e7
    elif kind == "repeats":  # one point many times among others: a long run, in order
        x[::3] = 0.5
    elif kind == "two":  # two close points alternating, and a far one
        x[:] = np.where(rng.random((n, 1)) < 0.5, 0.0, 1e-3)
        x[-1] = 1e4
    elif kind == "grid":
        x = rng.integers(0, 64, (n, 3)).astype(np.float32)
    return x, rng.integers(0, 1 << 32, n, dtype=np.uint32)


@pytest.mark.parametrize("kind,n", [("primitives", 1), ("primitives", 2047), ("primitives", 2049), ("primitives", 8192),
                                    ("primitives", 8193), ("primitives", 70001), ("terrain", 300007),
                                    ("terrain", 5000001), ("equal", 100003), ("outlier", 200001), ("repeats", 150000),
                                    ("two", 120001), ("grid", 250001)])
def test_orders(ctx, kind, n):
    xyz, rgba = _cloud(kind, n)
    sizes = [(10240, 2), (10240, 0)] if n > 1000000 else [
        (10240, 2), (10240, 1), (10240, 0), (508, 2), (512, 2), (5120, 1), (5124, 2), (10244, 0), (20480, 2), (20484, 1)]
    for S, order in sizes:
        say(f"build {kind} n={n} S={S} order={order}")
        dc = gpu_build(ctx, xyz, rgba, S, order)
        assert_build_equal(gpu_build_outputs(dc), oracle.build_cloud(xyz, rgba, S, morton=order))
        dc.close()


def test_context_after_a_refused_build(ctx):
    """A non-finite cloud leaves nothing behind for the next build of the same context."""
    import paper_2204_01287_amd as pr

    xyz, rgba = _cloud("primitives", 3001)
    for order in (0, 1, 2):
        bad = xyz.copy()
        bad[1234, 1] = np.inf
        say(f"build of a non-finite cloud, order {order}")
        with pytest.raises(pr.PrError, match="PR_ENONFINITE"):
            gpu_build(ctx, bad, rgba, 1024, order)
        dc = gpu_build(ctx, xyz, rgba, 1024, order)
        assert_build_equal(gpu_build_outputs(dc), oracle.build_cloud(xyz, rgba, 1024, morton=order))


def test_scratch_size_is_what_it_was():
    """The scratch bytes asked of callers: the sort areas of tiles of 4,096 points, plus 4 KiB."""
    import paper_2204_01287_amd as pr

    def a256(x):
        return (x + 255) // 256 * 256

    for n in (1, 4095, 4097, 8192, 12289, 1 << 20, 20_000_003, 2_000_000_000, (1 << 32) - 2):
        tiles = -(-n // 4096)
        m = 256 * tiles
        want = 4096 + 256 + 2 * a256(8 * n) + a256(4 * n) + a256(4 * m) + a256(4 * -(-m // 4096))
        assert pr.pr_cloud_sizes(n, 10240, 1).scratch == a256(want)
