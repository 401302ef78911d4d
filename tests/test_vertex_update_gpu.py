"""GPU parity of the vertex update (the second stage of the bilateral
denoising the paper cites; restated, pinned in the oracle tests) through the
C ABI: identical float32 inputs, points within 1e-5 relative of the FP64
oracle (Euclidean, per vertex), invalid points copied bitwise, on grids
spanning several 256-point blocks with ragged tails, NaN holes, 0-5 sweeps,
float32 and float16 normals, and the full-size synthetic frames."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
VERTEX_RTOL = 1e-5


@pytest.fixture(scope="module")
def pl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2007_12065_amd as pl
    return pl


def to_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def say(*a):
    print("[case]", *a, flush=True)


def check(pl, pts, normals, iters):
    import torch
    got = pl.pl_vertex_update(to_dev(pts), to_dev(normals), iters)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    want = oracle.vertex_update(pts.astype(np.float64), normals.astype(np.float64), iters, threads=8)
    bad = np.isnan(pts).any(-1)
    assert np.array_equal(np.isnan(got).any(-1), bad)
    assert np.array_equal(got[bad].view(np.uint32), pts[bad].view(np.uint32))
    ok = ~bad
    rel = np.linalg.norm(got[ok].astype(np.float64) - want[ok], axis=-1) / np.linalg.norm(want[ok], axis=-1)
    assert rel.max() <= VERTEX_RTOL, rel.max()
    return got


@pytest.mark.parametrize("M,N,seed", [(2, 2, 1), (3, 300, 2), (37, 520, 3), (64, 257, 4), (9, 1000, 5),
                                      (70000, 3, 6)])
def test_random_grids(pl, orc, M, N, seed):
    g = synth.random_grid(M, N, seed, nan_frac=0.1, noise=0.02)
    n, _ = orc.tri_normals(g)
    nf = orc.bilateral(n.astype(np.float32), _.astype(np.float32), 3, 0.1, 0.1, 1).astype(np.float32)
    for iters in (0, 1, 2, 5):
        say("vertex update", M, N, "iters", iters)
        check(pl, g, nf, iters)
    say("vertex update f16", M, N)
    check(pl, g, nf.astype(np.float16), 2)


@pytest.mark.parametrize("kind", ["rgbd", "lidar"])
def test_full_frames(pl, orc, kind):
    k = synth.KINDS[kind]
    p = synth.make_frame(kind, 41)
    r = orc.pipeline(p, k.kernel_lap, k.lam, k.iters_lap, k.kernel_bil, k.sigma_length,
                     k.sigma_angle, k.iters_bil, threads=8)
    pts = r["points"].astype(np.float32)
    nf = r["filtered"].astype(np.float32)
    say("vertex update full", kind)
    check(pl, pts, nf, 3)


@pytest.mark.parametrize("M,N", [(22, 44), (23, 45), (16, 33), (31, 65), (2, 40), (50, 2)])
def test_sweeps_over_launches(pl, orc, M, N):
    """Several sweeps share a launch, whose regions of 32 x 32 points keep 32 - 2 F
    squared: at their edges, in one, two and three launches."""
    g = synth.random_grid(M, N, 7 * M + N, nan_frac=0.1, noise=0.02)
    n, _ = orc.tri_normals(g)
    for iters in (1, 3, 4, 5, 6, 8, 11, 17):
        say("vertex update", M, N, "iters", iters)
        check(pl, g, n.astype(np.float32), iters)


@pytest.mark.parametrize("M,N", [(16, 33), (40, 50), (31, 65), (64, 257), (300, 3)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_points_lost_during_the_sweeps(pl, orc, M, N, dtype):
    """A point that turns NaN in a sweep (infinite coordinates beside it) is a
    missing one from the next sweep on, however the sweeps share launches:
    the oracle's missing and infinite coordinates, finite ones within the
    bound."""
    import torch
    rng = np.random.default_rng(M * N)
    g = synth.random_grid(M, N, 3 * M + N, nan_frac=0.05, noise=0.02).astype(np.float32)
    n, _ = orc.tri_normals(g.astype(np.float64))
    n = n.astype(dtype)
    n[M // 2:, :, :, 0] = np.where(np.isnan(n[M // 2:, :, :, 0]), n[M // 2:, :, :, 0], 0)   # planes along x
    at = rng.choice(M * N, max(2, M * N // 200), replace=False)
    g.reshape(-1, 3)[at, rng.integers(0, 3, len(at))] = rng.choice([np.inf, -np.inf], len(at))
    for iters in (1, 2, 3, 4, 5, 7, 8, 11, 17):
        say("vertex update with infinities", M, N, dtype.__name__, "iters", iters)
        got = pl.pl_vertex_update(to_dev(g), to_dev(n), iters)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        with np.errstate(all="ignore"):
            want = oracle.vertex_update(g.astype(np.float64), n.astype(np.float64), iters)
        assert np.array_equal(np.isnan(got), np.isnan(want)), np.count_nonzero(np.isnan(got) != np.isnan(want))
        inf = np.isinf(want)
        assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
        fin = np.isfinite(want).all(-1)
        rel = np.linalg.norm(got[fin] - want[fin], axis=-1) / np.linalg.norm(want[fin], axis=-1)
        assert rel.max() <= VERTEX_RTOL, rel.max()


@pytest.mark.parametrize("M,N", [(5000, 2), (3, 5000), (8000, 5), (6000, 16), (40, 50)])
def test_narrow_frames(pl, orc, M, N):
    """Frames narrower than a region, and single sweeps of small ones: around
    where a thread per point takes over from the regions."""
    g = synth.random_grid(M, N, M + N, nan_frac=0.1, noise=0.02)
    n, _ = orc.tri_normals(g)
    for iters in (1, 2, 3, 7):
        say("vertex update narrow", M, N, "iters", iters)
        check(pl, g, n.astype(np.float32), iters)
        check(pl, g, n.astype(np.float16), iters)
