"""The tile-pair path (every pair once, in tiles of 128 points) at sizes around
its thresholds and tile edges: velocity sums against the oracle and against the
one-sided kernel (swim_pair_velocity_noalloc always takes it), and forward
steps of a batch against the same system's alone and in the one-sided step.  Bars: 1e-5 of the norm
per FP32 velocity evaluation against the oracle; two orders of the same FP64
sums of FP32 products, rounded once to FP32, differ by a few 1e-7."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = swim.Context(0)
    yield c
    c.close()


def _systems(sizes, seed, far=False):
    xs, ys, fxs, fys = [], [], [], []
    for k, n in enumerate(sizes):
        rng = np.random.Generator(np.random.PCG64(seed + k))
        s = np.linspace(0.0, 1.0, n)
        x, y = 3.0 * s, 0.1 * np.sin(9.0 * s) + 1e-3 * rng.standard_normal(n)
        if far and n > 3:
            x[n // 2] = 3e6  # beyond the table of eps ~ 1e-3
        fx, fy = rng.standard_normal(n), rng.standard_normal(n)
        xs.append(x), ys.append(y), fxs.append(fx - fx.sum() / max(n, 1)), fys.append(fy - fy.sum() / max(n, 1))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return off, [np.concatenate(v).astype(np.float32) for v in (xs, ys, fxs, fys)]


@pytest.mark.parametrize("sizes,far", [([4096], False), ([4100, 513, 512, 511, 64, 1, 0, 129], False),
                                       ([4097, 700], True), ([4096] * 16, False), ([2100] * 61 + [600], False)])
def test_velocity_tiles(ctx, sizes, far):
    off, arr = _systems(sizes, 3, far)
    n = len(sizes)
    alpha = np.where(np.arange(n) % 3 == 0, 0.0, 0.7 + 0.1 * np.arange(n))
    eps = np.full(n, 1.5e-3)
    dev = [torch.from_numpy(a).cuda() for a in arr]
    u, v, u1, v1 = (torch.full_like(dev[0], float("nan")) for _ in range(4))
    swim.swim_pair_velocity(ctx, off, alpha, eps, *dev, u, v)
    swim.swim_pair_velocity_noalloc(ctx, off, alpha, eps, *dev, u1, v1)
    torch.cuda.synchronize()
    g = [t.double().cpu().numpy() for t in (u, v, u1, v1)]
    for s in range(n):
        p = slice(off[s], off[s + 1])
        for a, b in ((g[0], g[2]), (g[1], g[3])):
            if sizes[s] > 0:
                err = np.linalg.norm(a[p] - b[p]) / max(np.linalg.norm(b[p]), 1e-30)
                assert err < 2e-6, (s, sizes[s], err)
    # the oracle at a few targets of the first system in the Stokes limit (closed forms)
    s, at = 0, np.array([0, 63, 64, 127, 128, sizes[0] // 2, sizes[0] - 2, sizes[0] - 1])
    p = slice(off[s], off[s + 1])
    with core.paper_blob():
        ru, rv = core.velocity_at(*(a[p].astype(np.float64) for a in arr), alpha[s], eps[s], at)
    scale = np.hypot(np.linalg.norm(g[0][p]), np.linalg.norm(g[1][p])) / np.sqrt(sizes[0])
    assert np.max(np.abs(g[0][p][at] - ru)) < 1e-5 * scale and np.max(np.abs(g[1][p][at] - rv)) < 1e-5 * scale


@pytest.mark.parametrize("N,nsw,n_sys", [(257, 2, 150), (512, 8, 16)])
def test_forward_steps(ctx, N, nsw, n_sys):
    """A system's run is the same in any batch, and that of the one-sided step."""
    P = np.zeros((n_sys, nsw, 9))
    rng = np.random.Generator(np.random.PCG64(4))
    P[:, :, 0] = rng.uniform(0, 5, n_sys)[:, None]
    P[:, :, 1], P[:, :, 2], P[:, :, 3], P[:, :, 4:6] = 0.005, 1e3, 0.1, 2 * np.pi
    P[:, :, 6] = rng.uniform(0, 6, (n_sys, nsw))
    P[:, :, 7] = 1.5 * np.arange(nsw) - 1.0

    def run(k):
        obs = torch.empty((k * nsw, 2, 2), dtype=torch.float32, device="cuda")
        sp = torch.empty(k * nsw, dtype=torch.float32, device="cuda")
        st = torch.empty(k, dtype=torch.int32, device="cuda")
        Pd = torch.from_numpy(P[:k].reshape(-1, 9).copy()).cuda()
        swim.swim_forward(ctx, np.full(k, N, np.int32), np.full(k, nsw, np.int32), Pd, 6, 2.5e-6, 3, 1.5, obs, sp, st)
        torch.cuda.synchronize()
        assert torch.all(st == 0)
        return obs.cpu().numpy()[:nsw], sp.cpu().numpy()[:nsw]
    (o1, s1), (o3, s3) = run(n_sys), run(1)
    assert np.array_equal(o1, o3) and np.array_equal(s1, s3)
    swim.swim_set_option(ctx, swim.SWIM_OPT_BIG_TPL, 1)
    try:
        o2, s2 = run(1)
    finally:
        swim.swim_set_option(ctx, swim.SWIM_OPT_BIG_TPL, 0)
    assert np.linalg.norm(o1 - o2) <= 1e-6 * np.linalg.norm(o2)
    # displacements of ~1e-5: one rounding of positions near 1.5 m is 1e-2 of
    # them, so speeds are compared for the swimmer whose head starts at 0
    assert abs(s1[0] - s2[0]) <= 1e-4 * abs(s2[0])
