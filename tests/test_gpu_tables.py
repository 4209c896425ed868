"""Kernel tables against the oracle's kernel functions, value by value: systems
of two points at one distance each, from contact to beyond the table, with the
force on the second point only, so that the first one's velocity is the kernel
itself.  Tolerances follow from the tables' construction: an FP64 table is
good to a few roundings of H1(0) (the bar of every FP64 velocity, 1e-12), an
FP32 one to the 1e-6 (Ht) and 5e-6 (H2) of its cubic pieces."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = swim.Context(0)
    yield c
    c.close()


def _two_point(ctx, alpha, eps, r, dt):
    n = len(r)
    x = np.zeros(2 * n)
    x[1::2] = r
    fx, fy = np.zeros(2 * n), np.zeros(2 * n)
    fx[1::2], fy[1::2] = 0.6, 0.8
    dev = [torch.from_numpy(a).to("cuda", dt) for a in (x, np.zeros(2 * n), fx, fy)]
    u, v = torch.empty_like(dev[0]), torch.empty_like(dev[0])
    off = np.arange(n + 1) * 2
    swim.swim_pair_velocity(ctx, off, np.full(n, alpha), np.full(n, eps), *dev, u, v)
    torch.cuda.synchronize()
    return u.double().cpu().numpy()[::2], v.double().cpu().numpy()[::2], dev[0].double().cpu().numpy()[1::2]


# alpha = 0, alpha -> 0, both sides of every switch (series, alpha r = 2, 8,
# 40, 316), alpha eps = 1
@pytest.mark.parametrize("alpha,eps", [(0.0, 0.02), (1e-4, 0.02), (2.0, 0.0118), (10.0, 0.0238), (25.0, 0.04)])
@pytest.mark.parametrize("blob", [swim.SWIM_BLOB_PAPER, swim.SWIM_BLOB_READING])
def test_table_values_match_oracle(ctx, alpha, eps, blob):
    d = np.array([1e-3, 0.1, 0.49, 0.499999, 0.500001, 0.51, 0.7, 1.0, 1.5, 3.0, 20.0, 400.0])
    z = np.array([1.99, 2.01, 7.9, 8.1, 39.9, 40.1, 41.5, 79.0, 81.0, 315.0, 317.0]) / max(alpha, 1e-300)
    far = np.array([2.0 ** 21 * 0.9, 2.0 ** 23]) * eps  # the last octaves, and beyond the table
    r = np.concatenate([eps * d, z[(z > 0.5 * eps) & (z < 900.0)], far])
    swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, blob)
    try:
        got = {dt: _two_point(ctx, alpha, eps, r, dt) for dt in (torch.float64, torch.float32)}
    finally:
        swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, swim.SWIM_BLOB_PAPER)
    for dt, (u, v, rr) in got.items():
        with (core.paper_blob() if blob == swim.SWIM_BLOB_PAPER else core.reading_blob()):
            H1, H2 = core.kernel(alpha, eps, rr * rr)
            h0 = core.kernel(alpha, eps, np.zeros(1))[0][0]
        scale = abs(h0) + np.abs(H1)
        bar = 1e-12 if dt == torch.float64 else 6e-6
        eu = np.abs(u - 0.6 * (H1 + H2 * rr * rr)) / scale
        ev = np.abs(v - 0.8 * H1) / scale
        print(alpha, eps, blob, dt, eu.max(), ev.max())
        assert eu.max() <= bar and ev.max() <= bar, (dt, eu, ev)


def test_fp64_batches_beyond_one_chunk(ctx):
    """More FP64 systems than tables are kept for at once run in chunks: the
    systems at the chunk's ends give what a call of their own gives."""
    n, N = 16384 + 3, 5
    rng = np.random.Generator(np.random.PCG64(7))
    pick = np.array([0, 16383, 16384, n - 1])
    al, e = rng.uniform(0.1, 5.0, n), np.full(n, 1.5 / (N - 1))
    arr = [rng.uniform(-1, 1, n * N) for _ in range(4)]

    def run(idx):
        p = (idx[:, None] * N + np.arange(N)).ravel()
        dev = [torch.from_numpy(a[p]).cuda() for a in arr]
        u, v = torch.empty_like(dev[0]), torch.empty_like(dev[0])
        swim.swim_pair_velocity(ctx, np.arange(len(idx) + 1) * N, al[idx] * 0.1, e[idx], *dev, u, v)
        P = np.zeros((len(idx), 9))
        P[:, 0], P[:, 1], P[:, 2], P[:, 3], P[:, 4:6] = al[idx] * 0.1, 0.1, 100.0, 0.1, 2 * np.pi
        obs = torch.empty((len(idx), 1, 2), dtype=torch.float64, device="cuda")
        sp = torch.empty(len(idx), dtype=torch.float64, device="cuda")
        st = torch.empty(len(idx), dtype=torch.int32, device="cuda")
        swim.swim_forward(ctx, np.full(len(idx), N, np.int32), None, torch.from_numpy(P).cuda(), 3, 1e-4, 3, 1.5, obs,
                          sp, st)
        sh = swim.sperm_shape(4, 4, 1, 0.2)
        S = np.tile([1.0, 8.0, 1e2, 1e2, 0.8, 50.0, 1e2, 0.1, 6.28, 12.57], (len(idx), 1))
        S[:, 0] = al[idx] * 0.1
        hd = torch.empty((len(idx), 2, 2), dtype=torch.float64, device="cuda")
        tl = torch.empty_like(hd)
        ss = torch.empty(len(idx), dtype=torch.int32, device="cuda")
        swim.swim_sperm_forward(ctx, swim.SWIM_F64, sh, torch.from_numpy(S).cuda(),
                                torch.zeros((len(idx), 3), dtype=torch.float64, device="cuda"), 2, 1e-5, 2, hd, tl, ss)
        torch.cuda.synchronize()
        return [a.cpu().numpy().reshape(len(idx), -1) for a in (u, v, obs, sp, st, hd, tl, ss)]
    whole, few = run(np.arange(n)), run(pick)
    for a, b in zip(whole, few):
        assert np.array_equal(a[pick], b)
        assert np.all(np.isfinite(a))
