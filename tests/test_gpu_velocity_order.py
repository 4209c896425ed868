"""One system's velocity sum has the same bits whatever kernel and call it is part
of: swim_pair_velocity and swim_pair_velocity_noalloc, alone or among others, with
tile pairs (from 1024 points, from 512 in calls of 2^24 pairs) or one-sided, at the
edges of tiles (128), blocks (64) and rounds (512), with pairs beyond the table; and
the FP64 sum of the same inputs to a few FP32 roundings of the kernel values
(1e-6 of the velocities' norm)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = swim.Context(0)
    yield c
    c.close()


def _system(n, seed, far=False):
    rng = np.random.Generator(np.random.PCG64(seed))
    a = [rng.uniform(0, 1, n), rng.uniform(0, 0.3, n), rng.normal(size=n), rng.normal(size=n)]
    if far:  # every 7th point 1e7 away: beyond r = 2^21 eps
        a[0][::7] += 1e7
    return [v.astype(np.float32) for v in a]


def _call(fn, ctx, systems, alpha, eps, dtype=torch.float32):
    off = np.concatenate([[0], np.cumsum([len(s[0]) for s in systems])]).astype(np.int64)
    d = [torch.from_numpy(np.concatenate([s[k] for s in systems])).cuda().to(dtype) for k in range(4)]
    u, v = torch.full_like(d[0], np.nan), torch.full_like(d[0], np.nan)
    fn(ctx, off, alpha, eps, *d, u, v)
    torch.cuda.synchronize()
    return [np.stack([u.cpu().numpy()[a:b], v.cpu().numpy()[a:b]]) for a, b in zip(off, off[1:])]


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("n", [64, 511, 512, 513, 577, 640, 1000, 1023, 1024, 1025, 1088, 1153, 2100, 4096])
def test_same_bits_in_every_call(ctx, n, far):
    s, alpha, eps = _system(n, n, far), 1.7, 1.5 / (n - 1)
    one = _call(swim.swim_pair_velocity, ctx, [s], [alpha], [eps])[0]
    assert np.all(np.isfinite(one))
    na = _call(swim.swim_pair_velocity_noalloc, ctx, [s], [alpha], [eps])[0]
    assert np.array_equal(one, na)
    # among others, in a call of more than 2^24 pairs
    other = _system(4200, 1)
    many = _call(swim.swim_pair_velocity, ctx, [other, s, other], [0.5, alpha, 0.0], [1e-3, eps, 1e-3])
    assert np.array_equal(one, many[1])
    many = _call(swim.swim_pair_velocity_noalloc, ctx, [other, s, s], [0.5, alpha, alpha], [1e-3, eps, eps])
    assert np.array_equal(one, many[1]) and np.array_equal(one, many[2])
    if not far:
        ref = _call(swim.swim_pair_velocity, ctx, [s], [alpha], [eps], torch.float64)[0]
        assert np.linalg.norm(one - ref) <= 1e-6 * np.linalg.norm(ref)


def test_systems_past_the_partial_sums_limit(ctx):
    """512 systems of 4096 points want 8 GiB of partial sums: those past the first
    GiB are summed one-sided, to the same bits."""
    n, n_sys = 4096, 520
    s = _system(n, 5)
    out = _call(swim.swim_pair_velocity, ctx, [s] * n_sys, [1.7] * n_sys, [1.5 / (n - 1)] * n_sys)
    for k in (1, 300, n_sys - 1):
        assert np.array_equal(out[0], out[k])


def test_more_systems_than_a_chunk(ctx):
    n_sys, n = 262144 + 70, 3
    rng = np.random.Generator(np.random.PCG64(3))
    base = [rng.uniform(0, 1, 3).astype(np.float32) for _ in range(4)]
    off = np.arange(n_sys + 1, dtype=np.int64) * n
    d = [torch.from_numpy(np.tile(v, n_sys)).cuda() for v in base]
    u, v = torch.full_like(d[0], np.nan), torch.full_like(d[0], np.nan)
    swim.swim_pair_velocity(ctx, off, np.full(n_sys, 0.4), np.full(n_sys, 0.5), *d, u, v)
    for q in (u, v):
        q = q.cpu().numpy().reshape(n_sys, n)
        assert np.all(np.isfinite(q)) and np.array_equal(q, np.tile(q[0], (n_sys, 1)))


def test_same_bits_where_forces_cancel(ctx):
    """Forces of alternating sign between close points, as stretched filaments have:
    the velocities are a small rest of their terms, so that another order of the
    FP64 sums shows in the last FP32 bit of a few of 524288 values."""
    n, n_sys = 4096, 64
    rng = np.random.Generator(np.random.PCG64(8))
    systems = []
    for _ in range(n_sys):
        T = 1e4 * rng.standard_normal((2, n + 1))
        T[:, 0] = T[:, -1] = 0.0
        systems.append([v.astype(np.float32) for v in
                        (np.linspace(0, 1, n), 0.1 * np.sin(np.linspace(0, 6, n)), *(T[:, 1:] - T[:, :-1]))])
    alpha, eps = rng.uniform(0.1, 5, n_sys), np.full(n_sys, 1.5 / (n - 1))
    a, b = (_call(f, ctx, systems, alpha, eps) for f in (swim.swim_pair_velocity, swim.swim_pair_velocity_noalloc))
    assert sum(int(np.sum(p != q)) for p, q in zip(a, b)) == 0
