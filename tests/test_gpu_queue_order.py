"""The device's queue order of a merged size bucket: every system runs exactly
once, with the result it has for any other order of the call's systems."""
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


def _run(ctx, sizes, P, steps, dt):
    n = len(sizes)
    obs = torch.empty((n, 2, 2), dtype=torch.float32, device="cuda")
    sp = torch.empty(n, dtype=torch.float32, device="cuda")
    st, done = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    swim.swim_forward(ctx, sizes, np.ones(n, np.int32), torch.from_numpy(P).cuda(), steps, dt, 3, 1.5, obs, sp, st, done)
    torch.cuda.synchronize()
    return [v.cpu().numpy() for v in (obs, sp, st, done)]


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("long_runs", ["all", "some", "none"])
def test_any_order_gives_the_same_runs(ctx, n, long_runs):
    rng = np.random.Generator(np.random.PCG64(n))
    sizes = rng.choice([40, 96, 160, 200, 300, 330, 400, 512], n).astype(np.int32)
    plan = swim.swim_forward_plan(swim.SWIM_F32, sizes)
    assert set(plan[(sizes > 256)]) == {8} and np.sum(plan == 8) > 256  # a merged bucket that queues
    P = np.zeros((n, 9))
    lo, hi = {"all": (1e-5, 1e-4), "some": (1e-3, 1.0), "none": (50.0, 100.0)}[long_runs]
    P[:, 0], P[:, 1], P[:, 2], P[:, 3], P[:, 4:6] = rng.uniform(0, 5, n), rng.uniform(lo, hi, n), 1e3, 0.1, 2 * np.pi
    P[:, 6], P[:, 7] = rng.uniform(0, 6, n), -1.0
    steps, dt = 6, 2.5e-6
    a = _run(ctx, sizes, P, steps, dt)
    assert np.all(a[2] >= 0) and np.all(a[3] >= 0) and np.all(a[3] <= steps)
    perm = rng.permutation(n)
    b = _run(ctx, sizes[perm], P[perm], steps, dt)
    for x, y in zip(a, b):
        assert np.array_equal(x[perm], y, equal_nan=True)
