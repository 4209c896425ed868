"""The untuned number of waves per system, and with it the order of a run's FP32 sums,
is chosen once per call: a run's bits do not depend on its place in a batch that
is larger than a chunk (262144 systems), and abc_prescreened's re-runs have the bits
of abc_step's runs of all the draws, however few survive."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import swim  # noqa: E402
from paper_1910_12007_amd import surrogate_abc as sa  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = swim.Context(0)
    swim.swim_set_option(c, swim.SWIM_OPT_BLOB, swim.SWIM_BLOB_READING)
    yield c
    c.close()


@pytest.mark.parametrize("N,n_prop", [(40, 1100), (150, 700), (128, 700)])
def test_reruns_have_the_plain_runs_bits(ctx, N, n_prop):
    # stable steps, so that every run completes
    model = sa.batch_model(steps=60, dt=1e-6, obs_every=10)
    rng = np.random.Generator(np.random.PCG64(2))
    data = np.stack([1.0 + 1e-3 * rng.normal(size=6), 1e-3 * rng.normal(size=6)], 1)
    plain = swim.abc_step(ctx, model, data, np.full(n_prop, N, np.int32), 9, 0, 0.5)
    p = torch.zeros(207393, dtype=torch.float32, device="cuda")
    z5, o5, z33, o33 = (torch.full((n,), v, dtype=torch.float32, device="cuda") for n, v in ((5, 0.), (5, 1.), (33, 0.), (33, 1.)))
    cap = 30
    # every draw survives a surrogate that predicts no motion; the first 30 are re-run
    out = swim.abc_prescreened(ctx, model, N, p, z5, o5, z33, o33, np.arange(16) % 6, data, 1.0, 10.0, n_prop, 9, cap)
    theta, dist = out["theta"][:cap], out["dist"][:cap]
    assert np.array_equal(theta, plain["theta"][:cap]) and np.all(np.isfinite(dist))
    assert np.array_equal(dist, plain["dist"][:cap])


def test_bits_do_not_follow_the_chunk(ctx):
    n, N = 262144 + 9, 64
    P = np.zeros((1, 9))
    P[0, :8] = (1.3, 0.01, 300.0, 0.1, 2 * np.pi, 2 * np.pi, 0.3, -1.0)
    rows = torch.from_numpy(P).cuda().repeat(n, 1)
    obs = torch.empty((n, 2, 2), dtype=torch.float32, device="cuda")
    speed = torch.empty(n, dtype=torch.float32, device="cuda")
    st = torch.empty(n, dtype=torch.int32, device="cuda")
    swim.swim_forward(ctx, np.full(n, N, np.int32), None, rows, 20, 2e-6, 10, 1.5, obs, speed, st)
    torch.cuda.synchronize()
    assert torch.all(st == 0) and torch.isfinite(obs).all()
    assert torch.equal(obs, obs[:1].expand_as(obs)) and torch.equal(speed, speed[:1].expand_as(speed))
