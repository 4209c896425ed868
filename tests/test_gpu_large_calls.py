"""Calls whose launches would pass 2^32 threads, or whose scratch memory grows with the
batch, run in parts: identical systems give identical bits wherever they lie."""
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
    swim.swim_set_option(c, swim.SWIM_OPT_BLOB, swim.SWIM_BLOB_READING)
    yield c
    c.close()
    torch.cuda.empty_cache()


def _same(t):
    assert torch.isfinite(t).all()
    assert torch.equal(t, t[:1].expand_as(t))


def test_large_systems(ctx):
    """32000 systems of 8 x 512 points: 528 tile pairs and 2 MB of partial sums each."""
    n, nsw, N = 32000, 8, 512
    P = np.zeros((nsw, 9))
    P[:, :6] = (1.0, 0.01, 300.0, 0.1, 2 * np.pi, 2 * np.pi)
    P[:, 7], P[:, 8] = 1.5 * (np.arange(nsw) % 4) - 1.0, 1.5 * (np.arange(nsw) // 4)
    rows = torch.from_numpy(P).cuda().repeat(n, 1)
    obs = torch.empty((n * nsw, 1, 2), dtype=torch.float32, device="cuda")
    speed = torch.empty(n * nsw, dtype=torch.float32, device="cuda")
    st = torch.empty(n, dtype=torch.int32, device="cuda")
    swim.swim_forward(ctx, np.full(n, N, np.int32), np.full(n, nsw, np.int32), rows, 2, 2e-7, 2, 1.5, obs, speed, st)
    torch.cuda.synchronize()
    assert torch.all(st == 0)
    _same(obs.view(n, -1))
    _same(speed.view(n, -1))


def test_velocity_of_many_points(ctx):
    """270000 systems of 2048 points (5.5e8 points)."""
    n_sys, n = 270000, 2048
    rng = np.random.Generator(np.random.PCG64(1))
    d = [torch.from_numpy(rng.uniform(-0.5, 0.5, n).astype(np.float32)).cuda().repeat(n_sys) for _ in range(4)]
    u, v = torch.full_like(d[0], float("nan")), torch.full_like(d[0], float("nan"))
    swim.swim_pair_velocity(ctx, np.arange(n_sys + 1, dtype=np.int64) * n, np.full(n_sys, 0.4), np.full(n_sys, 0.01), *d,
                            u, v)
    torch.cuda.synchronize()
    _same(u.view(n_sys, n))
    _same(v.view(n_sys, n))


def test_sperm_systems_beyond_a_chunk(ctx):
    n = 262144 + 9
    shape = swim.sperm_shape(30, 6, 1, 0.045, 0.05)
    P = torch.tensor([[1.0, 8.0, 1e4, 1e4, 0.8, 500.0, 1e4, 0.1, 6.0, 12.0]], dtype=torch.float64, device="cuda").repeat(n, 1)
    W = torch.tensor([[0.0, 0.0, 0.3]], dtype=torch.float64, device="cuda").repeat(n, 1)
    head = torch.empty((n, 2, 2), dtype=torch.float32, device="cuda")
    tail = torch.empty_like(head)
    st = torch.empty(n, dtype=torch.int32, device="cuda")
    swim.swim_sperm_forward(ctx, swim.SWIM_F32, shape, P, W, 20, 1e-5, 20, head, tail, st)
    torch.cuda.synchronize()
    assert torch.all(st == 0)
    _same(head)
    _same(tail)
