"""The untuned number of waves per system, at the batch sizes where it changes
(one and two systems per compute unit) and in a call of two size classes: the
run has to be, bit for bit, the run with that number set explicitly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu
CU = 256


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != CU:
        pytest.skip("thresholds below are for 256 compute units")
    c = swim.Context(0)
    yield c
    c.close()


def _run(ctx, sizes, dtype, wps):
    n = len(sizes)
    rng = np.random.Generator(np.random.PCG64(1))
    P = np.zeros((n, 9))
    P[:, 0], P[:, 1], P[:, 2], P[:, 3], P[:, 4:6] = rng.uniform(0, 5, n), 0.002, 1e3, 0.1, 2 * np.pi
    P[:, 6], P[:, 7] = rng.uniform(0, 6, n), -1.0
    obs = torch.empty((n, 2, 2), dtype=dtype, device="cuda")
    sp = torch.empty(n, dtype=dtype, device="cuda")
    st = torch.empty(n, dtype=torch.int32, device="cuda")
    swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, wps)
    try:
        swim.swim_forward(ctx, np.asarray(sizes, np.int32), np.ones(n, np.int32), torch.from_numpy(P).cuda(), 6, 2.5e-6,
                          3, 1.5, obs, sp, st)
        torch.cuda.synchronize()
    finally:
        swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, 0)
    assert torch.all(st == 0) and torch.isfinite(obs).all()
    return obs.cpu().numpy(), sp.cpu().numpy()


@pytest.mark.parametrize("N,n_sys,dtype,wps", [
    (64, 2 * CU, torch.float32, 8), (64, 2 * CU + 1, torch.float32, 4), (40, 1, torch.float32, 8),
    (128, 2 * CU + 1, torch.float32, 8), (129, CU, torch.float32, 16), (129, CU + 1, torch.float32, 8),
    (384, CU + 1, torch.float32, 8), (385, CU + 1, torch.float32, 16), (64, 2 * CU + 1, torch.float64, 8)])
def test_untuned_waves(ctx, N, n_sys, dtype, wps):
    a, b = _run(ctx, [N] * n_sys, dtype, 0), _run(ctx, [N] * n_sys, dtype, wps)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_untuned_waves_two_classes(ctx):
    sizes = [129] * (2 * CU) + [64] * CU
    small = np.arange(len(sizes)) >= 2 * CU
    a, e16, e8 = (_run(ctx, sizes, torch.float32, w) for w in (0, 16, 8))
    for k in range(2):
        assert np.array_equal(a[k][~small], e16[k][~small]) and np.array_equal(a[k][small], e8[k][small])
