"""FP64 velocity sums in units 2^e times as long (positions and eps scaled, alpha
by the inverse): u = sum H1 F + H2 (F.d) d is the same in every unit, and powers of
two scale exactly.  1e-14 of the velocities' norm, 2^6 roundings, is left to the
hardware's reciprocal estimates."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("e", [-240, -120, 120, 240])
def test_scaled_units(e):
    ctx = swim.Context(0)
    swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, swim.SWIM_BLOB_PAPER)
    rng = np.random.Generator(np.random.PCG64(9))
    n, eps = 40, 1.5 / 39
    a = [rng.uniform(0, 1, n), rng.uniform(0, 0.2, n), rng.normal(size=n), rng.normal(size=n)]
    out = []
    for s in (1.0, 2.0 ** e):
        d = [torch.from_numpy(v * (s if k < 2 else 1.0)).cuda() for k, v in enumerate(a)]
        u, v = torch.empty_like(d[0]), torch.empty_like(d[0])
        swim.swim_pair_velocity(ctx, np.array([0, n], np.int64), [1.3 / s], [eps * s], *d, u, v)
        out.append(np.concatenate([u.cpu().numpy(), v.cpu().numpy()]))
    ctx.close()
    assert np.all(np.isfinite(out[1]))
    assert np.linalg.norm(out[1] - out[0]) <= 1e-14 * np.linalg.norm(out[0])
