"""FP64 flow fields on both sides of the rule that takes closed forms directly
(alpha = 0, or fewer than 32 forces with the reading's blob) or from the system's
table: against the oracle with test_gpu_field's bar (1e-12 of the field's norm,
targets near contact and beyond the tables among them), and a target's bits the
same whatever the others."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu


def _field(blob, alpha, eps, src, tgt):
    ctx = swim.Context(0)
    swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, blob)
    s, t = ([torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in q] for q in (src, tgt))
    out = [torch.full_like(t[0], float("nan")) for _ in range(3)]
    swim.swim_flow_field(ctx, *s, alpha, eps, *t, *out)
    out = [o.cpu().numpy() for o in out]
    ctx.close()
    return out


@pytest.mark.parametrize("blob", [swim.SWIM_BLOB_READING, swim.SWIM_BLOB_PAPER])
@pytest.mark.parametrize("n,alpha", [(1, 0.0), (1, 2.0), (31, 2.0), (32, 2.0), (31, 0.0), (300, 0.0)])
def test_closed_forms_and_tables(blob, n, alpha):
    rng = np.random.Generator(np.random.PCG64(n))
    src = [rng.uniform(0, 1, n), rng.uniform(0, 0.2, n), rng.normal(size=n), rng.normal(size=n)]
    eps, nt = 0.02, 300
    tx, ty = rng.uniform(-0.5, 1.5, nt), rng.uniform(-0.5, 0.7, nt)
    k = rng.integers(0, n, 40)
    tx[:40], ty[:40] = src[0][k] + 1e-4 * rng.normal(size=40) * (np.arange(40) > 9), src[1][k]
    tx[40], ty[41] = 3e5, -2e6  # beyond r = 2^21 eps
    got = _field(blob, alpha, eps, src, (tx, ty))
    if blob == swim.SWIM_BLOB_PAPER:
        with core.paper_blob():
            ref = core.field(*src, alpha, eps, tx, ty)
    else:
        with core.reading_blob():
            ref = core.field(*src, alpha, eps, tx, ty)
    for g, r in zip(got, ref):
        assert np.linalg.norm(g - r) <= 1e-12 * np.linalg.norm(r)
    part = _field(blob, alpha, eps, src, (tx[30:50], ty[30:50]))
    for g, p in zip(got, part):
        assert np.array_equal(g[30:50], p)


def test_no_forces():
    z = np.zeros(0)
    for alpha in (0.0, 2.0):
        for o in _field(swim.SWIM_BLOB_READING, alpha, 0.02, (z, z, z, z), (np.ones(3), np.ones(3))):
            assert np.array_equal(o, np.zeros(3))
