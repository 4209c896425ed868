"""FP64 velocity sums on both sides of the size (24 points) up to which closed forms
are evaluated directly: against the oracle with the library's FP64 bar (1e-12 of the
velocities' norm), and each system's bits the same alone, among systems with tables,
and without scratch memory."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_1910_12007_amd import swim  # noqa: E402

pytestmark = pytest.mark.gpu


def _call(fn, ctx, systems, alpha):
    off = np.concatenate([[0], np.cumsum([len(s[0]) for s in systems])]).astype(np.int64)
    d = [torch.from_numpy(np.concatenate([s[k] for s in systems])).cuda() for k in range(4)]
    u, v = torch.full_like(d[0], np.nan), torch.full_like(d[0], np.nan)
    fn(ctx, off, alpha, [0.05] * len(systems), *d, u, v)
    torch.cuda.synchronize()
    return [np.stack([u.cpu().numpy()[a:b], v.cpu().numpy()[a:b]]) for a, b in zip(off, off[1:])]


@pytest.mark.parametrize("blob", [swim.SWIM_BLOB_READING, swim.SWIM_BLOB_PAPER])
def test_direct_and_tables(blob):
    ctx = swim.Context(0)
    swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, blob)
    rng = np.random.Generator(np.random.PCG64(4))
    sizes, alpha = [1, 3, 8, 23, 24, 25, 70, 24, 25, 24], [0.0, 2.0, 0.0, 2.0, 0.0, 0.0, 1.0, 2.0, 2.0, 0.0]
    systems = [[rng.uniform(0, 1, n), rng.uniform(0, 0.2, n), rng.normal(size=n), rng.normal(size=n)] for n in sizes]
    systems[9][0][3] = 3e6  # a pair beyond r = 2^21 eps
    out = _call(swim.swim_pair_velocity, ctx, systems, alpha)
    na = _call(swim.swim_pair_velocity_noalloc, ctx, systems, alpha)
    for s, a, u, w in zip(systems, alpha, out, na):
        assert np.all(np.isfinite(u)) and np.array_equal(u, w)
        assert np.array_equal(u, _call(swim.swim_pair_velocity, ctx, [s], [a])[0])
        with (core.paper_blob() if blob == swim.SWIM_BLOB_PAPER else core.reading_blob()):
            ref = np.stack(core.velocity(*s, a, 0.05))
        assert np.linalg.norm(u - ref) <= 1e-12 * np.linalg.norm(ref)
    ctx.close()


def test_more_systems_than_a_table_chunk():
    """Closed forms, 3 points a system: one call without tables; the same with one
    system of 25 points, in chunks with tables."""
    ctx = swim.Context(0)
    rng = np.random.Generator(np.random.PCG64(6))
    s = [rng.uniform(0, 1, 3) for _ in range(4)]
    big = [rng.uniform(0, 1, 25) for _ in range(4)]
    n = 20000
    a = _call(swim.swim_pair_velocity, ctx, [s] * n, [0.0] * n)
    b = _call(swim.swim_pair_velocity, ctx, [s] * n + [big], [0.0] * (n + 1))
    assert all(np.array_equal(a[0], q) for q in a + b[:-1])
    assert np.array_equal(b[-1], _call(swim.swim_pair_velocity, ctx, [big], [0.0])[0])
    ctx.close()
