"""The FP32 field kernel's two launch shapes (one or two targets per thread, from
2^18 targets on), source tiles' remainders and targets beyond the tables."""
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


@pytest.mark.parametrize("n,alpha", [(1, 0.0), (255, 0.0), (257, 3.0), (600, 0.0)])
def test_shapes_agree_and_match_oracle(ctx, n, alpha):
    x, y = inputs.filament_geometry(max(n, 3), 5)
    fx, fy = inputs.force_pattern(max(n, 3), 6)
    src = [torch.from_numpy(a[:n].astype(np.float32)).cuda() for a in (x, y, fx, fy)]
    rng = np.random.Generator(np.random.PCG64(8))
    nt = (1 << 18) + 77
    tx, ty = rng.uniform(-1, 2, nt), rng.uniform(-1, 1, nt)
    tx[5], tx[nt - 1] = 1e6, -3e7  # beyond the tables of eps = 0.002
    tgt = [torch.from_numpy(a.astype(np.float32)).cuda() for a in (tx, ty)]

    def run(k0, k1):
        t = [a[k0:k1].clone() for a in tgt]
        out = [torch.full_like(t[0], float("nan")) for _ in range(3)]
        swim.swim_flow_field(ctx, *src, alpha, 0.002, *t, *out)
        torch.cuda.synchronize()
        return [o.cpu().numpy() for o in out]
    big, head, tail = run(0, nt), run(0, 300), run(nt - 300, nt)
    for b, h, t in zip(big, head, tail):
        assert np.all(np.isfinite(b))
        assert np.array_equal(b[:300], h) and np.array_equal(b[-300:], t)
    if alpha == 0.0:
        at = np.r_[0:8, nt - 8:nt]
        s64 = [a.double().cpu().numpy() for a in src]
        t64 = [a.double().cpu().numpy()[at] for a in tgt]
        with core.paper_blob():
            ref = core.field(*s64, alpha, 0.002, *t64)
        # 1e-5 of the field's scale: the FP32 velocity bar
        near = np.abs(t64[0]) < 10
        for b, r in zip(big, ref):
            assert np.max(np.abs(b[at] - r)[near]) < 1e-5 * np.max(np.abs(r[near]))
            assert np.max(np.abs(b[at] - r)[~near]) < 1e-5 * np.max(np.abs(r))
