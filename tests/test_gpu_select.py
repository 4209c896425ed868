"""Stream compaction (swim_select) at the edges of its spans and blocks, and
beyond the size from which a wave's span grows: the kept indices are numpy's."""
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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 4095, 4096, 4097, 262145, (1 << 22) + 1, 9000001])
@pytest.mark.parametrize("frac", [0.0, 0.03, 1.0])
def test_select_matches_nonzero(ctx, n, frac):
    rng = np.random.Generator(np.random.PCG64(n))
    v = (rng.uniform(size=n) < frac).astype(np.int32)
    # an odd address for the flags
    keep = torch.zeros(n + 1, dtype=torch.uint8, device="cuda")[1:]
    idx = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    nk = torch.zeros(1, dtype=torch.int64, device="cuda")
    swim.swim_select(ctx, keep, idx, nk, values=torch.from_numpy(v).cuda(), want=1)
    torch.cuda.synchronize()
    ref = np.flatnonzero(v)
    got = idx.cpu().numpy()
    assert nk.item() == len(ref)
    assert np.array_equal(got[:len(ref)], ref) and np.all(got[len(ref):] == -1)
