"""FP64 sperm runs with the table in LDS (no more systems than compute units, from
8 steps) and in place (all others): the same bits, up to the largest system that
has the first and one beyond.  Values are pinned to the oracle in
test_gpu_sperm.py and test_gpu_sperm_shapes.py, which run the first."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import inputs, swim  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = swim.Context(0)
    yield c
    c.close()


def _run(ctx, nf, nh, nsw, rows, sw, steps):
    head = torch.full((len(rows) * nsw, 2, 2), 7.0, dtype=torch.float64, device="cuda")
    tail = torch.full_like(head, 7.0)
    st = torch.full((len(rows),), -1, dtype=torch.int32, device="cuda")
    swim.swim_sperm_forward(ctx, swim.SWIM_F64, swim.sperm_shape(nf, nh, nsw, 0.045, 0.05, 1.0 / (nf - 1)),
                            torch.from_numpy(rows).cuda(), torch.from_numpy(sw).cuda(), steps, 1e-6, steps, head, tail, st)
    torch.cuda.synchronize()
    return [v.cpu().numpy() for v in (head, tail, st)]


@pytest.mark.parametrize("nf,nh,nsw", [(4, 4, 1), (50, 24, 1), (50, 24, 2), (50, 24, 3), (100, 28, 2), (58, 28, 3)])
@pytest.mark.parametrize("steps", [7, 8])
def test_tables_in_lds_and_in_place(ctx, nf, nh, nsw, steps):
    n = 300
    rows = inputs.sperm_rows(n)
    rows[:, 0] = np.where(np.arange(n) % 2, 0.0, 1.1)  # two kinds of systems in turn
    sw = np.tile(np.stack([np.zeros(nsw), 0.4 * np.arange(nsw), 0.5 * np.arange(nsw)], 1), (n, 1))
    many = _run(ctx, nf, nh, nsw, rows, sw, steps)
    for k in (1, 3):
        few = _run(ctx, nf, nh, nsw, rows[:k], sw[:k * nsw], steps)
        assert np.all(few[2] == 0) and np.all(many[2] == 0)
        for a, b in zip(few[:2], many[:2]):
            assert np.array_equal(a, b[:k * nsw]) and np.array_equal(b[:2 * nsw], b[-2 * nsw:])
