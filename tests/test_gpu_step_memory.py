"""Device memory of an ABC step: what grows with the draws beyond a chunk of forward
runs (262144) is one copy of each per-draw array, rows of parameters among them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1910_12007_amd import swim  # noqa: E402
from paper_1910_12007_amd import surrogate_abc as sa  # noqa: E402

pytestmark = pytest.mark.gpu


def test_rows_take_memory_once():
    model = sa.batch_model(steps=1, dt=1e-7, obs_every=1)
    data = np.array([[1.0, 0.0]])
    ctx = swim.Context(0)
    swim.swim_set_option(ctx, swim.SWIM_OPT_BLOB, swim.SWIM_BLOB_READING)
    used = []
    n0, n1 = 262144, 1 << 20
    for n in (n0, n1):
        swim.abc_step(ctx, model, data, np.full(n, 3, np.int32), 1, 0, 0.5)
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        used.append(total - free)
    ctx.close()
    # rows, observations, speed, status, distance, accept, steps: bytes per draw,
    # allocated with a quarter to spare, in 2 MiB pages
    per_draw = 72 + 8 + 4 + 4 + 8 + 1 + 4
    grown = used[1] - used[0]
    assert grown <= 1.25 * per_draw * (n1 - n0) + 8 * (2 << 20), grown
