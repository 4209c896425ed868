"""The sperm run's schedules at their edges, against the FP64 oracle with the
bars of test_gpu_sperm: points beyond the last full block (16 and 32 are where
the lane groups of the pairs among them change, 20 and 37 the most taken point
by point), more waves than points need, and systems that keep only the first
octaves of their FP32 table on chip while pairs lie beyond them."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("reading_blob_module")]

torch = pytest.importorskip("torch")

import test_gpu_sperm as tgs  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

EPS, HR = tgs.EPS, tgs.HR
ctx = tgs.ctx


def _run(ctx, dtype, nf, nh, nsw, rows, sw, steps, dt, oe):
    td = tgs.TD[dtype]
    head = torch.empty((len(rows) * nsw, steps // oe + 1, 2), dtype=td, device="cuda")
    tail = torch.empty_like(head)
    st = torch.empty(len(rows), dtype=torch.int32, device="cuda")
    swim.swim_sperm_forward(ctx, dtype, swim.sperm_shape(nf, nh, nsw, EPS, HR, 1.0 / (nf - 1)),
                            torch.from_numpy(rows).cuda(), torch.from_numpy(sw).cuda(), steps, dt, oe, head, tail, st)
    torch.cuda.synchronize()
    assert torch.all(st == 0)
    return head.cpu().double().numpy(), tail.cpu().double().numpy()


@pytest.mark.parametrize("dtype", [swim.SWIM_F64, swim.SWIM_F32])
@pytest.mark.parametrize("wps", [2, 8])
@pytest.mark.parametrize("nf,nh", [(8, 8), (9, 8), (12, 8), (13, 8), (56, 24), (57, 24), (72, 24), (73, 24), (77, 24),
                                   (78, 24), (40, 24)])
def test_points_beyond_the_last_block(ctx, oracle_core, nf, nh, wps, dtype):
    steps, dt, oe = 20, 2e-6, 10
    dn = 1.0 / (nf - 1)
    rows = inputs.sperm_rows(1, alpha=0.9, KC=5.0)
    sw = inputs.sperm_swimmers(1)
    swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, wps)
    try:
        head, tail = _run(ctx, dtype, nf, nh, 1, rows, sw, steps, dt, oe)
    finally:
        swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, 0)
    ref = oracle_core.sperm_forward(rows[0], sw, nf, nh, EPS, HR, dn, steps, dt, oe)
    assert ref["status"] == 0
    path = tgs.oracle_velocity_path_shape(oracle_core, rows[0], sw, nf, nh, dn, steps, dt)
    tgs.check(dtype, head, ref["head"], path, steps, "head")
    tgs.check(dtype, tail, ref["tail"], path, steps, "tail")


@pytest.mark.parametrize("d", [0.5, 230.0])
def test_pairs_beyond_the_octaves_on_chip(ctx, oracle_core, d):
    """1300 systems of two swimmers d apart: more than fit the GPU with whole
    tables.  d = 230 is 5111 blob widths, beyond the 4096 of the first octaves."""
    n, steps, dt, oe = 1300, 10, 1e-5, 5
    rows = inputs.sperm_rows(n)
    rows[:, 0] = np.linspace(0.0, 2.0, n)
    sw = np.tile(np.array([[0.0, 0.0, 0.2], [0.0, d, 1.4]]), (n, 1))
    head, tail = _run(ctx, swim.SWIM_F32, tgs.NF, tgs.NH, 2, rows, sw, steps, dt, oe)
    for s in (0, 1, 700, n - 1):
        ref = tgs.oracle_run(oracle_core, rows[s], sw[:2], steps, dt, oe)
        tgs.check(swim.SWIM_F32, head[2 * s:2 * s + 2], ref["head"], None, steps, "head")
        tgs.check(swim.SWIM_F32, tail[2 * s:2 * s + 2], ref["tail"], None, steps, "tail")
        alone = _run(ctx, swim.SWIM_F32, tgs.NF, tgs.NH, 2, rows[s:s + 1], sw[:2], steps, dt, oe)
        for a, b in zip(alone, (head, tail)):
            tgs.check(swim.SWIM_F32, b[2 * s:2 * s + 2], a, None, steps, "alone")
