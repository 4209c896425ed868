"""FP32 runs on the finer table pieces in LDS: runs that start beyond the pieces'
reach, or leave it on the way, go on with the whole table.  Against the oracle
with test_gpu_parity's trajectory bars (the first swimmer lies at the origin,
where FP32 outputs resolve its way), and bit for bit the same in a batch that
shares CUs (another build of the pair loop)."""
import math

import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("reading_blob_module")]

torch = pytest.importorskip("torch")

import test_gpu_parity as tgp  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

ctx = tgp.ctx


def _reach(N):
    """distance from the origin, in units of length, that the pieces cover"""
    return 23000.0 / 2.0 ** math.ceil(math.log2((N - 1) / 1.5))


@pytest.mark.parametrize("N,n", [(32, 600), (64, 600), (128, 1), (150, 300)])
@pytest.mark.parametrize("where", ["inside", "beyond", "leaving"])
def test_reach(ctx, oracle_core, N, n, where):
    n_swim = 1 if N == 128 else 2
    R = _reach(N)
    P1 = inputs.param_rows(n_swim, Sb=0.01, Ss=100.0, x0=-1.0)
    P1[:, 0] = 1.3
    if n_swim == 2:
        P1[1, 6] = 1.1
        # the last FP32 value within the reach: the beat carries points over it
        P1[1, 8] = {"inside": 0.4 * R, "beyond": 1.3 * R, "leaving": np.nextafter(np.float32(R), np.float32(0))}[where]
    steps, dt, every = 60, 2e-6, 20
    one = tgp.run_forward(ctx, swim.SWIM_F32, [N], [n_swim], P1, steps, dt, every)
    ref = oracle_core.forward(P1, N, steps, dt, every)
    assert one[2][0] == 0 and ref["status"] == 0
    for m in range(n_swim):
        tgp.check_traj(one[0][m], ref["obs"][m], np.array([0.0, P1[m, 8]]), 1e-4, swim.SWIM_F32, steps,
                       max(1.0, abs(P1[m, 8])))
    many = tgp.run_forward(ctx, swim.SWIM_F32, [N] * n, [n_swim] * n, np.tile(P1, (n, 1)), steps, dt, every)
    assert np.all(many[2] == 0)
    wps = {32: 4, 150: 8}.get(N, 8) if n > 256 else None
    if N in (64, 128):  # the same number of waves at either load
        assert np.array_equal(many[0], np.tile(one[0], (n, 1, 1)))
    else:
        swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, wps)
        try:
            one = tgp.run_forward(ctx, swim.SWIM_F32, [N], [n_swim], P1, steps, dt, every)
        finally:
            swim.swim_set_option(ctx, swim.SWIM_OPT_WPS, 0)
        assert np.array_equal(many[0], np.tile(one[0], (n, 1, 1)))


@pytest.mark.parametrize("N", [64, 150])
def test_blowup_keeps_its_status(ctx, N):
    """A step far beyond the stability bound: positions pass the pieces' reach
    (and the run bound) within a few steps."""
    P = inputs.param_rows(4, Sb=50.0, Ss=1e3, x0=-1.0)
    obs, speed, st = tgp.run_forward(ctx, swim.SWIM_F32, [N] * 4, None, P, 200, 2.5e-5, 10)
    assert np.all((st == 1) | (st == 2)) and np.all(np.isnan(speed))
