"""FP64 runs read their table from the caches below 8 steps and from LDS from 8 steps
on (up to 256 points): the state after 7 steps is the same bits in a run of 7 and in
one of 8, at the edges of the sizes that have both builds, and the runs of 7 match the
oracle with test_gpu_parity's trajectory bar."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("reading_blob_module")]

torch = pytest.importorskip("torch")

import test_gpu_parity as tgp  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

ctx = tgp.ctx


@pytest.mark.parametrize("N,n_swim,n", [(3, 1, 1), (64, 1, 300), (65, 1, 1), (128, 1, 1), (64, 3, 300), (193, 1, 1),
                                        (256, 1, 300), (257, 1, 1)])
def test_caches_and_lds(ctx, oracle_core, N, n_swim, n):
    P = inputs.param_rows(n_swim, Sb=0.01, Ss=100.0, x0=-1.0)
    P[:, 0], P[:, 4], P[:, 6], P[:, 8] = 1.3, 2 * np.pi * (1 + np.arange(n_swim)), 0.3, 0.6 * np.arange(n_swim)
    dt, rows = 2e-6, np.tile(P, (n, 1))
    a = tgp.run_forward(ctx, swim.SWIM_F64, [N] * n, [n_swim] * n, rows, 7, dt, 7)
    b = tgp.run_forward(ctx, swim.SWIM_F64, [N] * n, [n_swim] * n, rows, 8, dt, 7)
    assert np.all(a[2] == 0) and np.all(b[2] == 0)
    assert np.array_equal(a[0], b[0])
    assert np.array_equal(a[0], np.tile(a[0][:n_swim], (n, 1, 1)))
    ref = oracle_core.forward(P, N, 7, dt, 7)
    for m in range(n_swim):
        tgp.check_traj(a[0][m], ref["obs"][m], np.array([0.0, P[m, 8]]), 1e-12, swim.SWIM_F64, 7, 2.0)
