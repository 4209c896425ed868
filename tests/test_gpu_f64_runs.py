"""FP64 runs with the table in LDS (launches whose workgroups share no CU, from 8
steps) and from the caches (all others): the same bits, at the edges of the
sizes that have the first, with one and three filaments, and against the oracle
with test_gpu_parity's trajectory bar."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("reading_blob_module")]

torch = pytest.importorskip("torch")

import test_gpu_parity as tgp  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

ctx = tgp.ctx


@pytest.mark.parametrize("N,n_swim", [(3, 1), (20, 1), (64, 1), (65, 1), (128, 1), (20, 3), (64, 3), (256, 1), (257, 1)])
def test_tables_in_lds_and_in_the_caches(ctx, oracle_core, N, n_swim):
    P = inputs.param_rows(n_swim, Sb=0.01, Ss=100.0, x0=-1.0)
    P[:, 0], P[:, 4], P[:, 6], P[:, 8] = 1.3, 2 * np.pi * (1 + np.arange(n_swim)), 0.3, 0.6 * np.arange(n_swim)
    dt, n = 2e-6, 300
    for steps in (7, 8, 20):
        one = tgp.run_forward(ctx, swim.SWIM_F64, [N], [n_swim], P, steps, dt, steps)
        many = tgp.run_forward(ctx, swim.SWIM_F64, [N] * n, [n_swim] * n, np.tile(P, (n, 1)), steps, dt, steps)
        assert one[2][0] == 0 and np.all(many[2] == 0)
        assert np.array_equal(many[0], np.tile(one[0], (n, 1, 1)))
    ref = oracle_core.forward(P, N, steps, dt, steps)
    for m in range(n_swim):
        tgp.check_traj(one[0][m], ref["obs"][m], np.array([0.0, P[m, 8]]), 1e-12, swim.SWIM_F64, steps, 2.0)
