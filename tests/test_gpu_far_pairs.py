"""FP32 runs with two swimmers so far apart that pair distances pass 2^16 in units
of 1 / rho (v = 1 + d^2 beyond 2^32, octaves 32 and up of the table): every octave
of the table window holds its own entries.  Against the oracle with
test_gpu_parity's trajectory bar; the first swimmer lies at the origin, where FP32
outputs resolve its way.  The far swimmer's
forces sum to zero, so its pull vanishes unless the far pairs read entries of other
octaves, which differ from pair to pair."""
import math

import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("reading_blob_module")]

torch = pytest.importorskip("torch")

import test_gpu_parity as tgp  # noqa: E402
from paper_1910_12007_amd import inputs, swim  # noqa: E402

ctx = tgp.ctx


@pytest.mark.parametrize("N,n", [(150, 1), (150, 300), (250, 1)])
def test_distances_beyond_2_to_16(ctx, oracle_core, N, n):
    rho = 2.0 ** math.ceil(math.log2((N - 1) / 1.5))
    far = 1.03 * 65536.0 / rho
    assert far < 1e3  # within the run bound
    P = inputs.param_rows(2, Sb=0.01, Ss=100.0, x0=-1.0)
    P[:, 0] = 1.3
    P[1, 6], P[1, 8] = 1.1, far
    steps, dt, every = 60, 2e-6, 20
    obs, speed, st = tgp.run_forward(ctx, swim.SWIM_F32, [N] * n, [2] * n, np.tile(P, (n, 1)), steps, dt, every)
    assert np.all(st == 0)
    ref = oracle_core.forward(P, N, steps, dt, every)
    for k in range(0, 2 * n, max(1, n // 3) * 2):
        for m in range(2):
            tgp.check_traj(obs[k + m], ref["obs"][m], np.array([0.0, P[m, 8]]), 1e-4, swim.SWIM_F32, steps,
                           max(1.0, abs(P[m, 8])))
