"""The fused training step at the edges of its row tiles (16 rows a tile, 32 a
summation piece, two tiles a workgroup from 8192 rows on) against the oracle's
backward pass: the gradients' bar is that of every batch size, 3e-3 of each
layer's norm (bfloat16 operands on both sides; only a rounding decided
differently by the FP32 sums' order separates them)."""
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


def _data(n, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    X = rng.standard_normal((n, 5)).astype(np.float32)
    T = (np.tanh(X[:, :3] @ rng.standard_normal((3, 33))) + 0.1 * rng.standard_normal((n, 33))).astype(np.float32)
    return X, T


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 129, 1025, 8191, 8208])
def test_gradients_at_tile_edges(ctx, n):
    from oracle import mlp
    X, T = _data(n, n)
    _, flat = inputs.mlp_init(3)
    G = torch.full((swim.SWIM_MLP_NPARAM,), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    dev = [torch.from_numpy(a).cuda() for a in (X, T, flat)]
    swim.surrogate_grad(ctx, *dev, G, loss)
    torch.cuda.synchronize()
    lref, gref = mlp.backward(inputs.unflatten(flat), X.astype(np.float64), T.astype(np.float64), True)
    assert abs(loss.item() / (n * 33) / lref - 1) < 1e-4
    for l, ((gW, gb), (rW, rb)) in enumerate(zip(inputs.unflatten(G.cpu().numpy()), gref)):
        assert _rel(gW, rW) < 3e-3 and _rel(gb, rb) < 3e-3, (l, _rel(gW, rW), _rel(gb, rb))


@pytest.mark.parametrize("batch", [40, 8200])
def test_training_is_gradient_and_adam(ctx, batch):
    """One training step on permuted rows equals Adam's first step on the
    gradient of those rows (both from the library), and leaves packed weights
    that the second step reads: two steps equal one and then one more."""
    X, T = _data(2 * batch + 3, 5)
    _, flat = inputs.mlp_init(3)
    dX, dT = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    rng = np.random.Generator(np.random.PCG64(1))
    perm = rng.permutation(len(X)).astype(np.int32)
    p2 = torch.from_numpy(flat).cuda()
    m2, v2 = torch.zeros_like(p2), torch.zeros_like(p2)
    swim.surrogate_train(ctx, dX, dT, torch.from_numpy(perm).cuda(), 1, batch, 1e-3, p2, m2, v2)
    p, m, v = (torch.from_numpy(a).cuda() for a in (flat, 0 * flat, 0 * flat))
    for k in range(2):
        rows = torch.from_numpy(perm[k * batch:(k + 1) * batch].astype(np.int64)).cuda()
        G = torch.empty_like(p)
        swim.surrogate_grad(ctx, dX[rows].contiguous(), dT[rows].contiguous(), p, G)
        m = 0.9 * m + (1 - np.float32(0.9)) * G
        v = 0.999 * v + (1 - np.float32(0.999)) * G * G
        p = p - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / (torch.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
    torch.cuda.synchronize()
    # FP32 rounding of the update formula; from the second step on, bfloat16
    # roundings of weights that differ in the last bit
    assert _rel(m2.cpu().numpy(), m.cpu().numpy()) < 1e-3
    assert _rel((p2 - torch.from_numpy(flat).cuda()).cpu().numpy(), (p - torch.from_numpy(flat).cuda()).cpu().numpy()) < 1e-2


def test_bad_row_index_gives_nan(ctx):
    X, T = _data(64, 2)
    _, flat = inputs.mlp_init(3)
    p = torch.from_numpy(flat).cuda()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    perm = np.arange(64, dtype=np.int32)
    perm[5] = 64
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    swim.surrogate_train(ctx, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), torch.from_numpy(perm).cuda(), 1,
                         64, 1e-3, p, m, v, loss)
    torch.cuda.synchronize()
    assert np.isnan(loss.item())
