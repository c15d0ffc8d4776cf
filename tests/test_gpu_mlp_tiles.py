"""The training kernels at their tiles' edges: the gradient on row counts around
a 64-row tile and a batch of 32 tile sums against the oracle's FP64 network
(cosine of every parameter block), and a training run against Adam steps taken
in FP64 from the kernel's own gradients of the same drawn rows."""
import numpy as np
import pytest

from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu

BLOCKS = ((0, 1536), (1536, 1600), (1600, 5696), (5696, 5760), (5760, 5824), (5824, 5825))


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def rows(n, seed, dev):
    import torch
    rng = np.random.default_rng(seed)
    x = torch.from_numpy(rng.normal(0.0, 0.6, size=(n, 24)).astype(np.float32)).to(torch.bfloat16)
    y = rng.integers(0, 256, size=n).astype(np.uint8)
    x32 = torch.zeros(n, 32, dtype=torch.bfloat16)
    x32[:, :24] = x
    return x.float().numpy(), y, x32.view(torch.int16).to(dev), torch.from_numpy(y).to(dev)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 2113])
def test_gradient_at_tile_edges(dev, n):
    import oracle
    import paper_1801_08361_amd as rl
    x, y, xd, yd = rows(n, n, dev)
    banner(f"mlp gradient n={n}")
    m = rl.Mlp(9)
    g, loss = m.gradient(xd, yd)
    og, ol = oracle.mlp_grad(m.weights(), x, y)
    assert abs(loss - ol) <= 1e-4 * max(1.0, abs(ol))
    for a, b in BLOCKS:
        u, v = g[a:b].astype(np.float64), og[a:b]
        if np.linalg.norm(v) > 0.0:
            assert u @ v >= 0.9999 * np.linalg.norm(u) * np.linalg.norm(v), (n, a)
            assert abs(np.linalg.norm(u) / np.linalg.norm(v) - 1.0) < 1e-2, (n, a)


def drawn(seed, epoch, step, n, n_rows):
    import oracle
    key = (seed, 6)
    return np.array([(int(oracle.philox((epoch, step, j, 0), key)[0]) * n_rows) >> 64 for j in range(n)])


@pytest.mark.parametrize("n,batch", [(200, 64), (150, 65), (40, 100)])
def test_training_takes_adam_steps_on_the_drawn_rows(dev, n, batch):
    import torch
    import paper_1801_08361_amd as rl
    _, _, xd, yd = rows(n, 5 + n, dev)
    epochs, lr, seed = 2, 1e-3, 77
    banner(f"mlp train n={n} batch={batch}")
    m, ref = rl.Mlp(4), rl.Mlp(4)
    losses = m.train(xd, yd, epochs=epochs, batch_rows=batch, lr=lr, seed=seed)
    w = ref.weights().astype(np.float64)
    w0 = w.copy()
    m1, m2, t = np.zeros_like(w), np.zeros_like(w), 0
    for e in range(epochs):
        for s in range(max(1, n // batch)):
            pick = torch.from_numpy(drawn(seed, e, s, batch, n)).to(dev)
            g, loss = ref.gradient(xd[pick].contiguous(), yd[pick].contiguous())
            g = g.astype(np.float64)
            t += 1
            m1 = 0.9 * m1 + 0.1 * g
            m2 = 0.999 * m2 + 0.001 * g * g
            w = w - lr * (m1 / (1 - 0.9 ** t)) / (np.sqrt(m2 / (1 - 0.999 ** t)) + 1e-8)
            ref.set_weights(w.astype(np.float32))
        assert abs(losses[e] - loss) <= 1e-4 * max(1.0, loss)
    # FP32 steps round a weight by parts in 1e7; a bfloat16 copy that then rounds the other way
    # (by 2^-8) moves the next gradients, and so the next steps, by under 1 %
    assert np.linalg.norm(m.weights() - w) <= 0.02 * np.linalg.norm(w - w0)
