"""The training pass at the sizes where its split of the rows changes: one row, row blocks of 16
and their remainders, the most workgroups of one row block, the change to 64-row forward tiles and
several row blocks per workgroup, against the oracle's gradient."""
import numpy as np
import pytest

from oracle import oracle as o
from tests import inputs

kg = pytest.importorskip("paper_2109_11001_amd")
torch = pytest.importorskip("torch")


def _magnitudes(P, x, y):
    """Per parameter, a bound on the sum of the magnitudes of its gradient's terms (numpy, FP64)."""
    W, at = [], 0
    for rows, cols in ((128, 25), (128, 128), (128, 128), (1, 128)):
        w = np.clip(np.rint(P[at:at + rows * cols].reshape(rows, cols).astype(np.float64) * 64), -255, 255) / 64
        W.append((w, P[at + rows * cols:at + rows * (cols + 1)]))
        at += rows * (cols + 1)
    h = np.clip(np.rint(x.astype(np.float64) * 64), -255, 255) / 64
    acts, masks = [], []
    for k, (w, b) in enumerate(W):
        acts.append(np.abs(h))
        z = (h @ w.T).astype(np.float32) + b
        if k < 3:
            masks.append((z > 0) & (z < 255 / 16))
            h = np.clip(np.rint(np.maximum(z, 0) * 16.0), 0, 255).astype(np.float64) / 16
    d = np.abs(1 / (1 + np.exp(-z.astype(np.float64))) - y[:, None]) / len(y)
    S = []
    for k in (3, 2, 1, 0):
        S = [(d.T @ acts[k]).ravel(), d.sum(0)] + S
        if k:
            d = (d @ np.abs(W[k][0])) * masks[k - 1]
    return np.concatenate(S)


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")
@pytest.mark.parametrize("n", [1, 16, 17, 2048, 2049, 8193, 16384, 16385])
def test_gradient_at_the_edges_of_the_row_split(n):
    P = inputs.random_mlp_params(n, w_scale=0.2, b_scale=0.3)
    x = np.random.default_rng(n).normal(0, 1.0, size=(n, 25)).astype(np.float32)
    y = inputs.random_labels(n, n, p=0.4)
    dev = [torch.as_tensor(a).cuda() for a in (P, x, y)]
    g, loss = kg.mlp_grad(*dev)
    go, lo = o.mlp_grad(P, x, y)
    assert float(loss.cpu()[0]) == pytest.approx(lo, rel=1e-12)
    # FP64 on both sides: sums of at most 16,385 x 128 x 128 terms in different orders, whose errors
    # stay below 1e-11 of the terms' magnitudes
    S = _magnitudes(P, x, y)
    assert np.all(np.abs(g.cpu().numpy() - go) <= 1e-11 * S + 1e-300)
    g2, _ = kg.mlp_grad(*dev)
    assert torch.equal(g, g2)


def test_workspace_grows_with_the_rows():
    # a workspace for n rows serves any smaller batch
    from paper_2109_11001_amd._lib import load
    sizes = [load().kgdb_mlp_workspace_bytes(n) for n in list(range(1, 300)) + list(range(300, 70000, 61))]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
