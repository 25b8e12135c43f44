"""The training gradient where the spread of its work over the chip changes: fewer than
eight chunks of 256 rows (one after another) and eight or more (chunk c to XCD c mod 8, with
idle slots where the number is no multiple of eight), whole and broken rounds of 128 tiles;
against the oracle, with the tolerances of the other gradient tests (bfloat16 products)."""
import numpy as np
import pytest

from oracle import mlp

from test_gpu_warmstart import _net_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [16, 1792, 1793, 2032, 2048, 2049, 4096])
def test_gradient_at_chunk_edges(n_rows):
    n_out = 6
    s, theta = _net_solver(n_out, seed=n_rows)
    rng = np.random.default_rng(n_rows)
    X = rng.standard_normal((n_rows, 8)).astype(np.float32)
    T = (rng.standard_normal((n_rows, n_out)) - 2.0).astype(np.float32)
    loss, g = s.mlp_loss_grad(X, T)
    rl, rg = mlp.loss_and_grad(theta.astype(np.float64), X.astype(np.float64), T.astype(np.float64), n_out,
                               round_bf16=True)
    assert abs(loss - rl) < 1e-4 * rl
    k = 0
    for o, i in mlp.layer_shapes(n_out):
        for size in (o * i, o):
            a, b = g[k:k + size].astype(np.float64), rg[k:k + size]
            k += size
            assert np.linalg.norm(a - b) < 1e-2 * np.linalg.norm(b), (o, i, size)
