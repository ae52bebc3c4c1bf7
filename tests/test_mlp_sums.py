"""GPU: the embedding gradients' ordered sums against the CPU oracle where
lists are longer than one round of 256 entries, end inside a row or a place,
or are empty."""
import sys

import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_03039_amd as e
    return e


# occurrences per column: about 8 (one place), 33 (a second row), 257 and 700
# (two and three rounds); columns from `used` on never occur
@pytest.mark.parametrize("M,used,B", [(40, 40, 64), (9, 9, 60), (12, 7, 450), (6, 6, 1200)])
def test_embedding_gradients(E, M, used, B):
    rng = np.random.default_rng(M * B)
    lmax = min(used, 6)
    series = [rng.choice(used, size=int(rng.integers(1, lmax + 1)), replace=False)
              for _ in range(B)]
    off = np.zeros(B + 1, dtype=np.int32)
    off[1:] = np.cumsum([len(s) for s in series])
    cols = np.concatenate(series).astype(np.int32)
    t = rng.standard_normal(B).astype(np.float32)
    D, H = 32, 256
    with E.Mlp(M, seed=11) as net:
        print(f"[sums] M={M} used={used} B={B}", flush=True)
        sys.stdout.flush()
        _, g = net.gradients(off, cols, t)
        _, again = net.gradients(off, cols, t)
        assert np.array_equal(g, again)
        _, ref, _ = omlp.loss_and_grad(net.params(), off, cols, t, M, D, H, bf16=True)
    # each table within 1e-2 of its largest reference gradient (the same BF16
    # rounding points, FP32 sums in another order)
    at = 0
    for name, rows in (("E", M), ("F", M), ("T", M), ("Z", M + 1)):
        sl = slice(at, at + rows * D)
        at += rows * D
        bound = 1e-2 * float(np.max(np.abs(ref[sl])))
        assert float(np.max(np.abs(g[sl] - ref[sl]))) <= bound, name
        empty = np.abs(ref[sl]).reshape(rows, D).max(1) == 0
        assert not g[sl].reshape(rows, D)[empty].any(), name
