"""GPU: the gradient lists built on the device.  Their order decides the bits
of the embedding gradients, so batches around the edges of the sort's tiles
are compared with the float64 oracle, and a network too wide for the device's
counters (lists built on the host) with the same network and columns mapped
into a narrow one."""
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


def _batch(rng, M, B, longest):
    series = [rng.choice(M, size=int(rng.integers(1, min(longest, M) + 1)), replace=False)
              for _ in range(B)]
    off = np.zeros(B + 1, dtype=np.int32)
    off[1:] = np.cumsum([len(s) for s in series])
    return off, np.concatenate(series).astype(np.int32)


def _tables(g, M, D=32):
    sizes = [("E", M), ("F", M), ("T", M), ("Z", M + 1)]
    out, at = {}, 0
    for name, rows in sizes:
        out[name] = g[at:at + rows * D].reshape(rows, D)
        at += rows * D
    return out


# one item; a wave, a tile and one more item; many tiles of one to many keys
@pytest.mark.parametrize("M,B,longest", [(1, 1, 1), (1, 300, 1), (2, 64, 1), (3, 256, 1),
                                         (7, 257, 2), (65, 1025, 9), (513, 3000, 20)])
def test_gradients_at_tile_edges(E, M, B, longest):
    rng = np.random.default_rng(M + B)
    off, cols = _batch(rng, M, B, longest)
    t = rng.standard_normal(B).astype(np.float32)
    with E.Mlp(M, seed=3) as net:
        print(f"[lists] M={M} B={B}", flush=True)
        sys.stdout.flush()
        _, g = net.gradients(off, cols, t)
        _, ref, _ = omlp.loss_and_grad(net.params(), off, cols, t, M, 32, 256, bf16=True)
    for name, r in _tables(ref, M).items():
        # 1e-2 of the table's largest gradient: FP32 sums, the same BF16 points
        assert np.max(np.abs(_tables(g, M)[name] - r)) <= 1e-2 * max(np.max(np.abs(r)), 1e-30), name


def test_host_and_device_lists_agree(E):
    # columns 0..59 of a narrow network placed at spread-out columns of a wide
    # one: the same sums in the same order, bit for bit
    rng = np.random.default_rng(9)
    M, wide, B = 60, 8400, 700
    off, cols = _batch(rng, M, B, 14)
    place = np.sort(rng.choice(wide, size=M, replace=False)).astype(np.int32)
    t = rng.standard_normal(B).astype(np.float32)
    with E.Mlp(M, seed=3) as a, E.Mlp(wide, seed=4) as b:
        p, q = a.params(), b.params()
        for name, table in _tables(p, M).items():
            into = _tables(q, wide)[name]
            into[:] = 0
            into[place if name != "Z" else np.arange(M + 1)] = table
        q[(4 * wide + 1) * 32:] = p[(4 * M + 1) * 32:]
        b.set_params(q)
        print("[lists] wide", flush=True)
        _, g = a.gradients(off, cols, t)
        _, h = b.gradients(off, place[cols], t)
        for name, table in _tables(g, M).items():
            rows = place if name != "Z" else np.arange(M + 1)
            assert np.array_equal(_tables(h, wide)[name][rows], table), name
        assert np.array_equal(h[(4 * wide + 1) * 32:], g[(4 * M + 1) * 32:])


def test_batches_of_changing_size(E):
    # one network, batches that grow and shrink, training left queued between
    # them: the staging and the lists are reused
    rng = np.random.default_rng(2)
    M = 90
    batches = [(_batch(rng, M, B, 10), rng.standard_normal(B).astype(np.float32))
               for B in (50, 3000, 7, 1200)]
    results = []
    for rep in range(2):
        with E.Mlp(M, seed=6) as net:
            out = []
            for (off, cols), t in batches:
                out.append(net.train(off, cols, t, 3))
                out.append(net.predict(off, cols))
            out.append(net.params())
            results.append(out)
    for x, y in zip(*results):
        assert np.array_equal(np.asarray(x), np.asarray(y))
    with E.Mlp(M, seed=6) as net:
        fresh = []
        for (off, cols), t in batches:
            with E.Mlp(M, seed=6) as one:
                one.set_params(net.params())
                fresh.append(one.predict(off, cols))
            assert np.array_equal(net.predict(off, cols), fresh[-1])
