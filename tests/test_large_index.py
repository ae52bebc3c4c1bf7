"""GPU: order indexes of more than 4 GiB (row offsets in units of 128 bytes,
64-bit addresses) against the CPU oracle, bit for bit, in every tiling: series
of the highest columns, some of them tied, and series of any columns."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ebic():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_03039_amd as e
    return e


# 1, 2 and 4 words per lane, flattened tiles
@pytest.mark.parametrize("n,m", [(8190, 2048), (20000, 1500), (40000, 1000), (70000, 760)])
def test_past_4_gib(ebic, n, m):
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, m), dtype=np.float32)
    top = np.arange(m - 30, m)
    a[7, top[::5]] = 0.25                       # few pairs of the highest columns tie
    a[n - 3:, top[1::2]] = np.float32(-0.5)     # ... and every second one with each other
    pop = [rng.permutation(top)[:int(rng.integers(2, 20))] for _ in range(20)]
    pop += [rng.permutation(top[1::2])[:12], top[::-1][:16], np.array([m - 1, 0]), np.array([0, m - 1])]
    pop += [rng.choice(m, size=int(rng.integers(1, 16)), replace=False) for _ in range(20)]
    off, cols = synth.pack_cbf([x.astype(np.int32) for x in pop])
    with ebic.Context(a, path="index") as ctx:
        assert ctx.info()["index_bytes"] > 1 << 32
        for k in (0, 1, 2, 5, 9):
            for neg in (False, True):
                print(f"[large] n={n} m={m} k={k} neg={neg}", flush=True)
                sys.stdout.flush()
                ref = oracle.evaluate(a, off, cols, sigma=4, max_violations=k,
                                      negative_trends=neg, want_masks=True)
                got = ctx.evaluate(off, cols, sigma=4, max_violations=k, negative_trends=neg,
                                   want_masks=True)
                assert np.array_equal(got["counts"], ref["counts"])
                assert np.array_equal(got["fitness"].view(np.int64), ref["fitness"].view(np.int64))
                assert np.array_equal(got["masks"], ref["masks"])
