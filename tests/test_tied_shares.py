"""GPU: matrices of which a share of the column pairs ties, around the share at
which a workgroup changes its loop, against the CPU oracle, bit for bit, in
every tiling (1, 2 and 4 words per lane, flattened; batches with 8)."""
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


def _tied(rng, n, m, share):
    """About `share` of the column pairs tie, on one or two rows each."""
    a = rng.standard_normal((n, m)).astype(np.float32)
    pairs = [(p, q) for p in range(m) for q in range(p)]
    for i in rng.choice(len(pairs), size=int(round(share * len(pairs))), replace=False):
        p, q = pairs[i]
        for r in rng.integers(0, n, size=int(rng.integers(1, 3))):
            a[r, p] = a[r, q]
    return a


@pytest.mark.parametrize("words", [16, 130, 330, 1030])
@pytest.mark.parametrize("share", [0.03, 0.08, 0.13, 0.3, 0.9])
def test_shares(ebic, words, share):
    rng = np.random.default_rng(words)
    n, m = words * 64 - 11, 40
    a = _tied(rng, n, m, share)
    off, cols = synth.pack_cbf(synth.random_population(rng, m, 30, 2, 20))
    with ebic.Context(a, path="index") as ctx:
        for k in (0, 1, 2, 5):
            print(f"[tied] words={words} share={share} k={k}", flush=True)
            sys.stdout.flush()
            ref = oracle.evaluate(a, off, cols, sigma=4, max_violations=k, negative_trends=True,
                                  want_masks=True)
            got = ctx.evaluate(off, cols, sigma=4, max_violations=k, negative_trends=True,
                               want_masks=True)
            assert np.array_equal(got["counts"], ref["counts"])
            assert np.array_equal(got["fitness"].view(np.int64), ref["fitness"].view(np.int64))
            assert np.array_equal(got["masks"], ref["masks"])


@pytest.mark.parametrize("shape", [(2, 8, 1), (1, 8, 0), (4, 4, 1), (4, 2, 1), (8, 1, 0)])
def test_batches(ebic, shape):
    rng = np.random.default_rng(sum(shape))
    mats = [_tied(rng, n, 30, share) for n in (300, 1500) for share in (0.05, 0.2, 0.7)]
    pops = [synth.pack_cbf(synth.random_population(rng, 30, 200, 2, 20)) for _ in mats]
    with ebic.Batch(mats) as b:
        b.set_tuning(-1, *shape)
        for k in (0, 1, 3):
            print(f"[tied] batch {shape} k={k}", flush=True)
            got = b.evaluate(pops, sigma=4, max_violations=k, negative_trends=True)
            for a, (o, c), g in zip(mats, pops, got):
                ref = oracle.evaluate(a, o, c, sigma=4, max_violations=k, negative_trends=True)
                assert np.array_equal(g["counts"], ref["counts"])
                assert np.array_equal(g["fitness"].view(np.int64), ref["fitness"].view(np.int64))
