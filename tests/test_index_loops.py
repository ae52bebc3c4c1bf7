"""GPU: the index evaluator's loops against the CPU oracle, bit for bit: pairs
that never tie, a few tied pairs, mostly tied pairs, repeated columns, and
series past the workgroup's staging area; in every tiling (1, 2 and 4 words
per lane, flattened tiles)."""
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


def _note(msg):
    print(f"[loops] {msg}", flush=True)
    sys.stdout.flush()


def _device(ctx, off, cols, k, neg):
    import torch
    P = len(off) - 1
    d = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda() for x in (off, cols)]
    counts = torch.zeros(P, dtype=torch.int32, device="cuda")
    fit = torch.zeros(P, dtype=torch.float64, device="cuda")
    masks = torch.zeros((P, 2, ctx.W), dtype=torch.int64, device="cuda")
    ctx.evaluate_device(*d, counts, fit, masks, sigma=4, max_violations=k, negative_trends=neg)
    return {"counts": counts.cpu().numpy(), "fitness": fit.cpu().numpy(),
            "masks": masks.cpu().numpy().view(np.uint64)}


def _same(got, ref):
    assert np.array_equal(got["counts"], ref["counts"])
    assert np.array_equal(got["fitness"].view(np.int64), ref["fitness"].view(np.int64))
    assert np.array_equal(got["masks"], ref["masks"])


def _definition(a, pop, k, neg):
    """Counts and masks by the definition (the oracle refuses repeated columns)."""
    counts, masks = [], []
    for series in pop:
        v = a[:, list(series)]
        up = (~(v[:, :-1] < v[:, 1:])).sum(1) <= k
        down = ((~(v[:, :-1] > v[:, 1:])).sum(1) <= k) & neg
        counts.append((up | down).sum())
        masks.append(synth.rows_to_masks([np.nonzero(up)[0], np.nonzero(down)[0]], len(a)))
    return np.array(counts, dtype=np.int32), np.stack(masks)


def _matrix(rng, n, m, ties):
    a = rng.standard_normal((n, m)).astype(np.float32)
    if ties == "few":
        for p, q in ((0, 1), (5, 3), (2, 8)):
            a[n // 2, q] = a[n // 2, p]
    elif ties == "nan":
        a[n - 1, 4] = np.nan
    elif ties == "many":
        a = np.round(a * 2) / 2
    return np.ascontiguousarray(a, dtype=np.float32)


# words: 1, 4 (several series per wave), 128 | 129 (1 | 2 words per lane),
# 320 | 321 (2 | 4), 1024 | 1025 (4 | flattened)
@pytest.mark.parametrize("words", [1, 4, 128, 129, 320, 321, 1024, 1025])
@pytest.mark.parametrize("ties", ["none", "few", "nan", "many"])
def test_loops_match_oracle(ebic, words, ties):
    rng = np.random.default_rng(words)
    n, m = words * 64 - 5, 14
    a = _matrix(rng, n, m, ties)
    pop = synth.random_population(rng, m, 41, 1, 13)
    off, cols = synth.pack_cbf(pop)
    with ebic.Context(a, path="index") as ctx:
        for k in (0, 1, 2, 3, 5):
            for neg in (False, True):
                _note(f"words={words} ties={ties} k={k} neg={neg}")
                ref = oracle.evaluate(a, off, cols, sigma=4, max_violations=k,
                                      negative_trends=neg, want_masks=True)
                _same(_device(ctx, off, cols, k, neg), ref)


@pytest.mark.parametrize("words", [1, 130, 330])
def test_repeated_columns(ebic, words):
    # device populations may repeat a column, also right after itself: such a
    # pair breaks both trends on every row
    rng = np.random.default_rng(words)
    a = _matrix(rng, words * 64, 9, "few")
    pop = [[3, 3], [1, 2, 2, 4], [5, 5, 5, 6, 7], [0, 8, 0, 8], [2], [4, 4, 4, 4, 4, 4, 4, 4]]
    pop += [list(rng.integers(0, 9, size=int(rng.integers(1, 20)))) for _ in range(40)]
    off, cols = synth.pack_cbf(pop)
    with ebic.Context(a, path="index") as ctx:
        for k in (0, 1, 3, 6):
            for neg in (False, True):
                _note(f"repeats words={words} k={k} neg={neg}")
                counts, masks = _definition(a, pop, k, neg)
                got = _device(ctx, off, cols, k, neg)
                assert np.array_equal(got["counts"], counts)
                assert np.array_equal(got["masks"], masks)
                fit = [oracle.fitness(int(c), len(s), 4) for c, s in zip(counts, pop)]
                assert np.array_equal(got["fitness"], np.array(fit))


@pytest.mark.parametrize("length", [32, 33, 70])
def test_series_past_the_staging_area(ebic, length):
    # 64 one-word series per workgroup: 64 * 32 columns are staged, more are not
    rng = np.random.default_rng(length)
    m = 80
    a = rng.standard_normal((50, m)).astype(np.float32)
    off, cols = synth.pack_cbf(synth.random_population(rng, m, 150, length, length))
    with ebic.Context(a, path="index") as ctx:
        for k in (0, 2, 20):
            for neg in (False, True):
                _note(f"staging length={length} k={k} neg={neg}")
                ref = oracle.evaluate(a, off, cols, sigma=4, max_violations=k,
                                      negative_trends=neg, want_masks=True)
                _same(_device(ctx, off, cols, k, neg), ref)
                # a column outside the matrix spoils its own series only
                bad = cols.copy()
                bad[off[7] + 3] = m
                got = _device(ctx, off, bad, k, neg)
                assert got["counts"][7] == -1 and np.isnan(got["fitness"][7])
                keep = np.arange(150) != 7
                assert np.array_equal(got["counts"][keep], ref["counts"][keep])
