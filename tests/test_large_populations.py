"""GPU: host populations large enough to be checked after the launch: same
results as the oracle, same refusals, and outputs untouched by a refusal."""
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


def _population(rng, m, entries, longest):
    series, total = [], 0
    while total < entries:
        series.append(rng.choice(m, size=int(rng.integers(1, longest + 1)), replace=False))
        total += len(series[-1])
    return synth.pack_cbf(series)


# below and above the number of entries checked on the device; series of more
# than one wave's columns and longer than the device compares
@pytest.mark.parametrize("entries,m,longest", [(3000, 30, 20), (6000, 30, 20), (9000, 200, 150),
                                               (9000, 600, 520)])
@pytest.mark.parametrize("path", ["index", "direct"])
def test_checks(ebic, path, entries, m, longest):
    rng = np.random.default_rng(entries + m)
    a = rng.standard_normal((150, m)).astype(np.float32)
    off, cols = _population(rng, m, entries, longest)
    P = len(off) - 1
    lens = np.diff(off)
    two = [int(c) for c in np.nonzero(lens >= 2)[0]]
    late, early = two[-1], two[1]
    kw = dict(sigma=5, max_violations=1, negative_trends=True)
    print(f"[large] {path} entries={entries} m={m} longest={longest} P={P}", flush=True)
    sys.stdout.flush()
    ref = oracle.evaluate(a, off, cols, **kw)
    E = ebic.binding
    with ebic.Context(a, path=path) as ctx:
        def evaluate(o, c):
            counts, fit = np.full(P, 77, dtype=np.int32), np.full(P, 7.5)
            prm = E.make_params(5, 1, True)
            o, c = (np.ascontiguousarray(x, dtype=np.int32) for x in (o, c))
            st = E._evaluate(ctx.handle, E._np_ptr(o), E._np_ptr(c), P, E.ctypes.byref(prm), None,
                             E._np_ptr(counts), E._np_ptr(fit))
            return st, E._last_error(ctx.handle).decode(), counts, fit

        def same():
            st, _, counts, fit = evaluate(off, cols)
            assert st == 0 and np.array_equal(counts, ref["counts"])
            assert np.array_equal(fit.view(np.int64), ref["fitness"].view(np.int64))

        same()
        repeat, outside, both, order = (cols.copy() for _ in range(4))
        repeat[off[late + 1] - 1] = repeat[off[late]]
        outside[off[late]] = m
        both[off[late] + 1] = -1
        both[off[early] + 1] = both[off[early]]
        bad_off = off.copy()
        bad_off[late + 1] = bad_off[late]                 # an empty series
        for o, c, status, text in (
                (off, repeat, E.EBIC_E_ARG, f"duplicate column in candidate {late}"),
                (off, outside, E.EBIC_E_RANGE, f"column out of range in candidate {late}"),
                (off, both, E.EBIC_E_ARG, f"duplicate column in candidate {early}"),
                (bad_off, order, E.EBIC_E_ARG, f"candidate {late}")):
            st, msg, counts, fit = evaluate(o, c)
            assert st == status and text in msg, (st, msg)
            assert (counts == 77).all() and (fit == 7.5).all()
        same()


def test_batch_checks(ebic):
    rng = np.random.default_rng(5)
    mats = [rng.standard_normal((n, m)).astype(np.float32) for n, m in ((300, 20), (90, 50), (700, 9))]
    pops = [_population(rng, a.shape[1], 5000, 8) for a in mats]
    with ebic.Batch(mats) as b:
        def check(k, neg):
            got = b.evaluate(pops, sigma=4, max_violations=k, negative_trends=neg)
            for a, (o, c), g in zip(mats, pops, got):
                ref = oracle.evaluate(a, o, c, sigma=4, max_violations=k, negative_trends=neg)
                assert np.array_equal(g["counts"], ref["counts"])
                assert np.array_equal(g["fitness"].view(np.int64), ref["fitness"].view(np.int64))

        check(1, True)
        check(5, False)              # the direct kernel
        for run, value, status, text in ((1, None, "E_ARG", "duplicate column"),
                                         (2, 9, "E_RANGE", "column out of range")):
            o, c = pops[run]
            at = int(np.nonzero(np.diff(o) >= 2)[0][-1])
            bad = c.copy()
            bad[o[at] + 1] = bad[o[at]] if value is None else value
            wrong = [p if r != run else (o, bad) for r, p in enumerate(pops)]
            with pytest.raises(ebic.EbicError) as ex:
                b.evaluate(wrong, sigma=4)
            assert str(ex.value).startswith(status)
            assert f"run {run}: {text}" in str(ex.value) and f"candidate {at}" in str(ex.value)
        check(0, False)
