"""GPU: what a refused host population leaves behind.  Large populations are
checked after their launch; to a caller the refusal is the same as if they had
been checked first."""
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


def _population(rng, m, P, longest=9):
    return synth.pack_cbf([rng.choice(m, size=int(rng.integers(2, longest + 1)), replace=False)
                           for _ in range(P)])


def _note(msg):
    print(f"[refused] {msg}", flush=True)
    sys.stdout.flush()


# below and above the number of entries that is checked after the launch
@pytest.mark.parametrize("P", [100, 2000])
@pytest.mark.parametrize("wrong", ["repeat", "outside"])
def test_no_index_is_left_behind(ebic, P, wrong):
    rng = np.random.default_rng(P)
    a = rng.standard_normal((300, 30)).astype(np.float32)
    off, cols = _population(rng, 30, P)
    bad = cols.copy()
    bad[off[P // 2] + 1] = bad[off[P // 2]] if wrong == "repeat" else 30
    kw = dict(sigma=4, max_violations=1, negative_trends=True)
    with ebic.Context(a) as ctx:
        _note(f"index P={P} {wrong}")
        with pytest.raises(ebic.EbicError, match=f"candidate {P // 2}"):
            ctx.evaluate(off, bad, **kw)
        info = ctx.info()
        assert info["index_built"] == 0 and info["index_build_ms"] == 0
        ref = oracle.evaluate(a, off, cols, **kw)
        for _ in range(2):
            got = ctx.evaluate(off, cols, **kw)
            assert np.array_equal(got["counts"], ref["counts"])
            assert np.array_equal(got["fitness"], ref["fitness"])
        assert ctx.info()["index_built"] == 1
        with pytest.raises(ebic.EbicError, match=f"candidate {P // 2}"):
            ctx.evaluate(off, bad, **kw)
        assert ctx.info()["index_built"] == 1        # (it was there before the call)
        assert np.array_equal(ctx.evaluate(off, cols, **kw)["counts"], ref["counts"])


def test_refusal_before_other_errors(ebic):
    # more candidates than the direct kernel takes in one launch: the wrong
    # column is still what the call names
    P = (1 << 21) + 8
    off = np.arange(P + 1, dtype=np.int32)
    cols = np.zeros(P, dtype=np.int32)
    with ebic.Context(np.ones((8, 3), dtype=np.float32), path="direct") as ctx:
        _note("too many candidates")
        with pytest.raises(ebic.EbicError, match="too large"):
            ctx.evaluate(off, cols, sigma=1)
        cols[P - 3] = 3
        with pytest.raises(ebic.EbicError, match=f"out of range in candidate {P - 3}"):
            ctx.evaluate(off, cols, sigma=1)


@pytest.mark.parametrize("P", [60, 3000])
def test_batch_keeps_no_refused_launch(ebic, P):
    rng = np.random.default_rng(P)
    mats = [rng.standard_normal((n, 20)).astype(np.float32) for n in (200, 700)]
    first = [_population(rng, 20, 50) for _ in mats]
    pops = [_population(rng, 20, P) for _ in mats]
    o, c = pops[1]
    bad = c.copy()
    bad[o[7] + 1] = bad[o[7]]
    with ebic.Batch(mats) as b:
        b.evaluate(first, sigma=4)
        ms = b.last_ms()
        assert ms > 0 and b.time_replays(2) > 0
        _note(f"batch P={P}")
        with pytest.raises(ebic.EbicError, match="run 1: duplicate column in candidate 7"):
            b.evaluate([pops[0], (o, bad)], sigma=4)
        assert b.last_ms() == ms
        # the refused population has taken the place of the first one's
        with pytest.raises(ebic.EbicError, match="no batched launch"):
            b.time_replays(2)
        for a, p, g in zip(mats, pops, b.evaluate(pops, sigma=4)):
            assert np.array_equal(g["counts"], oracle.evaluate(a, *p, sigma=4)["counts"])
        assert b.time_replays(2) > 0
