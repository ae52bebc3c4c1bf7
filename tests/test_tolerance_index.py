"""GPU: tolerances above 3 evaluated from the order index (binary violation
counters) against the CPU oracle, bit for bit: every counter width and its
edges, every tiling (1 and 2 words per lane, flattened), ties and NaN."""
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


def _same(got, ref):
    assert np.array_equal(got["counts"], ref["counts"])
    assert np.array_equal(got["fitness"].view(np.int64), ref["fitness"].view(np.int64))
    assert np.array_equal(got["masks"], ref["masks"])


# 128 words end the 1-word-per-lane tiles, 640 the 2-word ones.
@pytest.mark.parametrize("n", [1, 65, 1000, 64 * 128, 64 * 128 + 1, 64 * 640, 64 * 640 + 1])
def test_large_tolerances_match_oracle(ebic, n):
    rng = np.random.default_rng(n)
    m = 70
    a = rng.standard_normal((n, m)).astype(np.float32)
    special = min(n, 40)                                  # rows with ties, NaN, infinities
    a[:special] = synth.adversarial_matrix(rng, special, m)
    pop = synth.random_population(rng, m, 24, 1, 24) + synth.random_population(rng, m, 6, 60, 70)
    order = np.argsort(a[n // 2], kind="stable")           # one long series a row follows
    pop += [order.astype(np.int32), order[::-1][:40].astype(np.int32)]
    off, cols = synth.pack_cbf(pop)
    with ebic.Context(a, path="index") as ctx:
        for k in (4, 5, 7, 8, 15, 16, 31, 63, 64):         # 64: the direct kernel
            for neg in (False, True):
                print(f"[tolerance] n={n} k={k} neg={neg}", flush=True)
                sys.stdout.flush()
                ref = oracle.evaluate(a, off, cols, sigma=7, max_violations=k,
                                      negative_trends=neg, want_masks=True)
                _same(ctx.evaluate(off, cols, sigma=7, max_violations=k, negative_trends=neg,
                                   want_masks=True), ref)


def test_large_tolerance_follows_the_path(ebic):
    # The order index serves a large tolerance only if it exists: AUTO does
    # not build it for one, and every route gives the same results, the
    # allocation-free call and malformed candidates included.
    import torch
    rng = np.random.default_rng(3)
    a = synth.adversarial_matrix(rng, 700, 12)
    off, cols = synth.pack_cbf(synth.random_population(rng, 12, 50, 2, 12))
    ref = oracle.evaluate(a, off, cols, sigma=5, max_violations=5, negative_trends=True,
                          want_masks=True)
    kw = dict(sigma=5, max_violations=5, negative_trends=True)
    with ebic.Context(a) as ctx:
        _same(ctx.evaluate(off, cols, want_masks=True, **kw), ref)
        assert ctx.info()["index_built"] == 0
        for path in ("index", "auto", "direct"):
            ctx.set_path(path)
            _same(ctx.evaluate(off, cols, want_masks=True, **kw), ref)
        ctx.set_path("index")
        bad_cols, bad_off = cols.copy(), off.copy()
        bad_cols[off[1]] = 99                              # candidate 1: column out of range
        bad_off[-1] = off[-1] + 30                         # the last: past the entries
        d = [torch.from_numpy(x).cuda() for x in (bad_off, bad_cols)]
        counts = torch.zeros(50, dtype=torch.int32, device="cuda")
        fit = torch.zeros(50, dtype=torch.float64, device="cuda")
        for noalloc in (False, True):
            ctx.evaluate_device(*d, counts, fit, noalloc=noalloc, **kw)
            c, f = counts.cpu().numpy(), fit.cpu().numpy()
            assert c[1] == -1 and np.isnan(f[1]) and c[-1] == -1 and np.isnan(f[-1])
            assert c[0] == ref["counts"][0] and np.array_equal(c[2:-1], ref["counts"][2:-1])
