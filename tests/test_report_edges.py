"""GPU: Step 6 row lists and the accuracy scores at the edges of their
kernels' tiles, against the oracle, bit for bit."""
import sys

import numpy as np
import pytest

import synth
from oracle import scores as oscores

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_03039_amd as e
    return e


def _dev(x):
    import torch
    x = np.ascontiguousarray(x)
    return torch.from_numpy(x.view(np.int64) if x.dtype == np.uint64 else x).to("cuda:0")


# words: one step of one wave, one block's 64, two chunks, 16 chunks and one
# word more; 3 planes take the general form
@pytest.mark.parametrize("words,K,planes", [(16, 3, 1), (64, 2, 2), (65, 5, 3), (1024, 4, 1),
                                            (1025, 3, 2), (3000, 2, 1)])
def test_row_lists(E, words, K, planes):
    rng = np.random.default_rng(words)
    n = words * 64 - 9
    masks = rng.integers(0, 2**63, size=(K, planes, words), dtype=np.uint64)
    masks[0] = ~np.uint64(0)                          # every row, and bits past the last
    masks[-1, :, ::2] = 0
    print(f"[report] rows words={words} K={K} planes={planes}", flush=True)
    sys.stdout.flush()
    want = oscores.mask_rows(masks, n)
    total = sum(len(w) for w in want)
    for capacity in (None, total, total - 1, 5):
        off, rows = E.mask_rows(_dev(masks), n, capacity=capacity)
        off, rows = off.cpu().numpy(), rows.cpu().numpy()
        assert np.array_equal(np.diff(off), [len(w) for w in want])
        assert np.array_equal(rows, np.concatenate(want)[:len(rows)])
        assert len(rows) == (total if capacity is None else capacity)


def test_row_lists_longer_than_the_first_guess(E):
    # every row of 9 biclusters of 120000 rows: more than 2^20 entries
    words = 1875
    masks = np.full((9, 1, words), ~np.uint64(0), dtype=np.uint64)
    off, rows = E.mask_rows(_dev(masks), words * 64)
    assert off.cpu().tolist() == [i * 120000 for i in range(10)]
    assert np.array_equal(rows.cpu().numpy(), np.tile(np.arange(120000, dtype=np.int32), 9))


# pairs per wave: one below 1024 waves, four above; columns: up to 64 entries
# in lanes, longer lists in memory; scores: 512 columns, 128 rows per chunk
@pytest.mark.parametrize("F,Ec,m,longest", [(3, 5, 200, 64), (3, 5, 300, 150), (130, 33, 60, 20),
                                            (129, 37, 200, 70), (7, 600, 40, 12)])
def test_scores(E, F, Ec, m, longest):
    rng = np.random.default_rng(F * Ec)
    n = 700

    def make(count, planes):
        rows = [np.sort(rng.choice(n, size=int(rng.integers(0, n)), replace=False))
                for _ in range(count)]
        cols = [rng.integers(0, m, size=int(rng.integers(1, longest + 1))).astype(np.int32)
                for _ in range(count)]                # columns repeat; they count once
        masks = synth.rows_to_masks(rows, n)
        if planes == 2:
            masks = np.stack([masks, masks & np.uint64(0xF0F0)], axis=1)
        off, flat = synth.pack_cbf([list(c) for c in cols])
        return list(zip(rows, cols)), tuple(_dev(x) for x in (masks, off, flat))

    fo, fs = make(F, 2)
    eo, es = make(Ec, 1)
    print(f"[report] scores F={F} E={Ec} longest={longest}", flush=True)
    sys.stdout.flush()
    J, rec, rel = E.match_scores(fs, es, n)
    Jr, rec_r, rel_r = oscores.match_scores(fo, eo)
    assert np.array_equal(J.cpu().numpy().view(np.int64), Jr.view(np.int64))
    assert np.float64(rec).view(np.int64) == np.float64(rec_r).view(np.int64)
    assert np.float64(rel).view(np.int64) == np.float64(rel_r).view(np.int64)
