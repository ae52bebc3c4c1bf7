"""GPU: every place of a gradient list counts, exactly once.  All candidates
but one have their own prediction as target, so that their gradients are zero
to the bit; the embedding gradients are then the one candidate's, wherever it
stands in its columns' lists and in its length's, with one rounding each:

    dZ[L] = dx,  dE[c] = fl(dx / L),
    dF[c_t] = fl(dx' T[c_t+1] / (L - 1)),  dT[c_t+1] = fl(dx' F[c_t] / (L - 1))

With tables F and T of powers of two the pair gradients are one vector, scaled
exactly.  These relations are checked bit for bit; dx itself against the
float64 oracle with the same BF16 rounding points.  There, a sum in FP32 that
falls on the other side of a rounding point moves one of 256 terms of a
gradient by 2^-8 of itself: 2^-7 of a row's largest gradient allows for several."""
import sys

import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

D, H, L = 32, 256, 5


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_03039_amd as e
    return e


def _tables(g, M):
    out, at = {}, 0
    for name, rows in (("E", M), ("F", M), ("T", M), ("Z", M + 1)):
        out[name] = g[at:at + rows * D].reshape(rows, D)
        at += rows * D
    return out


# column 0 is in every series, so a candidate's number is its place in that
# column's list and in its length's: ends of 16 places, rows (32), rounds (256)
@pytest.mark.parametrize("B", [1, 33, 257, 700, 3000])
def test_every_place_counts_once(E, B):
    M = 40
    rng = np.random.default_rng(B)
    series = []
    for b in range(B):
        s = 1 + rng.choice(M - 1, size=L, replace=False)
        s[int(rng.integers(L))] = 0
        series.append(s)
    off = np.arange(B + 1, dtype=np.int32) * L
    cols = np.concatenate(series).astype(np.int32)
    scale = (2.0 ** -(np.arange(M) % 6)).astype(np.float32)
    places = sorted({p for p in (0, 1, 15, 16, 31, 32, 47, 48, 63, 64, 239, 240, 255, 256, 257, 271,
                                 272, 511, 512, 513, 2815, 2816, B - 33, B - 2, B - 1) if 0 <= p < B})
    with E.Mlp(M, seed=5) as net:
        p = net.params()
        t = _tables(p, M)
        t["F"][:], t["T"][:] = scale[:, None], scale[::-1][:, None]
        t["Z"][:] = 0.1 * rng.standard_normal((M + 1, D))
        net.set_params(p)
        y = net.predict(off, cols)
        for place in places:
            print(f"[places] B={B} place={place}", flush=True)
            sys.stdout.flush()
            target = y.copy()
            target[place] += np.float32(100)
            _, g = net.gradients(off, cols, target)
            _, ref, _ = omlp.loss_and_grad(p, off, cols, target, M, D, H, bf16=True)
            g, r = _tables(g, M), _tables(ref, M)
            s = series[place]
            dx = g["Z"][L]
            assert np.max(np.abs(dx - r["Z"][L])) <= 2.0 ** -7 * np.max(np.abs(r["Z"][L]))
            assert np.max(np.abs(dx)) > 0
            assert not np.delete(g["Z"], L, axis=0).any()
            for c in s:
                assert np.array_equal(g["E"][c], dx * (np.float32(1) / np.float32(L)))
            # the pair gradient, unscaled
            v = g["F"][s[0]] / scale[::-1][s[1]]
            want = r["F"][s[0]] / scale[::-1][s[1]]
            assert np.max(np.abs(v - want)) <= 2.0 ** -7 * np.max(np.abs(want)) and v.any()
            for i in range(L - 1):
                assert np.array_equal(g["F"][s[i]], v * scale[::-1][s[i + 1]])
                assert np.array_equal(g["T"][s[i + 1]], v * scale[s[i]])
            assert not g["F"][s[L - 1]].any() and not g["T"][s[0]].any()
            others = np.setdiff1d(np.arange(M), s)
            for name in "EFT":
                assert not g[name][others].any()


def _ordered(entries):
    """The kernel's sum of a list: entry o belongs to row (o / 32) mod 8, place
    o mod 32; entries of one row and place first, in list order, then a row's
    places, then the rows; an entry of None adds nothing.  In FP32."""
    v = np.zeros((8, 32, D), dtype=np.float32)
    for o, x in enumerate(entries):
        if x is not None:
            v[(o // 32) % 8, o % 32] += x
    total = np.zeros(D, dtype=np.float32)
    for row in v:
        acc = np.zeros(D, dtype=np.float32)
        for x in row:
            acc += x
        total += acc
    return total


def test_order_of_the_sums(E):
    # each candidate's dx from a call in which it alone counts, the sums of all
    # in the documented order: the same bits
    M, B = 12, 600
    rng = np.random.default_rng(4)
    series = [rng.choice(M, size=L, replace=False) for _ in range(B)]
    off = np.arange(B + 1, dtype=np.int32) * L
    cols = np.concatenate(series).astype(np.int32)
    with E.Mlp(M, seed=5) as net:
        p = net.params()
        t = _tables(p, M)
        t["F"][:], t["T"][:] = 1, 1
        t["E"][:] = rng.standard_normal((M, D))
        net.set_params(p)
        y = net.predict(off, cols)
        full = (y + 10 * rng.standard_normal(B)).astype(np.float32)
        print("[places] one candidate at a time", flush=True)
        dx, pair = [], []
        for b in range(B):
            target = y.copy()
            target[b] = full[b]
            g = _tables(net.gradients(off, cols, target)[1], M)
            dx.append(g["Z"][L].copy())
            pair.append(g["F"][series[b][0]].copy())
        g = _tables(net.gradients(off, cols, full)[1], M)
    assert np.array_equal(g["Z"][L], _ordered(dx))
    inv = np.float32(1) / np.float32(L)
    for j in range(M):
        at = [(b, int(np.nonzero(s == j)[0][0])) for b, s in enumerate(series) if j in s]
        assert np.array_equal(g["E"][j], _ordered([dx[b] * inv for b, _ in at]))
        assert np.array_equal(g["F"][j], _ordered([pair[b] if i < L - 1 else None for b, i in at]))
        assert np.array_equal(g["T"][j], _ordered([pair[b] if i > 0 else None for b, i in at]))
