"""GPU: populations whose workgroups need more or less than the staging area
that the launch sizes for them, against the CPU oracle, bit for bit: at the
area's smallest and largest size, one entry more, and where only some
workgroups exceed it and read their columns from memory."""
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


def _matrix(rng, n, m, ties):
    a = rng.standard_normal((n, m)).astype(np.float32)
    if ties == "few":
        a[n // 2, 1] = a[n // 2, 0]
    elif ties == "some":
        a[: m // 3, ::3] = 0.5                 # a ninth of the pairs
    elif ties == "many":
        a = np.round(a).astype(np.float32)
    return a


def _device(ctx, off, cols, k, neg, slack=0):
    import torch
    P = len(off) - 1
    cols = np.concatenate([cols, np.full(slack, -7, dtype=np.int32)])
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
    if "masks" in ref:
        assert np.array_equal(got["masks"], ref["masks"])


def _pack(rng, m, lengths):
    return synth.pack_cbf([rng.choice(m, size=int(L), replace=False) for L in lengths])


# 64 one-word series per workgroup: 2048 entries at length 32, 4096 at 64
@pytest.mark.parametrize("lengths", [[24] * 130, [32] * 64, [33] * 129, [64] * 70, [65] * 70,
                                     [70] * 40 + [3] * 400, [2] * 300 + [66] * 64])
@pytest.mark.parametrize("ties", ["none", "few", "some", "many"])
def test_one_word(ebic, lengths, ties):
    rng = np.random.default_rng(len(lengths) + lengths[0])
    a = _matrix(rng, 61, 75, ties)
    off, cols = _pack(rng, 75, lengths)
    with ebic.Context(a, path="index") as ctx:
        for k in (0, 1, 3, 6):
            for neg in (False, True):
                print(f"[staging] {lengths[0]}x{len(lengths)} {ties} k={k} neg={neg}", flush=True)
                sys.stdout.flush()
                ref = oracle.evaluate(a, off, cols, sigma=4, max_violations=k,
                                      negative_trends=neg, want_masks=True)
                _same(_device(ctx, off, cols, k, neg), ref)
        # room past the last series counts into the area's size only
        _same(_device(ctx, off, cols, 6, True, slack=40000), ref)


@pytest.mark.parametrize("ties", ["none", "few"])
def test_repeated_columns_from_memory(ebic, ties):
    # series past the area that repeat a column right after itself: such a
    # pair breaks both trends on every row, with or without tied pairs
    rng = np.random.default_rng(8)
    a = _matrix(rng, 60, 9, ties)
    pop = [list(rng.integers(0, 9, size=80)) for _ in range(70)]
    off, cols = synth.pack_cbf(pop)
    with ebic.Context(a, path="index") as ctx:
        for k in (1, 3, 40):
            got = _device(ctx, off, cols, k, True)
            for c, series in enumerate(pop):
                v = a[:, series]
                up = (~(v[:, :-1] < v[:, 1:])).sum(1) <= k
                down = (~(v[:, :-1] > v[:, 1:])).sum(1) <= k
                assert got["counts"][c] == (up | down).sum()


# unroll, words per lane, whole candidates; 512 rows are one lane's words at 8
# words per lane: 256 series per workgroup
@pytest.mark.parametrize("shape", [(2, 8, 1), (2, 8, 0), (1, 8, 1), (4, 4, 1), (8, 2, 0), (4, 1, 1)])
@pytest.mark.parametrize("ties", ["none", "some"])
def test_batch_shapes(ebic, shape, ties):
    rng = np.random.default_rng(sum(shape))
    rows = (60, 512, 513, 1500)
    mats = [_matrix(rng, n, 40, ties) for n in rows]
    pops = {L: [_pack(rng, 40, rng.integers(1, L + 1, size=600)) for _ in rows]
            for L in (6, 20, 40)}
    with ebic.Batch(mats) as b:
        for graph in (0, 1):
            b.set_tuning(-1, *shape, use_graph=graph)
            # (the area grows from one call to the next, and shrinks)
            for L in (6, 40, 20):
                for k, neg in ((0, False), (1, True), (3, True)):
                    print(f"[staging] batch {shape} {ties} graph={graph} L={L} k={k}", flush=True)
                    got = b.evaluate(pops[L], sigma=4, max_violations=k, negative_trends=neg)
                    for a, (o, c), g in zip(mats, pops[L], got):
                        _same(g, oracle.evaluate(a, o, c, sigma=4, max_violations=k,
                                                 negative_trends=neg))
