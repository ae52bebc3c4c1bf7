"""GPU: row lists without a capacity hold their own entries and no more, on
torch's current stream and on another one."""
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


# shares of the rows listed: nothing, less and more than a quarter, all
@pytest.mark.parametrize("share", [0.0, 0.1, 0.6, 1.0])
@pytest.mark.parametrize("other_stream", [False, True])
def test_exact_storage(E, share, other_stream):
    import torch
    rng = np.random.default_rng(int(share * 10))
    n = 3000
    rows = [np.sort(rng.choice(n, size=int(share * n), replace=False)) for _ in range(7)]
    masks = synth.rows_to_masks(rows, n)[:, None, :]
    d = torch.from_numpy(masks.view(np.int64)).to("cuda:0")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if other_stream else None
    print(f"[rows] share={share} other={other_stream}", flush=True)
    off, got = E.mask_rows(d, n, stream=stream)
    if stream is not None:
        stream.synchronize()
    want = np.concatenate(oscores.mask_rows(masks, n))
    assert np.array_equal(got.cpu().numpy(), want)
    assert off.cpu().tolist() == [i * int(share * n) for i in range(8)]
    assert got.untyped_storage().nbytes() <= 4 * max(len(want), 1)
