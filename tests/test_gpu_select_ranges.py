"""celty_select at the edges of its workgroups' ranges: lists are bit-exact
against the oracle where a range is full, holds one column, follows part of an
8192-column count, takes two steps (K > 64 * 2048) and two chunks (K >
16 * 64 * 2048), with every column active (tau < 0, also the zeros past K in
the last word), none, a share, and NaN activations."""
import numpy as np
import pytest

from oracle import spmspv as ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1025, 2047, 2048, 2049, 8193, 10240, 10241, 28672, 34816, 131072, 131073, 2097153, 2200001])
@pytest.mark.parametrize("tau", [-1.0, 0.7, 1e4])
def test_select_ranges(K, tau):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_01536_amd as celty
    print(f"select ranges K={K} tau={tau}", flush=True)
    rng = np.random.default_rng(K)
    x = rng.laplace(size=K).astype(np.float16)
    x[rng.integers(0, K, size=5)] = np.float16(np.nan)
    x[[0, K - 1]] = np.float16(3.0)
    xt = torch.from_numpy(x.view(np.int16)).cuda()
    idx = torch.full((K,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    celty.celty_select(xt, tau, idx, cnt)
    torch.cuda.synchronize()
    want = ref.select_active(x, tau)
    n = int(cnt.item())
    got = idx.cpu().numpy()
    assert n == len(want)
    assert np.array_equal(got[:n], want)
    assert np.all(got[n:] == -7)
