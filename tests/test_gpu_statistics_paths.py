"""The statistics at the edges of their dispatch, against A^T A of the tokens'
multiplicity matrix: the last call whose workgroups add to coact directly and
the first with a reduce (by chunks and by E), few and many chunks, the cap on
workgroups with many bands (and where it gives way, so that the bins are
uint16), every width of the id loads (K and address), K that fills the
registers and K that does not; a few tokens repeat an id or hold one out of
range."""
import numpy as np
import pytest
import torch

from paper_2609_36959_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    B.lib()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,E,K,shift", [
    (1, 1, 1, 0), (255, 2, 2, 0), (513, 16, 2, 1), (700, 7, 3, 0),
    (4351, 128, 8, 0), (4352, 128, 8, 0),   # 16 and 17 chunks of 256: the direct limit
    (4096, 129, 8, 2),                      # E past the direct limit
    (16383, 64, 6, 0), (16640, 64, 6, 2), (5000, 100, 5, 0), (5000, 100, 7, 1),
    (3000, 40, 12, 0), (3000, 40, 16, 4), (1500, 60, 13, 0), (2000, 50, 10, 2),
    (16895, 200, 8, 0), (17000, 200, 8, 0),  # 32 and 33 chunks of 512: lanes of the reduce
    (131072, 300, 4, 0),
    (20000, 1024, 8, 0),                    # 16 bands: chunks capped at 16
    (70000, 1024, 8, 0),                    # 18 chunks, so that the bins are uint16
    (140001, 1024, 8, 0),                   # 16 chunks of uint32 bins
    (140000, 1024, 16, 0),
    (4096, 1500, 6, 0),
])
def test_statistics(T, E, K, shift):
    print(f"statistics T={T} E={E} K={K} shift={shift}", flush=True)
    rng = np.random.default_rng(T + E + K)
    # distinct ids with a skew, from a random order of the experts per token
    topk = np.argsort(rng.random((T, E)) * (1 + np.arange(E)), axis=1)[:, :K] if E <= 300 else \
        (rng.integers(0, E, (T, 1)) + np.cumsum(rng.integers(1, max(2, E // K), (T, K)), 1)) % E
    topk = topk.astype(np.int32)
    odd = rng.random(T) < 0.002
    topk[odd] = rng.integers(-1, E + 1, (int(odd.sum()), K))
    buf = torch.empty(T * K + shift, dtype=torch.int32, device="cuda")
    t = buf[shift:].view(T, K)
    t.copy_(torch.from_numpy(topk))
    start = rng.integers(0, 1000, (E, E)).astype(np.int32)
    coact = torch.from_numpy(start).cuda()
    count = torch.full((E,), 5, dtype=torch.int32, device="cuda")
    ws = torch.full((B.cobalt_coact_stats_workspace_bytes(T, K, E),), 255, dtype=torch.uint8,
                    device="cuda")
    B.cobalt_coact_stats(t, E, coact, count, ws)
    torch.cuda.synchronize()

    want = torch.zeros(E, E, dtype=torch.float64)
    wcount = torch.zeros(E, dtype=torch.float64)
    for a in range(0, T, 8192):
        ids = torch.from_numpy(topk[a:a + 8192].astype(np.int64))
        ok = (ids >= 0) & (ids < E)
        A = torch.zeros(len(ids), E + 1)
        A.scatter_add_(1, torch.where(ok, ids, E), torch.ones(ids.shape))
        A = A[:, :E]
        c = A.sum(0).double()
        want += A.t().mm(A).double() - torch.diag(c)   # whole numbers below 2^24: exact
        wcount += c
    assert np.array_equal(coact.cpu().numpy() - start, want.numpy().astype(np.int32))
    assert np.array_equal(count.cpu().numpy() - 5, wcount.numpy().astype(np.int32))
