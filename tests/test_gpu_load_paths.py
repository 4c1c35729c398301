"""Replica loads where the bands begin at multiples of eight bins in different
ways (G odd, twice or four times odd, a multiple of eight), the last band is
short or single, chunks are one, few and all, pairs come with and without
16-byte loads, against numpy's histogram; in a workspace held for a larger
call, with bytes on both sides that have to stay as they are."""
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


@pytest.mark.parametrize("T,K,shift", [(1, 1, 0), (5, 3, 0), (4096, 8, 0), (7001, 7, 1),
                                       (58000, 8, 0), (60000, 8, 2), (140000, 8, 0)])
@pytest.mark.parametrize("E,G", [(1, 1), (17, 1), (300, 3), (31, 2), (25, 6), (100, 4), (64, 32),
                                 (37, 24), (384, 64), (130, 125), (70, 512), (4096, 9)])
def test_replica_load(T, K, shift, E, G):
    print(f"loads T={T} K={K} shift={shift} E={E} G={G}", flush=True)
    rng = np.random.default_rng(T + E + G)
    topk = np.minimum(rng.integers(-1, E + 1, (T, K)), rng.integers(0, E + 1, (T, K)))
    ranks = rng.integers(-1, G + 1, (T, K))

    def device(a):
        buf = torch.empty(a.size + shift, dtype=torch.int32, device="cuda")
        buf[shift:].copy_(torch.from_numpy(a.astype(np.int32)).view(-1))
        return buf[shift:].view(a.shape)

    load = torch.full((E, G), 3, dtype=torch.int32, device="cuda")
    need = B.cobalt_replica_load_workspace_bytes(T, K, E, G)
    held = B.cobalt_replica_load_workspace_bytes(T + 7000, K, E, G)
    buf = torch.full((256 + held + 256,), 255, dtype=torch.uint8, device="cuda")
    B.cobalt_replica_load(device(topk), device(ranks), E, G, load, buf[256:256 + held])
    torch.cuda.synchronize()
    ok = (topk >= 0) & (topk < E) & (ranks >= 0) & (ranks < G)
    want = np.bincount((topk * G + ranks)[ok], minlength=E * G).reshape(E, G)
    assert np.array_equal(load.cpu().numpy() - 3, want)
    assert bool((buf[:256] == 255).all()) and bool((buf[256 + need:] == 255).all())
