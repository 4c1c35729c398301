"""The layouts of both dispatches at the edges of the layout kernels' ranges,
against a stable sort in numpy: whole-call workgroups up to their pair limits
(8192, or up to 32768, by the number of ranks, with source ranks given; 1024
and 4096 tokens for the node rows) and beyond, per-source tiles of 4096 pairs (512 tokens) with one pair too
many, tiles of several passes (past 1024 tiles, or 256 with source ranks
given), windows over the sources that do not fit, G up to 64 and above, ids at
addresses that allow only 4- or 8-byte reads, and workspaces of exactly the
size asked for, filled with ones."""
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


def sources(kind, T, G, rng):
    if kind == "null":
        return None
    if kind == "one":      # a process that holds one rank's tokens
        return np.full(T, G // 2, np.int32)
    return np.sort(rng.integers(0, G, T)).astype(np.int32)


def on_device(a, shift):
    """a on the device, `shift` ints past a 256-byte boundary."""
    buf = torch.empty(a.size + shift, dtype=torch.int32, device="cuda")
    out = buf[shift:].view(a.shape)
    out.copy_(torch.from_numpy(a))
    return out


CASES = [
    # T, K, N, g, sources, shift
    (1, 1, 1, 1, "null", 0),
    (1, 16, 16, 32, "any", 0),
    (128, 8, 8, 8, "null", 1),           # 1024 pairs: one tile of a whole-call workgroup
    (129, 8, 3, 5, "any", 0),
    (1024, 8, 8, 8, "null", 2),          # 8192 pairs, 1024 tokens: the limits
    (1088, 8, 8, 8, "null", 0),          # beyond: per-source tiles
    (4096, 8, 8, 8, "any", 0),           # 32768 pairs, 4096 tokens: the limits with sources
    (4097, 8, 8, 8, "any", 4),
    (4097, 8, 8, 8, "one", 0),
    (8192, 1, 1, 1, "any", 0),           # 8192 pairs: the limit for one rank
    (8193, 1, 1, 1, "any", 0),
    (70001, 3, 1, 1, "any", 1),          # one rank, several tiles
    (2133, 6, 2, 1, "any", 0),           # 12798 and 12804 pairs, two ranks: 12800
    (2134, 6, 1, 2, "any", 1),
    (3328, 8, 2, 4, "any", 0),           # 26624 pairs: the limit for eight ranks
    (3329, 8, 2, 4, "one", 0),
    (8192, 1, 4, 2, "null", 0),
    (1040, 16, 13, 5, "null", 0),        # G = 65: no whole-call workgroups
    (1025, 16, 13, 5, "any", 0),         # first rows from the scan kernel
    (512, 7, 16, 32, "null", 0),         # G = 512, seven pairs a source
    (4099, 6, 16, 32, "any", 1),         # a window of 512 x 512 does not fit
    (4096 * 3, 1, 3, 1, "null", 0),      # a full tile per source
    (4097 * 3, 1, 3, 1, "null", 0),      # one pair in a second tile
    (4096 + 1, 6, 1, 1, "null", 0),
    (4096 * 4, 6, 4, 8, "null", 2),      # 8-byte reads
    (4096 * 2, 6, 2, 4, "any", 0),
    (8192, 12, 1, 32, "one", 0),         # one node: every token one row
    (540672, 8, 8, 8, "null", 0),        # 4.3 M pairs: passes of 4096 in tiles of 8192
    (530001, 4, 2, 3, "any", 0),         # 2.1 M pairs: 256 tiles of three passes
    (300000, 16, 5, 5, "one", 0),
]


@pytest.mark.parametrize("T,K,N,g,kind,shift", CASES)
def test_layouts(T, K, N, g, kind, shift):
    print(f"layouts T={T} K={K} N={N} g={g} sources={kind} shift={shift}", flush=True)
    G = N * g
    rng = np.random.default_rng(T + K)
    a = np.minimum(rng.integers(0, G, (T, K)), rng.integers(0, G, (T, K))).astype(np.int32)
    a[rng.random((T, K)) < 0.01] = -1    # skipped slots
    src = sources(kind, T, G, rng)
    t_a = on_device(a, shift)
    t_src = None if src is None else on_device(src, 1)

    def workspace(n):
        return torch.full((n,), 255, dtype=torch.uint8, device="cuda")

    counts = torch.full((G, G), -9, dtype=torch.int32, device="cuda")
    offsets = torch.full((G * G + 1,), -9, dtype=torch.int64, device="cuda")
    pos = torch.full((T, K), -9, dtype=torch.int32, device="cuda")
    B.cobalt_dispatch_pack(t_a, t_src, G, None, counts, offsets, pos, None,
                           workspace(B.cobalt_dispatch_workspace_bytes(T, K, G)))
    cap = T * min(K, N)
    ncounts = torch.full((G, N), -9, dtype=torch.int32, device="cuda")
    noffsets = torch.full((G * N + 1,), -9, dtype=torch.int64, device="cuda")
    npos = on_device(np.full((T, N), -9, np.int32), shift)
    fwd = torch.full((cap,), -9, dtype=torch.int32, device="cuda")
    tok = torch.full((cap,), -9, dtype=torch.int32, device="cuda")
    B.cobalt_node_dispatch_pack(t_a, t_src, N, g, None, ncounts, noffsets, npos, fwd, tok, None,
                                workspace(B.cobalt_node_dispatch_workspace_bytes(T, N, g)))
    torch.cuda.synchronize()

    # the pairs with a rank, stably sorted by bucket
    s = np.arange(T) // max(1, T // G) if src is None else src
    ok = a >= 0
    key = (s[:, None].astype(np.int64) * G + a)[ok]
    want = np.full(T * K, -1, np.int64)
    order = np.argsort(key, kind="stable")
    rows = np.empty(order.size, np.int64)
    rows[order] = np.arange(order.size)
    want[ok.ravel()] = rows
    hist = np.bincount(key, minlength=G * G)
    assert np.array_equal(counts.cpu().numpy().ravel(), hist)
    assert np.array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(hist)]))
    assert np.array_equal(pos.cpu().numpy().ravel(), want)

    # the rows (t, n), sorted by source, node and token
    reach = np.zeros((T, N), bool)
    mask = np.zeros((T, N), np.uint32)
    for j in range(K):
        t = np.nonzero(ok[:, j])[0]
        n = a[t, j] // g
        reach[t, n] = True
        mask[t, n] |= np.uint32(1) << (a[t, j] % g).astype(np.uint32)
    t, n = np.nonzero(reach)
    order = np.lexsort((t, n, s[t]))
    node_rows = np.full((T, N), -1, np.int64)
    node_rows[t[order], n[order]] = np.arange(order.size)
    nhist = np.bincount(s[t].astype(np.int64) * N + n, minlength=G * N)
    assert np.array_equal(ncounts.cpu().numpy().ravel(), nhist)
    assert np.array_equal(noffsets.cpu().numpy(), np.concatenate([[0], np.cumsum(nhist)]))
    assert np.array_equal(npos.cpu().numpy(), node_rows)
    assert np.array_equal(tok.cpu().numpy()[:order.size], t[order])
    assert np.array_equal(fwd.cpu().numpy().view(np.uint32)[:order.size], mask[t, n][order])
    assert (tok.cpu().numpy()[order.size:] == -9).all()
