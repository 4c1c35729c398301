"""Every call on rows at the edges of the row copies' and folds' slices (one
chunk per lane up to 64 chunks of 16 bytes, three from 129 to 192, else two),
with fewer and more slots than folding waves, and rows of many slices, bit for
bit against the oracle; packs larger than the memory-side cache, which move
the rows in shapes of their own; and fp32 sums stored in either way."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_random_shapes as shapes
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


@pytest.mark.parametrize("nch", [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 384, 512,
                                 640, 896, 2049, 2176])
@pytest.mark.parametrize("K,N", [(1, 3), (2, 2), (3, 2), (7, 3), (8, 3), (16, 9)])
def test_row_width(nch, K, N):
    shapes.test_random_shape(N, 2, 18 if N != 2 else 20, 18, K, 37, 8 * nch, "ragged", nch + K)


# rows of more than 2048 chunks whose combine needs no workgroup per token:
# eight slots and others, few waves and (K > 12) many, a short last slice, and
# the same split into many launches
@pytest.mark.parametrize("T,nch", [(70, 2049), (64, 2113), (64, 4096), (130, 2176)])
@pytest.mark.parametrize("K", [8, 9, 13, 16])
@pytest.mark.parametrize("limit", [None, 1 << 16])
def test_wide_row(T, nch, K, limit, monkeypatch):
    if limit:
        monkeypatch.setenv("COBALT_MAX_LAUNCH_ITEMS", str(limit))
    shapes.test_random_shape(3, 2, 18, 18, K, T, 8 * nch, "ragged", nch + K)


# outputs of more than 256 MiB: every K with 1 KiB slices (two rows per wave
# from K = 3), rows of an odd number of KiB, of no power of two, of no whole
# KiB; equal blocks of sources with buckets of 16 MiB, and sources given
@pytest.mark.parametrize("K,d", [(1, 2048), (2, 2560), (3, 2048), (3, 2560), (6, 2048), (6, 3072),
                                 (8, 4096), (10, 2560), (16, 2048), (16, 2560), (8, 2056)])
@pytest.mark.parametrize("ragged", [False, True])
def test_large_pack(K, d, ragged):
    G = 8
    T = 1 << 14 if (K, d) == (8, 4096) else ((1 << 28) // (K * d * 2) // G + 3) * G
    print(f"large pack T={T} K={K} d={d} ragged={ragged}", flush=True)
    rng = np.random.default_rng(K + d)
    a = rng.integers(0, G, (T, K)).astype(np.int32)
    if ragged:
        a[rng.random((T, K)) < 0.01] = -1    # skipped slots
    a = torch.from_numpy(a).cuda()
    src = torch.from_numpy(np.sort(rng.integers(0, G, T)).astype(np.int32)).cuda() if ragged else None
    x = torch.randint(-2**15, 2**15, (T, d), dtype=torch.int16, device="cuda")
    packed = torch.full((T * K, d), 0x7fff, dtype=torch.int16, device="cuda")
    counts = torch.empty(G, G, dtype=torch.int32, device="cuda")
    offsets = torch.empty(G * G + 1, dtype=torch.int64, device="cuda")
    pos = torch.empty(T, K, dtype=torch.int32, device="cuda")
    B.cobalt_dispatch_pack(a, src, G, x.view(torch.bfloat16), counts, offsets, pos,
                           packed.view(torch.bfloat16), B.workspace_for(T, K, G))
    placed = int(offsets[-1])
    assert placed == int((a >= 0).sum())
    # token of each row: pos names every row up to `placed` once
    token = torch.full((T * K,), -1, dtype=torch.int64, device="cuda")
    flat = pos.view(-1).long()
    token[flat[flat >= 0]] = torch.arange(T, device="cuda").repeat_interleave(K)[flat >= 0]
    assert bool((token[:placed] >= 0).all()) and bool((token[placed:] < 0).all())
    assert torch.equal(packed[:placed], x[token[:placed]])
    assert bool((packed[placed:] == 0x7fff).all())


# y_f32 below 2 MiB (5 rows of a chunk; 1.98 MB, 2.03 MB); of 40 to 256 MiB (42
# MB, a row of 129 chunks; 43 MB, a row of 1025; 42 and 268 MB), but not for
# short rows of many slots or many slots at all; others
@pytest.mark.parametrize("T,K,d", [(5, 12, 8), (510, 6, 1016), (517, 6, 1016), (3, 16, 1544),
                                   (10304, 2, 1032), (1300, 4, 8200), (20480, 4, 512),
                                   (32768, 1, 2048), (20480, 8, 512), (5200, 12, 2048),
                                   (5200, 13, 2048), (32800, 1, 2048)])
def test_fp32_sums(T, K, d):
    print(f"fp32 sums T={T} K={K} d={d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + K + d)
    eo = torch.randn(T * K, d, device="cuda", generator=g).bfloat16()
    pos = torch.randperm(T * K, device="cuda", generator=g).int().view(T, K)
    gates = torch.rand(T, K, device="cuda", generator=g)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    y32 = torch.full((T, d), float("nan"), device="cuda")
    B.cobalt_combine(eo, pos, gates, y, y32)
    assert torch.equal(y, y32.bfloat16())
    t = torch.cat([torch.arange(3), torch.randint(0, T, (40,)), torch.arange(T - 3, T)]).cuda()
    rows = eo[pos[t].long().view(-1)].view(torch.int16).cpu().numpy().view(np.uint16)
    ref, ref32 = oracle.combine(rows, np.arange(len(t) * K, dtype=np.int32).reshape(-1, K),
                                gates[t].cpu().numpy())
    assert np.array_equal(y[t].view(torch.int16).cpu().numpy().view(np.uint16), ref)
    assert np.array_equal(y32[t].cpu().numpy().view(np.uint32), ref32.view(np.uint32))
