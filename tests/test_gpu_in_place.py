"""Outputs in the memory of inputs that the call has no more use for: assigned
ranks over the expert ids, rows over the assigned ranks or (K = 1) over the
sources. Each gives what the same call with buffers of its own gives, on small calls (whole-call
workgroups) and larger ones, with sources in equal blocks and given."""
import pytest
import torch

from paper_2609_36959_amd import binding as B
from paper_2609_36959_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    B.lib()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,K,N,g", [(512, 8, 4, 4), (1024, 4, 4, 8), (6400, 4, 4, 8),
                                     (70400, 4, 4, 2)])
@pytest.mark.parametrize("ragged", [False, True])
def test_rows_over_ranks(T, K, N, g, ragged):
    print(f"rows over ranks T={T} K={K} N={N} g={g} ragged={ragged}", flush=True)
    G = N * g
    w = W.Workload("in-place", T, 64, K, 8, N, g, 64 // G + 1, zipf_alpha=1.0)
    topk, _ = W.routing(w, 1, device="cuda")
    table, owner = W.layout(w, 1)
    layout = B.cobalt_layout_create(N, g, w.E, table.shape[1], table, owner)
    src = torch.from_numpy(W.ragged_src(T, G, 1)).cuda() if ragged else None
    assigned = torch.empty(T, K, dtype=torch.int32, device="cuda")
    B.cobalt_assign(layout, topk, src, 5, 0, 0, assigned)
    over = topk.clone()
    B.cobalt_assign(layout, over, src, 5, 0, 0, over)
    assert torch.equal(over, assigned)

    ws = B.workspace_for(T, K, G)
    def dispatch(a, s, pos):
        counts = torch.empty(G, G, dtype=torch.int32, device="cuda")
        offsets = torch.empty(G * G + 1, dtype=torch.int64, device="cuda")
        B.cobalt_dispatch_pack(a, s, G, None, counts, offsets, pos, None, ws)
        return counts, offsets, pos
    want = dispatch(assigned, src, torch.empty_like(assigned))
    got = dispatch(over, src, over)
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    if ragged:
        one = assigned[:, :1].contiguous()
        want = dispatch(one, src, torch.empty_like(one))
        s = src.clone()
        got = dispatch(one, s, s.view(T, 1))
        assert all(torch.equal(a, b) for a, b in zip(want, got))

    nws = B.node_workspace_for(T, N, g)
    def node(a, s, node_pos):
        counts = torch.empty(G, N, dtype=torch.int32, device="cuda")
        offsets = torch.empty(G * N + 1, dtype=torch.int64, device="cuda")
        fwd = torch.zeros(T * min(K, N), dtype=torch.int32, device="cuda")
        B.cobalt_node_dispatch_pack(a, s, N, g, None, counts, offsets, node_pos, fwd, None, None,
                                    nws)
        return counts, offsets, fwd, node_pos
    if N == K:
        want = node(assigned, src, torch.empty(T, N, dtype=torch.int32, device="cuda"))
        over = assigned.clone()
        got = node(over, src, over)
        assert all(torch.equal(a, b) for a, b in zip(want, got))
