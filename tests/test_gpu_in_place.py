"""Outputs in the memory of inputs that the call has no more use for: assigned
ranks over the expert ids, rows over the assigned ranks or (K = 1) over
the sources, and the node-level combine's y over the expert rows. Each gives
what the same call with buffers of its own gives, on small calls (whole-call
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


@pytest.mark.parametrize("T,K,N,g,d", [(96, 2, 3, 2, 8), (520, 8, 4, 2, 1032), (3000, 4, 2, 4, 2048)])
def test_node_combine_over_expert_rows(T, K, N, g, d):
    print(f"node combine over expert rows T={T} K={K} N={N} d={d}", flush=True)
    G = N * g
    gen = torch.Generator(device="cuda").manual_seed(T)
    assigned = torch.randint(0, G, (T, K), device="cuda", generator=gen).int()
    src = torch.from_numpy(W.ragged_src(T, G, 1)).cuda()
    pos = torch.empty(T, K, dtype=torch.int32, device="cuda")
    B.cobalt_dispatch_pack(assigned, src, G, None,
                           torch.empty(G, G, dtype=torch.int32, device="cuda"),
                           torch.empty(G * G + 1, dtype=torch.int64, device="cuda"), pos, None,
                           B.workspace_for(T, K, G))
    node_pos = torch.empty(T, N, dtype=torch.int32, device="cuda")
    cap = T * min(K, N)
    B.cobalt_node_dispatch_pack(assigned, src, N, g, None,
                                torch.empty(G, N, dtype=torch.int32, device="cuda"),
                                torch.empty(G * N + 1, dtype=torch.int64, device="cuda"), node_pos,
                                torch.empty(cap, dtype=torch.int32, device="cuda"), None, None,
                                B.node_workspace_for(T, N, g))
    eo = torch.randn(T * K, d, device="cuda", generator=gen).bfloat16()
    gates = torch.rand(T, K, device="cuda", generator=gen)
    partial = [torch.zeros(cap, d, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    y = torch.empty(T, d, dtype=torch.bfloat16, device="cuda")
    B.cobalt_node_combine(eo, pos, assigned, gates, node_pos, N, g, partial[0], y)
    for p, first in ((partial[1], 0), (partial[2], T * K - T)):
        rows = eo.clone()
        B.cobalt_node_combine(rows, pos, assigned, gates, node_pos, N, g, p, rows[first:first + T])
        assert torch.equal(rows[first:first + T].view(torch.int16), y.view(torch.int16))
        assert torch.equal(p.view(torch.int16), partial[0].view(torch.int16))
