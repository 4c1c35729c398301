"""Workspace sizes over the calls that one buffer may serve: a program
allocates once, for its largest call, and then makes smaller ones. The
sizes asked for statistics do not fall as T or K grows, those for replica
loads not as any of T, K, E and G grows."""
import pytest

from paper_2609_36959_amd import binding as B

# around every multiple of the largest uint16 chunk and the ends of the plan's
# ranges, and a ladder over the rest
CHUNKS = (1, 2, 16, 17, 31, 32, 64, 127, 128, 129)
STEPS = sorted({m * n + d for m in (255, 511, 1023, 1024, 4095, 4096) for n in CHUNKS
                for d in (-1, 0, 1)} | {int(256 * 1.01 ** i) for i in range(830)} | {0, 1})
# around every number of pairs where a chunk is added (16384 each), and the
# end of uint16 counts (64 chunks of 65535 pairs)
LOAD_STEPS = sorted({16384 * n // K + d for n in [*range(1, 66), 255, 256, 257] for K in (1, 8, 16)
                     for d in (-1, 0, 1)} | {1, 100})


@pytest.mark.parametrize("E", [1, 2, 16, 100, 128, 129, 200, 256, 300, 384, 512, 700, 1024, 1500,
                               2048, 3000, 4096])
def test_statistics_workspace_serves_smaller_calls(E):
    by_k = []
    for K in (k for k in (1, 2, 6, 8, 16) if k <= E):
        sizes = [B.cobalt_coact_stats_workspace_bytes(T, K, E) for T in STEPS]
        falls = [(a, b) for a, b, x, y in zip(STEPS, STEPS[1:], sizes, sizes[1:]) if y < x]
        assert not falls, f"E={E} K={K}: falls between T of {falls[:5]}"
        by_k.append(sizes)
    for small, large in zip(by_k, by_k[1:]):
        assert all(x <= y for x, y in zip(small, large)), f"E={E}: falls as K grows"


@pytest.mark.parametrize("E", [1, 8, 16, 25, 31, 64, 100, 384, 1000, 4096])
def test_replica_load_workspace_serves_smaller_calls(E):
    for G in (1, 2, 3, 5, 6, 8, 12, 24, 32, 64, 65, 208, 512):
        for K in (1, 8, 16):
            sizes = [B.cobalt_replica_load_workspace_bytes(T, K, E, G) for T in LOAD_STEPS]
            falls = [(a, b) for a, b, x, y in zip(LOAD_STEPS, LOAD_STEPS[1:], sizes, sizes[1:])
                     if y < x]
            assert not falls, f"E={E} G={G} K={K}: falls between T of {falls[:5]}"
