"""The mask passes at every tile length (16, 4 or 1 rounds of 64 nodes, chosen by the graph's
size) and on both sides of its steps, against the oracle; and the longest tiles, which take the
smaller workspaces, against the chosen ones (tolerance 0)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def dg():
    import paper_2405_05231_amd as m
    return m


def graph(n, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 9, n)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=off[1:])
    # a quarter of the edges lead to a few hubs, so that words with many bits occur
    idx = rng.integers(0, n, off[-1]).astype(np.int32)
    hub = rng.random(idx.size) < 0.25
    idx[hub] = rng.integers(0, max(1, n // 50), int(hub.sum()))
    return off, idx


def dev(x):
    return torch.from_numpy(x).to(DEV)


@pytest.mark.parametrize("n", [1, 255, 257, 4097, 499_999, 500_000, 1_000_003, 3_999_999,
                               4_000_001])
@pytest.mark.parametrize("B", [3, 64])
def test_every_tile_length(dg, orc, n, B, monkeypatch):
    off, idx = graph(n, n + B)
    rng = np.random.default_rng(n)
    S = min(40, n)
    seeds = np.stack([rng.choice(n, S, replace=False) for _ in range(B)]).astype(np.int32)
    slot = np.full(n, -1, dtype=np.int32)
    cached = rng.choice(n, n // 5, replace=False)
    slot[cached] = np.arange(cached.size, dtype=np.int32)
    feats = rng.integers(0, 255, (n, 16)).astype(np.uint8)
    fan = [4, 3, 5]
    ref = orc.sample_group(off, idx, seeds, fan, 77)
    refp = orc.pack_group(feats, slot, ref["nodes"])
    args = (dev(off), dev(idx), dev(seeds), fan, 77, dev(feats), dev(slot))

    def check(sr, pr):
        rows = refp["packed_rows"]
        assert pr.sizes["packed_rows"] == rows
        assert np.array_equal(pr.packed_ids[:rows].cpu().numpy(), refp["packed_ids"])
        assert np.array_equal(pr.packed[:rows].cpu().numpy(), refp["packed"])
        assert np.array_equal(pr.packed_ptr.cpu().numpy(), pr.packed_ptr_host)
        for b in range(B):
            k, e = int(sr.hop_ptr[b, -1]), int(sr.edge_ptr[b, -1])
            assert np.array_equal(sr.batch_nodes(b).cpu().numpy(), ref["nodes"][b])
            assert np.array_equal(sr.edge_src[b, :e].cpu().numpy(), ref["edge_src"][b])
            assert np.array_equal(sr.edge_dst[b, :e].cpu().numpy(), ref["edge_dst"][b])
            assert np.array_equal(pr.loc[b, :k].cpu().numpy(), refp["loc"][b])

    def two_calls(direct):
        mem = torch.zeros(n, dtype=torch.int64, device=DEV)
        lines = torch.full((dg.member_lines_bytes(n),), 9, dtype=torch.uint8, device=DEV)
        sr = dg.sample_group(*args[:5], membership=mem, member_lines=lines, direct=direct)
        has = torch.zeros(lines.numel() * 8, dtype=torch.bool, device=DEV)
        has[:n] = mem != 0
        assert torch.equal(lines != 0, has.view(-1, 8).any(1))
        return sr, dg.pack_group(args[5], args[6], sr.nodes, sr.node_count, membership=mem,
                                 member_lines=lines)

    def lists_only():
        sr = dg.sample_group(*args[:5], layered=False)
        return sr, dg.pack_group(args[5], args[6], sr.nodes, sr.node_count)

    forms = [lambda: dg.sample_pack_group(*args), lambda: two_calls(True), lists_only]
    for form in forms:
        check(*form())
    # workspaces too small for short tiles (below 4M nodes) take the longest ones
    if n < 4_000_000:
        monkeypatch.setattr(dg, "_workspace", lambda nbytes, d, ws: torch.empty(
            nbytes - 256, dtype=torch.uint8, device=d))
        if n <= 257:  # so small that both layouts round to the same size
            return
        for form in forms:
            check(*form())
