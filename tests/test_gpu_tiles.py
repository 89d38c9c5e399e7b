"""The mask passes at every tile length (16, 4 or 1 rounds of 64 nodes, chosen by the graph's
size) and in both layouts of the count matrix, on both sides of their steps, against the oracle;
and the longest tiles, which take the smaller workspaces, against the chosen ones (tolerance 0)."""
import re

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


# the matrix is block-major from 4096 blocks of 4096 nodes on, in chunks of 64 blocks
@pytest.mark.parametrize("n,B", [(n, B) for n in (1, 255, 257, 4097, 499_999, 500_000, 1_000_003,
                                                  3_999_999, 4_000_001) for B in (3, 64)]
                         + [(4095 * 4096, 64), (4095 * 4096 + 1, 64), (4160 * 4096 + 1, 3)])
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
    # workspaces of the least size take the longest tiles
    if n < 4_000_000:
        for form in forms:
            check(*with_least(dg, form, monkeypatch))


def with_least(dg, form, monkeypatch):
    """form() with the smallest workspaces its calls take (sampling's, packing's)."""
    sizes = [256, 256]
    for _ in range(3):
        at = iter(sizes)
        monkeypatch.setattr(dg, "_workspace", lambda nbytes, d, ws: torch.empty(
            next(at), dtype=torch.uint8, device=d))
        try:
            return form()
        except dg.DGError as e:
            need = re.search(r"workspace needs (\d+) bytes", str(e))
            sizes[1 if "dg_pack_group:" in str(e) or "packing" in str(e) else 0] = int(need[1])
    raise AssertionError(sizes)


@pytest.mark.big
def test_packing_of_more_chunks_than_one_step_of_their_scan(dg):
    """540M nodes: 131,837 blocks, 2,060 chunks (a step of the chunks' scan takes 2,048)."""
    n, B = 540_000_000, 3
    g = torch.Generator(device=DEV).manual_seed(5)
    lists = [torch.randint(0, n, (k,), device=DEV, generator=g).unique() for k in
             (300_000, 5, 2_000_000)]
    lists = [torch.cat([torch.tensor([0, n - 1], device=DEV), u]).unique() for u in lists]
    stride = max(u.numel() for u in lists)
    nodes = torch.zeros((B, stride), dtype=torch.int32, device=DEV)
    order = [torch.randperm(u.numel(), device=DEV, generator=g) for u in lists]
    for b, u in enumerate(lists):
        nodes[b, :u.numel()] = u[order[b]].int()
    feats = torch.randint(0, 256, (n, 1), dtype=torch.uint8, device=DEV, generator=g)
    slot = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    slot[lists[0][::7]] = torch.arange(lists[0][::7].numel(), dtype=torch.int32, device=DEV)
    pr = dg.pack_group(feats, slot, nodes, [u.numel() for u in lists], with_unique=True)
    u_all = torch.cat(lists).unique()
    assert pr.sizes["unique_nodes"] == u_all.numel()
    assert torch.equal(pr.unique.long(), u_all)
    for b, u in enumerate(lists):
        lo, hi = int(pr.packed_ptr_host[b]), int(pr.packed_ptr_host[b + 1])
        p_b = u[slot[u] < 0]
        assert torch.equal(pr.packed_ids[lo:hi].long(), p_b), b
        assert torch.equal(pr.packed[lo:hi], feats[p_b]), b
        v = u[order[b]]
        loc = torch.where(slot[v] >= 0, -slot[v].long() - 1, torch.searchsorted(p_b, v))
        assert torch.equal(pr.loc[b, :u.numel()].long(), loc), b
