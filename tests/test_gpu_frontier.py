"""Frontiers of thousands of tiles, on both sides of the length from which the tiles' sums are
scanned by a launch of their own, and of the number of seeds from which those enter by one, against
the oracle (tolerance 0)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EDGE = 8192 * 256  # entries of the longest frontier of a batch whose tiles are not scanned


@pytest.fixture(scope="module")
def dg():
    import paper_2405_05231_amd as m
    return m


def dev(x):
    return torch.from_numpy(x).to(DEV)


def check(orc, sr, off, idx, seeds, fan, layered=False):
    ref = orc.sample_group(off, idx, seeds, fan, 5, layered=layered)
    for b in range(seeds.shape[0]):
        e = int(sr.edge_ptr[b, -1])
        assert np.array_equal(sr.batch_nodes(b).cpu().numpy(), ref["nodes"][b])
        assert np.array_equal(sr.edge_src[b, :e].cpu().numpy(), ref["edge_src"][b])
        assert np.array_equal(sr.edge_dst[b, :e].cpu().numpy(), ref["edge_dst"][b])


def graph(n, rng):
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(rng.integers(0, 4, n), out=off[1:])
    return off, rng.integers(0, n, off[-1]).astype(np.int32)


@pytest.mark.parametrize("S,B,direct,layered", [(EDGE, 1, True, False), (EDGE + 1, 1, True, False),
                                                (EDGE + 1, 3, False, False),
                                                (EDGE, 4, True, False),  # 2^23 seeds: apart
                                                (EDGE - 100_000, 2, True, True)])
def test_long_frontiers(dg, orc, S, B, direct, layered):
    """The seeds fill the first hop's frontier; layered, the later hops' pass the step."""
    n = EDGE + 300_000
    rng = np.random.default_rng(S + B)
    off, idx = graph(n, rng)
    seeds = np.stack([rng.permutation(n)[:S] for _ in range(B)]).astype(np.int32)
    fan = [2, 1]
    sr = dg.sample_group(dev(off), dev(idx), dev(seeds), fan, 5, direct=direct, layered=layered)
    check(orc, sr, off, idx, seeds, fan, layered)


def test_long_frontier_beside_an_empty_one(dg, orc):
    """Batch 0's seeds have no neighbours, batch 1's lead to as many new nodes; then the same
    with one edge too few of room."""
    S = EDGE + 257
    rng = np.random.default_rng(3)
    ids = rng.permutation(3 * S).astype(np.int32)
    a, b, alone = ids[:S], ids[S:2 * S], ids[2 * S:]
    deg = np.zeros(3 * S, dtype=np.int64)
    deg[a] = 1
    deg[b] = 1
    off = np.zeros(3 * S + 1, dtype=np.int64)
    np.cumsum(deg, out=off[1:])
    idx = np.empty(2 * S, dtype=np.int32)
    idx[off[a]] = b
    idx[off[b]] = a
    seeds = np.stack([alone, a])
    args = (dev(off), dev(idx), dev(seeds), [1, 1], 5)
    sr = dg.sample_group(*args)
    check(orc, sr, off, idx, seeds, [1, 1])
    assert sr.edge_ptr[:, -1].tolist() == [0, 2 * S]
    for cap in (2 * S - 1, S - 1):
        with pytest.raises(dg.DGError) as e:
            dg.sample_group(*args, edge_cap=cap)
        assert e.value.status == -2
    assert dg.sample_group(*args, edge_cap=2 * S).edge_ptr[:, -1].tolist() == [0, 2 * S]


def test_bad_seeds_among_many(dg):
    """2^23 seeds enter by a launch of their own: a seed out of range or repeated is reported."""
    n, S, B = EDGE + 5, EDGE, 4
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    idx = torch.zeros(0, dtype=torch.int32, device=DEV)
    good = torch.randperm(n, device=DEV)[:S].int().repeat(B, 1).contiguous()
    assert dg.sample_group(off, idx, good, [1], 5).hop_ptr[:, -1].tolist() == [S] * B
    for at, value, text in (((3, S - 1), n, "outside"), ((0, 7), -1, "outside"),
                            ((2, 9), int(good[2, 10]), "twice")):
        bad = good.clone()
        bad[at] = value
        with pytest.raises(dg.DGError, match=text):
            dg.sample_group(off, idx, bad, [1], 5)


@pytest.mark.big
def test_more_edges_and_pairs_than_threads_of_a_launch(dg):
    """4.22e9 edges of the first hop and 1.3e8 packed pairs: each part of the relabelling fits a
    launch of 2^32 threads, together they do not.  Every node is a seed of every mini-batch, in
    an order rotated by the batch, so that local indices are known."""
    n, D, B, step = 2_000_000, 33, 64, 30_011
    assert n * D * B < 2**32 < n * (D + 1) * B
    g = torch.Generator(device=DEV).manual_seed(1)
    off = torch.arange(0, n * D + 1, D, dtype=torch.int64, device=DEV)
    idx = torch.randint(0, n, (n, D), device=DEV, generator=g).int()
    order = torch.arange(n, device=DEV)
    seeds = torch.stack([(order + b * step) % n for b in range(B)]).int()
    feats = torch.randint(0, 256, (n, 1), dtype=torch.uint8, device=DEV, generator=g)
    slot = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    sr, pr = dg.sample_pack_group(off, idx.view(-1), seeds, [-1, 1], 5, feats, slot, layered=True)
    assert sr.node_count.tolist() == [n] * B
    assert sr.edge_ptr.tolist() == [[0, n * D, n * D + n]] * B
    for b in range(B):
        want = (idx.roll(-(b * step % n), 0) - b * step) % n
        assert torch.equal(sr.edge_dst[b, :n * D].view(n, D), want), b
        last = sr.edge_dst[b, n * D:n * D + n].view(n, 1)
        assert bool((want == last).any(1).all()), b
        assert torch.equal(pr.loc[b, :n], seeds[b]), b  # P_b is every node in order
