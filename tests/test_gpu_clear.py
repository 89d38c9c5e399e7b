"""Loops over groups with the mask-clearing flags: sampling with
DG_SAMPLE_EXIT_CLEAR (and DG_SAMPLE_ENTRY_CLEAR from the second group on),
packing with DG_PACK_CLEAR_MEMBERSHIP and the member-lines map sampling
writes, on one workspace per call and one membership buffer.  Every output must equal that of independent calls without
the flags, the membership output must equal theirs, and packing must leave the
mask all-zero.  The workspaces and the mask start filled with garbage, which
the first call (without DG_SAMPLE_ENTRY_CLEAR) must not see."""
import random
import re

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def dg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_05231_amd as m
    return m


def same_sample(a, b):
    assert np.array_equal(a.hop_ptr, b.hop_ptr) and np.array_equal(a.edge_ptr, b.edge_ptr)
    for bb in range(a.hop_ptr.shape[0]):
        n, e = int(a.hop_ptr[bb, -1]), int(a.edge_ptr[bb, -1])
        assert torch.equal(a.nodes[bb, :n], b.nodes[bb, :n]), bb
        assert torch.equal(a.edge_src[bb, :e], b.edge_src[bb, :e]), bb
        assert torch.equal(a.edge_dst[bb, :e], b.edge_dst[bb, :e]), bb


def same_pack(a, b, counts, keys=None):
    """keys: the size fields to compare (default all of them)."""
    if keys is None:
        assert a.sizes == b.sizes
    else:
        assert {k: a.sizes[k] for k in keys} == {k: b.sizes[k] for k in keys}
    rows = a.sizes["packed_rows"]
    assert np.array_equal(a.packed_ptr_host, b.packed_ptr_host)
    assert torch.equal(a.packed_ids[:rows], b.packed_ids[:rows])
    assert torch.equal(a.packed[:rows], b.packed[:rows])
    nu = a.sizes["unique_nodes"]
    assert torch.equal(a.unique[:nu], b.unique[:nu])
    for bb, n in enumerate(counts):
        assert torch.equal(a.loc[bb, :int(n)], b.loc[bb, :int(n)]), bb


def sparse_graph(fan=(3, 3, 2)):
    """200k nodes, degrees 0..6, 4 batches of 16 seeds: every hop is small
    enough to use touched marks, except that the last one reads every word when
    the call asks for the member-lines map or a clear exit.  With a last
    fan-out of 0 the last hop runs no count pass, and the sampler writes the map
    with a pass of its own and clears its state with a fill."""
    n = 200_000
    off, idx = synth.uniform_graph(n, 0, 6, seed=31)
    rnd = random.Random(99)
    gen = torch.Generator().manual_seed(3)
    feats = torch.randn((n, 4), generator=gen).to(DEV)
    slot = torch.full((n,), -1, dtype=torch.int32)
    slot[torch.tensor(rnd.sample(range(n), n // 10))] = torch.arange(n // 10, dtype=torch.int32)
    seeds = [torch.tensor([rnd.sample(range(n), 16) for _ in range(4)], dtype=torch.int32,
                          device=DEV) for _ in range(3)]
    return (torch.from_numpy(off).to(DEV), torch.from_numpy(idx).to(DEV), feats, slot.to(DEV),
            seeds, list(fan), 1234)


def workload_groups(name):
    w = synth.make_workload(name, device=DEV)
    cfg = w.cfg
    seeds = [synth.seed_batches(cfg.n, cfg.B, cfg.S, cfg.seed + 1 + g, DEV, offsets=w.offsets)
             for g in range(3)]
    return w.offsets, w.indices, w.feats, w.cache_slot, seeds, list(cfg.fanouts), w.rng_seed


def case_inputs(case):
    if case == "sparse":
        return sparse_graph()
    if case == "sparse_f0":
        return sparse_graph((3, 3, 0))
    return workload_groups(case)


@pytest.mark.parametrize("case,layered,direct", [("M1", False, True), ("M1", False, False),
                                                 ("M1", True, True), ("sparse", False, True),
                                                 ("sparse_f0", False, True)])
def test_group_loop_with_clear_flags(dg, case, layered, direct):
    off, idx, feats, slot, groups, fan, rng = case_inputs(case)
    N = off.numel() - 1
    B, S = groups[0].shape
    node_cap, edge_cap = dg.sample_bounds(N, idx.numel(), S, fan, layered)
    flags = dg.sample_flags(layered, direct)
    ws_s = torch.full((dg._L.dg_sample_workspace_bytes(N, B, node_cap, edge_cap, flags),), 0xA5,
                      dtype=torch.uint8, device=DEV)
    mem = torch.full((N,), -1, dtype=torch.int64, device=DEV)
    lines = torch.full((dg.member_lines_bytes(N),), 0xAB, dtype=torch.uint8, device=DEV)
    ws_p = None
    for g, seeds in enumerate(groups):
        print(f"[{case} layered={layered} direct={direct}] group {g}", flush=True)
        sr = dg.sample_group(off, idx, seeds, fan, rng, batch_base=g * B, membership=mem,
                             workspace=ws_s, layered=layered, direct=direct, exit_clear=True,
                             entry_clear=g > 0, member_lines=lines)
        mem_f = torch.empty(N, dtype=torch.int64, device=DEV)
        sr_f = dg.sample_group(off, idx, seeds, fan, rng, batch_base=g * B, membership=mem_f,
                               layered=layered, direct=direct)
        same_sample(sr, sr_f)
        assert torch.equal(mem, mem_f)
        counts = sr.hop_ptr[:, -1].copy()
        if ws_p is None:
            ws_p = torch.full((dg._L.dg_pack_workspace_bytes(N, B, int(counts.sum())) * 2,), 0x5A,
                              dtype=torch.uint8, device=DEV)
        pr = dg.pack_group(feats, slot, sr.nodes, counts, with_unique=True, membership=mem,
                           workspace=ws_p, clear_membership=True, member_lines=lines)
        torch.cuda.synchronize()
        assert int(mem.count_nonzero()) == 0
        pr_f = dg.pack_group(feats, slot, sr_f.nodes, counts, with_unique=True, membership=mem_f)
        same_pack(pr, pr_f, counts)


def lines_ref(dg, mem):
    """The member-lines map computed from the membership words by torch."""
    N = mem.numel()
    nbytes = dg.member_lines_bytes(N)
    pad = torch.zeros(nbytes * 8, dtype=torch.int64, device=DEV)
    pad[:N] = mem
    return (pad.view(-1, 8) != 0).any(dim=1)


@pytest.mark.parametrize("case,layered,direct", [("M1", False, True), ("M1", True, False),
                                                 ("sparse", False, True),
                                                 ("sparse_f0", False, True)])
def test_member_lines(dg, case, layered, direct):
    """The map sampling writes (by its last count pass, or by a pass of its own
    when the last hop runs none) marks exactly the 8-node lines that hold a
    member; packing with it gives the outputs of packing without it, and a map
    that misses a member line is reported."""
    off, idx, feats, slot, groups, fan, rng = case_inputs(case)
    N = off.numel() - 1
    seeds = groups[0]
    B = seeds.shape[0]
    mem = torch.empty(N, dtype=torch.int64, device=DEV)
    lines = torch.full((dg.member_lines_bytes(N),), 0xAB, dtype=torch.uint8, device=DEV)
    sr = dg.sample_group(off, idx, seeds, fan, rng, membership=mem, member_lines=lines,
                         layered=layered, direct=direct)
    torch.cuda.synchronize()
    assert torch.equal(lines != 0, lines_ref(dg, mem))
    counts = sr.node_count
    ref = dg.pack_group(feats, slot, sr.nodes, counts, with_unique=True, membership=mem)
    mem2 = mem.clone()
    got = dg.pack_group(feats, slot, sr.nodes, counts, with_unique=True, membership=mem2,
                        member_lines=lines, clear_membership=True)
    torch.cuda.synchronize()
    assert int(mem2.count_nonzero()) == 0
    same_pack(got, ref, counts)
    # a map that misses a line holding a member
    bad = lines.clone()
    bad[int((lines != 0).nonzero()[0])] = 0
    with pytest.raises(dg.DGError) as e:
        dg.pack_group(feats, slot, sr.nodes, counts, membership=mem, member_lines=bad)
    assert e.value.status == -1


# (B, S, fan-outs, direct, layered, node_cap's margin, workspaces of the least size, one call)
MIXED = [(4, 16, (3, 3, 2), True, False, 0, False, True),
         (1, 300, (2, 2), False, False, 7, False, True),
         (64, 16, (3, 3), True, False, 0, True, True),
         (3, 64, (6, 6, 6, 6), False, True, 100, True, False),
         (64, 700, (5, 5), True, False, 1, False, False),
         (2, 16, (-1, 2), True, True, 0, True, True),
         (5, 33, (0, 3), True, True, 3, False, True),
         (4, 16, (3, 0), True, False, 0, True, False),
         (4, 16, (3, 3, 2), True, False, 0, False, True)]


@pytest.mark.parametrize("n", [70_000, 200_000, 700_000])
def test_one_workspace_for_calls_of_every_shape(dg, n):
    """DG_SAMPLE_ENTRY_CLEAR asks for the same number of nodes and nothing else: B, S, the
    fan-outs, the capacities, the relabelling mode, layering, the tile length (a workspace of the
    least size takes the longest tiles) and the form of the call change from call to call on one
    workspace and one membership mask."""
    rnd = random.Random(n)
    g = torch.Generator(device=DEV).manual_seed(n)
    deg = torch.randint(0, 7, (n,), device=DEV, generator=g)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=off[1:])
    idx = torch.randint(0, n, (int(off[-1]),), device=DEV, generator=g).int()
    feats = torch.randint(0, 256, (n, 16), dtype=torch.uint8, device=DEV, generator=g)
    slot = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    slot[::9] = torch.arange(slot[::9].numel(), dtype=torch.int32, device=DEV)
    caps, most = [], [0, 0]
    for B, S, fan, direct, layered, margin, _, _ in MIXED:
        nc, ec = dg.sample_bounds(n, idx.numel(), S, fan, layered)
        nc = min(nc + margin, n) if margin else nc
        caps.append((nc, ec))
        need = (dg._L.dg_sample_workspace_bytes(n, B, nc, ec, dg.sample_flags(layered, direct)),
                max(dg._L.dg_sample_pack_workspace_bytes(n, B, nc),
                    dg._L.dg_pack_workspace_bytes(n, B, B * nc)))
        most = [max(a, b) for a, b in zip(most, need)]
    ws, pws = (torch.full((m,), 0xA5, dtype=torch.uint8, device=DEV) for m in most)
    mem = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    for turn, ((B, S, fan, direct, layered, _, least, one), (nc, ec)) in \
            enumerate(zip(MIXED + MIXED[::-1], caps + caps[::-1])):
        print(f"[n={n}] call {turn}", flush=True)
        seeds = torch.stack([torch.randperm(n, device=DEV, generator=g)[:S]
                             for _ in range(B)]).int()
        kw = dict(node_cap=nc, edge_cap=ec, layered=layered, direct=direct)
        flags = dict(membership=mem, entry_clear=turn > 0, exit_clear=True)
        rng = rnd.randrange(2**40)
        fresh = dg.sample_group(off, idx, seeds, fan, rng, **kw)
        counts = fresh.node_count
        fresh_p = dg.pack_group(feats, slot, fresh.nodes, counts, with_unique=True)
        sizes = [ws.numel(), pws.numel()]

        def call():
            at = iter([ws[:sizes[0]], pws[:sizes[1]]])
            with pytest.MonkeyPatch.context() as patch:
                patch.setattr(dg, "_workspace", lambda nbytes, d, w: next(at))
                if one:
                    out = dg.PackResult(
                        packed=torch.empty_like(fresh_p.packed),
                        packed_ids=torch.empty_like(fresh_p.packed_ids),
                        packed_ptr=torch.empty_like(fresh_p.packed_ptr),
                        packed_ptr_host=np.zeros(B + 1, dtype=np.int64),
                        loc=torch.empty((B, nc), dtype=torch.int32, device=DEV),
                        unique=torch.empty_like(fresh_p.unique), sizes={}, timing=None,
                        row_bytes=16)
                    return dg.sample_pack_group(off, idx, seeds, fan, rng, feats, slot,
                                                pack_out=out, **kw, **flags)
                sr = dg.sample_group(off, idx, seeds, fan, rng, **kw, **flags)
                return sr, dg.pack_group(feats, slot, sr.nodes, sr.node_count, with_unique=True,
                                         membership=mem, clear_membership=True)

        if least:  # refused calls touch nothing and name what they need
            for k in (1, 0):
                keep, sizes[k] = sizes[k], 256
                if one or k == 0:
                    with pytest.raises(dg.DGError, match="workspace needs") as e:
                        call()
                    sizes[k] = int(re.search(r"needs (\d+) bytes", str(e.value))[1])
                else:
                    sizes[k] = keep
        sr, pr = call()
        same_sample(sr, fresh)
        rows = fresh_p.sizes["packed_rows"]
        assert pr.sizes["packed_rows"] == rows
        assert torch.equal(pr.packed[:rows], fresh_p.packed[:rows])
        assert torch.equal(pr.unique[:fresh_p.sizes["unique_nodes"]],
                           fresh_p.unique[:fresh_p.sizes["unique_nodes"]])
        for b in range(B):
            assert torch.equal(pr.loc[b, :int(counts[b])], fresh_p.loc[b, :int(counts[b])]), b
        assert int(mem.count_nonzero()) == 0
