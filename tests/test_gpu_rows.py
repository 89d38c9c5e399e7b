"""Row movement at every launch shape, odd size and alignment: the assembly, the row gather and
the packing gather against a library gather (bytes, tolerance 0), with guard bytes around every
output."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 64


@pytest.fixture(scope="module")
def dg():
    import paper_2405_05231_amd as m
    return m


def at(t, shift):
    """A copy of the byte tensor t whose address is `shift` past an aligned one."""
    buf = torch.empty(t.numel() + 256, dtype=torch.uint8, device=DEV)
    view = buf[shift:shift + t.numel()].view(t.shape)
    view.copy_(t)
    return view


class Guarded:
    """An output of `shape` bytes, `shift` past an aligned address, between guard bytes."""

    def __init__(self, n, R, shift):
        self.buf = torch.full((n * R + 2 * GUARD + shift,), 171, dtype=torch.uint8, device=DEV)
        self.lo, self.hi = GUARD + shift, GUARD + shift + n * R
        self.rows = self.buf[self.lo:self.hi].view(n, R)

    def check(self):
        assert bool((self.buf[:self.lo] == 171).all()) and bool((self.buf[self.hi:] == 171).all())


# the edges of every launch shape, the shortest and longest rows of the vector path and beyond
SIZES = [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 96, 100, 127, 128, 129, 200, 255, 256, 257,
         385, 511, 512, 513, 1023, 1024, 1025, 1540, 2047, 2049, 2408, 3071, 3073, 4095, 4096,
         4097]
# both sides of the lines between the kinds of stores
SIZES += [192, 576, 608, 624, 640, 899, 900, 1584, 1600, 2064, 2396, 2400]


@pytest.mark.parametrize("R", SIZES)
@pytest.mark.parametrize("shift", [0, 1, 4])
def test_rows_every_size_and_alignment(dg, R, shift):
    g = torch.Generator(device=DEV).manual_seed(R * 8 + shift)
    N = 301
    X = at(torch.randint(0, 256, (N, R), dtype=torch.uint8, device=DEV, generator=g), shift)
    for n in (1, 6, 517):
        ids = torch.randint(0, N, (n,), device=DEV, generator=g).int()
        out = Guarded(n, R, shift)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        dg.gather_rows(X, ids, out=out.rows, status=status)
        assert torch.equal(out.rows, X[ids.long()]) and int(status) == 0
        out.check()

        # assembly: rows below 100 are the cache table, the others the packed chunk; one
        # entry outside both where there is room for it
        loc = torch.where(ids < 100, -ids - 1, ids - 100)
        want = X[ids.long()].clone()
        if n > 1:
            loc[n // 2] = N
            want[n // 2] = 0
        out = Guarded(n, R, shift)
        dg.assemble_batch(X[:100], X[100:], loc, R, out=out.rows, status=status)
        assert torch.equal(out.rows, want) and int(status) == int(n > 1)
        out.check()

    # two batches in one launch, and the packing gather behind them
    nodes = torch.stack([torch.randperm(N, device=DEV, generator=g)[:211] for _ in range(2)]).int()
    slot = torch.full((N,), -1, dtype=torch.int32, device=DEV)
    slot[:100] = torch.arange(100, dtype=torch.int32, device=DEV)
    ref = dg.pack_group(X, slot, nodes, [211, 211])
    rows = ref.sizes["packed_rows"]
    packed = Guarded(rows, R, shift)
    table = Guarded(100, R, shift)
    pr = dg.PackResult(packed=packed.rows, packed_ids=ref.packed_ids[:rows].clone(),
                       packed_ptr=ref.packed_ptr, packed_ptr_host=ref.packed_ptr_host,
                       loc=ref.loc, unique=None, sizes={}, timing=None, row_bytes=R)
    dg.pack_group(X, slot, nodes, [211, 211], out=pr,
                  cache_nodes=torch.arange(100, dtype=torch.int32, device=DEV),
                  cache_table=table.rows)
    assert torch.equal(packed.rows, X[pr.packed_ids.long()])
    assert torch.equal(table.rows, X[:100])
    packed.check()
    table.check()
    outs = [Guarded(211, R, shift) for _ in range(2)]
    dg.assemble_batches(X[:100], pr, [211, 211], [o.rows for o in outs])
    for b, o in enumerate(outs):
        assert torch.equal(o.rows, X[nodes[b].long()])
        o.check()


@pytest.mark.parametrize("R", [192, 608, 901, 1616, 2404])
@pytest.mark.parametrize("large", [False, True])
def test_rows_on_both_sides_of_the_large_outputs(dg, R, large):
    """Outputs just below and above 320 MB, where the kind of stores changes: the row gather, and
    packing of two lists whose rows go to two chunks each."""
    N, n = 40_000, 320_000_000 // R + (1 if large else 0)
    g = torch.Generator(device=DEV).manual_seed(R)
    X = torch.randint(0, 256, (N, R), dtype=torch.uint8, device=DEV, generator=g)
    ids = torch.randint(0, N, (n,), device=DEV, generator=g).int()
    out = Guarded(n, R, 3)
    dg.gather_rows(X, ids, out=out.rows)
    want = X[ids.long()]
    assert torch.equal(out.rows, want)
    out.check()
    del want
    B = n // N + 1  # every node in each batch, and the rest in the last
    counts = [N] * (B - 1) + [n - N * (B - 1)]
    slot = torch.full((N,), -1, dtype=torch.int32, device=DEV)
    nodes = torch.stack([torch.randperm(N, device=DEV, generator=g) for _ in range(B)]).int()
    packed = Guarded(n, R, 5)
    pr = dg.pack_group(X, slot, nodes, counts, tables_only=True)
    pr.packed, pr.packed_ids = packed.rows, pr.packed_ids[:n].contiguous()
    pr = dg.pack_group(X, slot, nodes, counts, out=pr)
    assert pr.sizes["packed_rows"] == n
    assert torch.equal(packed.rows, X[pr.packed_ids.long()])
    packed.check()
