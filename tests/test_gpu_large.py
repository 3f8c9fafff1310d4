"""Counts of items above what one pass of a kernel's grid takes (2^20 workgroups):
rings of the per-ring passes, B polygons of the join, pairs of the relations,
sets of the sums.  Closed forms; inputs are made on the GPU."""

import time

import pytest

import paper_1208_0277_amd as sccg

pytestmark = pytest.mark.gpu


def _squares(n):
    """n rings, each the square [0, 3) x [0, 3)."""
    import torch
    one = torch.tensor([[0, 0], [3, 0], [3, 3], [0, 3]], dtype=torch.int32, device="cuda")
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * 4
    return sccg.DevicePolys(off, one.repeat(n, 1))


@pytest.fixture
def ctx():
    c = sccg.Context(0)
    yield c
    c.close()


def test_rings_validated(ctx):
    n = (1 << 24) + 37  # 16 rings a workgroup
    P = _squares(n)
    for bad in ([], [n - 1], [n - 1, (1 << 24) + 1], [n - 2, 16], [(1 << 24) - 1, 1 << 24]):
        for k in bad:
            P.xy[4 * k + 2] += 1
        out = ctx.validate_polys(P)
        ctx.sync()
        assert int(out.item()) == min(bad, default=-1)
        for k in bad:
            P.xy[4 * k + 2] -= 1


def test_polygons_joined(ctx):
    """Two A squares, one of them in every pair (16 B polygons a workgroup of
    the writing pass), some B polygons with no pair."""
    import torch
    n = (1 << 25) + 45
    A, B = _squares(2), _squares(n)
    A.xy[4:] += 100
    for k in (0, 1, n // 2, n - 2):
        B.xy[4 * k:4 * k + 4] += 10
    off = torch.tensor([0, 2], dtype=torch.int64, device="cuda")
    pa, pb, so = ctx.join_sets(A, B, off, torch.tensor([0, n], dtype=torch.int64, device="cuda"), cap=n)
    ctx.sync()
    want = torch.ones(n, dtype=torch.bool, device="cuda")
    want[[0, 1, n // 2, n - 2]] = False
    assert so.tolist() == [0, n - 4] and not pa.any()
    assert torch.equal(pb.long(), want.nonzero().squeeze(1))


def test_areas_and_pairs_related(ctx):
    import torch
    n = (1 << 24) + 21
    P = _squares(n)
    P.xy[-4 * 7:] *= 2  # the last seven have four times the area
    pa = torch.arange(n - 40, n, dtype=torch.int32, device="cuda")
    I = torch.full((40,), 9, dtype=torch.int64, device="cuda")
    got = ctx.relate_pairs(P, P, pa, pa.flip(0).contiguous(), I)
    ctx.sync()
    area = torch.tensor([9] * 33 + [36] * 7)
    inter, contains, within = area.flip(0) >= 9, area.flip(0) == 9, area == 9
    want = (inter * sccg.SCCG_REL_INTERSECTS + contains * sccg.SCCG_REL_CONTAINS + within * sccg.SCCG_REL_WITHIN
            + (contains & within) * sccg.SCCG_REL_EQUALS)
    assert torch.equal(got.cpu().long(), want.long())
    m = (1 << 28) + 300  # 256 pairs a workgroup
    i = torch.zeros(m, dtype=torch.int32, device="cuda")
    I = torch.zeros(m, dtype=torch.int64, device="cuda")
    I[::7] = 9
    got = ctx.relate_pairs(_squares(1), _squares(1), i, i, I)
    ctx.sync()
    both = sccg.SCCG_REL_INTERSECTS | sccg.SCCG_REL_CONTAINS | sccg.SCCG_REL_WITHIN | sccg.SCCG_REL_EQUALS
    assert bool((got[::7] == both).all())
    assert int((got == both).sum()) == (m + 6) // 7
    assert int((got == sccg.SCCG_REL_TOUCHES).sum()) == m - (m + 6) // 7


def test_sets_summed(ctx):
    """Sets of two pairs, some of three and none: four sets a workgroup of the
    pass that finishes sets of several waves and empty ones."""
    import torch
    n = (1 << 22) + 1003
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    size = torch.full((n,), 2, dtype=torch.int64, device="cuda")
    size[torch.randint(0, n, (n // 10,), generator=g, device="cuda")] = 0
    size[torch.randint(0, n, (n // 10,), generator=g, device="cuda")] = 3
    size[-5:] = 0
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), size.cumsum(0)])
    m = int(off[-1])
    U = torch.randint(1, 1000, (m,), generator=g, device="cuda")
    I = (U * torch.rand(m, generator=g, device="cuda")).long()
    si, su, nn, j, _ = ctx.jaccard_sets(off, I, U)
    ctx.sync()

    def sums(v):
        c = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), v.cumsum(0)])
        return c[off[1:]] - c[off[:-1]]

    on = (I > 0).long()
    assert torch.equal(si, sums(I)) and torch.equal(su, sums(U * on)) and torch.equal(nn, sums(on))
    assert torch.equal(j, torch.where(su > 0, si.double() / su.clamp_min(1).double(), torch.zeros_like(j)))


@pytest.mark.parametrize("sets,most_ms", [(2, 5), (3, 5), (40, 36)])
def test_cells_scanned(ctx, sets, most_ms):
    """Sets of 16 million cells of a pixel, 40,000 squares 20 px apart in each
    and their copies, each of which meets its own: the scan of 32 million counts
    and around, and of 640 million, in not much more than its bytes' time (26
    ms; 45 when every block sums the totals before its own)."""
    import torch
    k = torch.arange(sets * 40_000, device="cuda")
    x, y = 20 * (k % 200), 20 * ((k % 40_000) // 200)

    def squares(d):
        v = torch.stack([torch.stack([x + d + i * 12, y + d + j * 12], 1) for i, j in ((0, 0), (1, 0), (1, 1), (0, 1))], 1)
        off = torch.arange(k.shape[0] + 1, dtype=torch.int64, device="cuda") * 4
        return sccg.DevicePolys(off, v.reshape(-1, 2).to(torch.int32).contiguous())

    A, B = squares(0), squares(5)
    off = torch.arange(sets + 1, device="cuda") * 40_000
    best = 1e9
    for _ in range(4):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        pa, pb, so = ctx.join_sets(A, B, off, off, cell=1, cap=8 * k.shape[0])
        ctx.sync()
        best = min(best, (time.perf_counter() - t0) * 1e3)
        assert torch.equal(so, off) and torch.equal(pa, k.to(torch.int32)) and torch.equal(pb, k.to(torch.int32))
    print(f"{sets} sets: {best:.1f} ms", flush=True)
    assert best < most_ms


def test_polygons_counted(ctx):
    """The same with B polygons of more than one pass of the count, 64 a
    workgroup; a few have a pair."""
    import torch
    n = (1 << 26) + 77
    A, B = _squares(2), _squares(n)
    A.xy[4:] += 100
    B.xy += 10
    for k in (3, 1 << 25, (1 << 26) - 1, 1 << 26, (1 << 26) + 63, n - 1):
        B.xy[4 * k:4 * k + 4] -= 9
    off = torch.tensor([0, 2], dtype=torch.int64, device="cuda")
    pa, pb, so = ctx.join_sets(A, B, off, torch.tensor([0, n], dtype=torch.int64, device="cuda"), cap=100)
    ctx.sync()
    assert so.tolist() == [0, 6] and not pa.any()
    assert pb.tolist() == [3, 1 << 25, (1 << 26) - 1, 1 << 26, (1 << 26) + 63, n - 1]
