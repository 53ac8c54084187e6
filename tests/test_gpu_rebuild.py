"""Neighbour list and reverse slots where their kernels change path: periodic
images taken from the cells (three and more cells per edge, positions on cell
and box faces), ranks from buckets of r2 (perfect crystals: whole shells in
one bucket; up to 512 neighbours) or by comparison (more), and the reverse
search's look, second look and scan (short blocks, truncated and shuffled
lists, lists of more than one window).  Integers: exact."""
import numpy as np
import pytest

from oracle import nlist as onl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _build(coord, atype, sel, box, rc):
    import paper_2107_02103_amd as P
    n = len(coord)
    c, a = torch.from_numpy(coord).cuda(), torch.from_numpy(atype).cuda()
    nb = P.dpc_nlist_workspace_bytes(n, box, rc)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    nl = torch.full((n, sum(sel)), -7, dtype=torch.int32, device="cuda")
    P.dpc_nlist_build(torch.cuda.current_stream(), n, len(sel), sel, box, rc, c, a, ws, nb, nl, wait=False)
    return c, a, nl, tuple(ws[:8].view(torch.int32).cpu().tolist())


def _reverse(c, a, nl, sel, box):
    import paper_2107_02103_amd as P
    rev = torch.full(nl.shape, -7, dtype=torch.int32, device="cuda")
    P.dpc_nlist_reverse(torch.cuda.current_stream(), nl.shape[0], len(sel), sel, box, c, a, nl, rev)
    return rev.cpu().numpy()


def _reverse_expected(nl, atype, sel):
    off = np.concatenate([[0], np.cumsum(sel)])
    rev = np.full(nl.shape, -1, np.int32)
    for i in range(len(nl)):
        t = atype[i]
        for s in np.nonzero(nl[i] >= 0)[0]:
            if 0 <= t < len(sel):
                hit = np.nonzero(nl[nl[i, s], off[t]:off[t + 1]] == i)[0]
                rev[i, s] = off[t] + hit[0] if len(hit) else -1
    return rev


def _check(coord, atype, sel, box, rc):
    coord, atype = np.ascontiguousarray(coord), np.ascontiguousarray(atype, np.int32)
    c, a, nl, st = _build(coord, atype, sel, box, rc)
    ref, _, over = onl.neighbour_list(coord, atype, sel, box, rc)
    got = nl.cpu().numpy()
    assert st == (over, 0)
    np.testing.assert_array_equal(got, ref)
    np.testing.assert_array_equal(_reverse(c, a, nl, sel, box), _reverse_expected(got, atype, sel))
    return c, a, got


@pytest.mark.parametrize("cells", [3, 4, 5])
def test_positions_on_faces(cells):
    # all positions inside the box (the images come from the cells), many of
    # them on cell faces, on the box's lower faces or one unit below the upper
    rc, rng = 3.0, np.random.default_rng(cells)
    box = cells * rc * (1.0 + 1e-8)
    x = rng.uniform(0, box, size=(420, 3))
    grid = np.concatenate([np.arange(cells) * (box / cells), [np.nextafter(box, 0.0), np.nextafter(box / cells, 0.0)]])
    on = rng.random(x.shape) < 0.4
    x[on] = grid[rng.integers(0, len(grid), on.sum())]
    _check(x, rng.integers(-1, 2, size=len(x)), (70, 70), box, rc)
    # one atom outside: its batches take the rounded quotient
    x[17, 1] += box
    _check(x, rng.integers(0, 2, size=len(x)), (70, 70), box, rc)


@pytest.mark.parametrize("kind", ["sc", "fcc"])
def test_perfect_crystals(kind):
    # undisplaced lattices: shells of equal distances up to rounding, ordered
    # by the exact (r2, index)
    a, n = 2.0, 6
    g = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    b = np.zeros((1, 1, 3)) if kind == "sc" else np.array([[[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]]])
    x = ((g + b) * a).reshape(-1, 3)
    t = np.random.default_rng(2).integers(0, 3, size=len(x))
    for sel in ((200,), (90, 90, 90)):
        _check(x, t if len(sel) > 1 else 0 * t, sel, n * a, 3.999)


@pytest.mark.parametrize("near", [511, 512, 513, 700])
def test_many_neighbours(near):
    # atoms with `near` neighbours: the last lists ranked through buckets, the
    # first ones ranked by comparison; clustered, so that buckets fill unevenly
    rng = np.random.default_rng(near)
    x = np.concatenate([rng.normal(5.0, 0.3, size=(near + 1, 3)), rng.uniform(0, 40, size=(50, 3))])
    _check(x, rng.integers(0, 2, size=len(x)), (400, 500), 40.0, 9.0)


@pytest.mark.parametrize("sel", [(900,), (400, 500), (150, 150), (40, 30, 50, 20)])
@pytest.mark.parametrize("n,edge,cluster", [(1000, 2.01, 0), (3500, 3.02, 0), (1600, 2.2, 800)])
def test_lists_longer_than_512(n, edge, cluster, sel):
    # dense systems, ranked through buckets with up to 1,024 neighbours each; in one
    # a cluster's atoms have more, which the second counter says
    rc, rng = 3.0, np.random.default_rng(n + len(sel))
    x = rng.uniform(0, edge * rc, size=(n, 3))
    x[:cluster] = 0.5 * edge * rc + rng.normal(0, 0.3, size=(cluster, 3))
    t = np.ascontiguousarray(rng.integers(0, len(sel), size=n), np.int32)
    _, _, nl, st = _build(x, t, sel, edge * rc, rc)
    ref, _, over = onl.neighbour_list(x, t, sel, edge * rc, rc)
    d = x[:, None] - x[None]
    d -= edge * rc * np.rint(d / (edge * rc))
    count = ((d ** 2).sum(-1) < rc * rc).sum(1) - 1
    few = count <= 1024
    assert (count > 512).any() and st[1] == (~few).sum()
    assert cluster or st == (over, 0)
    np.testing.assert_array_equal(nl.cpu().numpy()[few], ref[few])


def test_long_lists_of_a_perfect_crystal():
    # whole shells in one bucket, more than 512 neighbours
    g = np.stack(np.meshgrid(*[np.arange(12.0)] * 3, indexing="ij"), -1).reshape(-1, 3)
    _check(g, np.zeros(len(g), int), (600,), 12.0, 5.001)
    _check(g, np.random.default_rng(1).integers(0, 2, size=len(g)), (300, 320), 12.0, 5.001)


@pytest.mark.parametrize("n,box", [(1, 7.0), (8191, 30.0), (8192, 90.0), (8193, 30.0), (700, 200.0)])
def test_cell_lists_of_one_workgroup_and_of_several(n, box):
    # both sides of the largest system whose cells one workgroup sorts, few and
    # many cells (4,096 are the most it takes; one cell per atom and axis at
    # most), crowded and empty ones
    rng = np.random.default_rng(n)
    x = rng.uniform(0, box, size=(n, 3))
    x[: n // 4] = rng.uniform(0, 2.0, size=(n // 4, 3)) + x[0]
    a = np.ascontiguousarray(rng.integers(0, 2, size=n), np.int32)
    c, at, nl, st = _build(x, a, (120, 120), box, 3.0)
    pick = np.unique(rng.integers(0, n, 400))
    ref, cnt, over = onl.neighbour_list(x, a, (120, 120), box, 3.0, centres=pick)
    few = np.asarray(cnt).sum(1) <= 1024 if np.ndim(cnt) == 2 else np.ones(len(pick), bool)
    np.testing.assert_array_equal(nl.cpu().numpy()[pick][few], ref[few])


@pytest.mark.parametrize("sel", [(3,), (16,), (17, 2), (9, 40), (2, 20, 30)])
def test_reverse_of_short_and_truncated_blocks(sel):
    rng = np.random.default_rng(sum(sel))
    x = rng.uniform(0, 9.5, size=(260, 3))
    _check(x, rng.integers(0, len(sel), size=260), sel, 9.5, 3.0)


def test_reverse_of_shuffled_lists_and_bad_entries():
    # shuffled slots over more than one window of 512, padding between them,
    # neighbours out of range and atoms of invalid type
    rng = np.random.default_rng(8)
    n, sel = 300, (400, 330)
    x = rng.uniform(0, 9.5, size=(n, 3))
    t = rng.integers(0, 2, size=n).astype(np.int32)
    c, a, got = _check(x, t, sel, 9.5, 4.0)
    off = np.concatenate([[0], np.cumsum(sel)])
    for i in range(n):
        for u in range(2):
            got[i, off[u]:off[u + 1]] = rng.permutation(got[i, off[u]:off[u + 1]])
    t[[4, 50]] = (-1, 2)
    ref = _reverse_expected(got, t, sel)
    bad = got.copy()
    pad = np.argwhere(bad < 0)
    for k in pad[rng.choice(len(pad), 40, replace=False)]:
        bad[tuple(k)] = n + 5
    out = _reverse(c, torch.from_numpy(t).cuda(), torch.from_numpy(bad).cuda(), sel, 9.5)
    np.testing.assert_array_equal(out, ref)
