"""The forward's moments of the first interval (systems of more than 6,144
atoms, or 1,024 above 128 channels; type blocks of 128 slots and more) against
the oracle: lists whose tail, or a random part, lies in the first interval or
below the table, whole chunk sets of such records, blocks too short to be
looked at, NaN and infinite rows, an invalid atom at every place of a wavefront, lists
of more than one window."""
import numpy as np
import pytest

from parity import TOL, normwise, oracle_fwd_bwd
from synth.edge import edge_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE, BAD, NAN = 43, 7, 19


def _inputs(sel, m1, m2, seed, order):
    x = edge_inputs(BASE, sel, m1, m2, seed=seed)
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sel)])
    lo, d1 = x.lo[0], x.cfg.d1
    for i in range(BASE):
        for b in range(len(sel)):
            k = int(rng.integers(0, sel[b] + 1))             # valid slots of the block
            near = int(rng.integers(0, k + 1))               # of these, in the first interval
            first = np.zeros(k, bool)
            first[k - near:] = True
            first = first if order == "sorted" else rng.permutation(first)
            slots = off[b] + (np.arange(k) if order == "sorted" else np.sort(rng.choice(sel[b], k, replace=False)))
            x.nlist[i, off[b]:off[b + 1]] = -1
            x.nlist[i, slots] = 0
            v = np.where(first, lo + d1 * rng.uniform(-0.3, 1.0, k), lo + d1 * rng.uniform(1.0, 280.0, k))
            v[first & (rng.random(k) < 0.05)] = lo           # exactly on the lower end
            if order == "sorted":
                v[~first] = np.sort(v[~first])[::-1]
            x.em[i, slots, 0] = v
            x.em[i, slots, 1:] = rng.normal(size=(k, 3))
    x.em[x.nlist < 0] = 0
    return x


@pytest.mark.parametrize("order", ["sorted", "shuffled"])
@pytest.mark.parametrize("sel,m1,m2,dtype,n", [((200,), 100, 16, "f64", 6149), ((150, 40, 130), 100, 16, "f64", 6170),
                                               ((128, 127), 64, 15, "f64", 6149), ((300,), 200, 16, "f64", 1033),
                                               ((200, 140), 100, 16, "f32", 6149), ((512,), 128, 16, "f32acc64", 6149),
                                               ((200,), 200, 16, "f32acc64", 2057), ((600,), 17, 4, "f64", 6149)])
def test_matches_the_oracle(sel, m1, m2, dtype, n, order):
    import paper_2107_02103_amd as P
    x = _inputs(sel, m1, m2, sum(sel) + m1, order)
    row = np.flatnonzero(x.nlist[NAN] >= 0)
    x.em[NAN, row[-1], 2] = np.nan                       # a first-interval record, if there is one
    good = np.array([i for i in range(BASE) if i not in (BAD, NAN)])
    ref = oracle_fwd_bwd(x, good, dtype)
    nan_ref = oracle_fwd_bwd(x, np.array([NAN]), dtype)
    x.atype[BAD] = -1
    c = x.cfg
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[dtype]
    op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=mode)
    base = [torch.from_numpy(v).cuda() for v in (x.em, x.nlist, x.atype, x.dT)]
    for k in (0, 3):
        base[k] = base[k].to(op.t_in)
    em, nl, at, dT = (t.repeat((n // BASE + 1,) + (1,) * (t.dim() - 1))[:n].contiguous() for t in base)
    out = (*op.forward(em, nl, at), op.backward(em, nl, at, dT))
    out = [t.cpu().numpy().astype(np.float64) for t in out]
    rows = np.arange(n) % BASE
    ok = np.isin(rows, good)
    pick = np.searchsorted(good, rows[ok])
    err = [normwise(g[ok], r[pick]) for g, r in zip(out, ref)]
    print(f"[gpu-first] sel {sel} m1 {m1} {dtype} {order}: {err}", flush=True)
    assert max(err) <= TOL[dtype], err
    assert all(np.isnan(g[rows == BAD]).all() for g in out)
    for g, r in zip(out, nan_ref):                       # NaN where the oracle has it
        np.testing.assert_array_equal(np.isfinite(g[rows == NAN]), np.isfinite(np.repeat(r, (rows == NAN).sum(), 0)))


QUADS = 20         # rows of five wavefronts: an invalid atom at each of the four places, and none


def _quadruples(sel, m1, m2, seed):
    """Sorted full lists whose last chunk sets hold first-interval records only, so that every wavefront takes
    moments; row 5 p (place p of wavefront p) is to become invalid, p = 0..3."""
    x = edge_inputs(QUADS, sel, m1, m2, seed=seed)
    rng = np.random.default_rng(seed)
    lo, d1, nnei = x.lo[0], x.cfg.d1, sel[0]
    near = rng.integers(40, 60, size=QUADS)
    x.nlist[:] = 0
    for i in range(QUADS):
        v = np.concatenate([np.sort(rng.uniform(1.0, 280.0, nnei - near[i]))[::-1], rng.uniform(-0.3, 1.0, near[i])])
        x.em[i, :, 0] = lo + d1 * v
        x.em[i, :, 1:] = rng.normal(size=(nnei, 3))
    bad = np.array([5 * p for p in range(4)])
    x.nlist[bad, nnei // 2:] = -1                        # it decides nothing about the chunk sets looked at
    x.em[x.nlist < 0] = 0
    # every wavefront's last chunk set (16 slots an atom) holds at least 12 first-interval records of valid atoms
    last = (nnei - 1) // 16 * 16
    first = (x.nlist >= 0) & (x.em[..., 0] < lo + d1)
    first[bad] = False
    assert (first[:, last:].reshape(QUADS // 4, -1).sum(1) >= 12).all()
    return x, bad


@pytest.mark.parametrize("sel,m1,m2,dtype,n", [((200,), 100, 16, "f64", 6160), ((200,), 60, 8, "f64", 6150),
                                               ((200,), 200, 16, "f64", 1040), ((160,), 100, 16, "f32", 6160),
                                               ((500,), 128, 16, "f32acc64", 6160),
                                               ((200,), 200, 16, "f32acc64", 2080)])
def test_invalid_atom_at_every_place_of_a_wavefront(sel, m1, m2, dtype, n):
    import paper_2107_02103_amd as P
    x, bad = _quadruples(sel, m1, m2, m1 + sel[0])
    good = np.setdiff1d(np.arange(QUADS), bad)
    ref = oracle_fwd_bwd(x, good, dtype)[:2]
    x.atype[bad] = (-1, 1, -7, 100)
    c = x.cfg
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[dtype]
    op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=mode)
    em, nl, at = (torch.from_numpy(v).cuda().repeat((n // QUADS + 1,) + (1,) * (v.ndim - 1))[:n].contiguous()
                  for v in (x.em, x.nlist, x.atype))
    out = [t.cpu().numpy().astype(np.float64) for t in op.forward(em.to(op.t_in), nl, at)]
    rows = np.arange(n) % QUADS
    ok = np.isin(rows, good)
    err = [normwise(g[ok], r[np.searchsorted(good, rows[ok])]) for g, r in zip(out, ref)]
    print(f"[gpu-first] invalid atoms, sel {sel} m1 {m1} {dtype}: {err}", flush=True)
    assert max(err) <= TOL[dtype], err
    assert all(np.isnan(g[~ok]).all() for g in out)


@pytest.mark.parametrize("m1,dtype,n", [(100, "f64", 6160), (200, "f64", 1040), (100, "f32", 6160),
                                        (100, "f32acc64", 6160)])
def test_infinite_components_stay_infinite(m1, dtype, n):
    import paper_2107_02103_amd as P
    x, _ = _quadruples((200,), m1, 16, 3 * m1)
    rows = np.array([1, 4, 6, 9])                        # full lists; their last slots: first-interval records
    x.em[rows[0], 199, 1] = np.inf
    x.em[rows[1], 198, 2] = -np.inf
    x.em[rows[2], [197, 199], 3] = np.inf, np.inf
    x.em[rows[3], 190, 1:] = np.inf
    with np.errstate(all="ignore"):
        ref = oracle_fwd_bwd(x, rows, dtype)[:2]
    assert np.isinf(ref[0]).any() and np.isinf(ref[1]).any()
    c = x.cfg
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[dtype]
    op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=mode)
    em, nl, at = (torch.from_numpy(v).cuda().repeat((n // QUADS + 1,) + (1,) * (v.ndim - 1))[:n].contiguous()
                  for v in (x.em, x.nlist, x.atype))
    out = [t.cpu().numpy().astype(np.float64) for t in op.forward(em.to(op.t_in), nl, at)]
    for g, r in zip(out, ref):
        for k, row in enumerate(rows):
            got = g[np.arange(n) % QUADS == row]
            for what in (np.isposinf, np.isneginf, np.isnan):
                np.testing.assert_array_equal(what(got), np.broadcast_to(what(r[k]), got.shape))
