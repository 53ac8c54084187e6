"""The ways a system's size maps atoms to wavefronts (one atom's runs shared
out, a few atoms' chunk sets shared out, no sharing) against the oracle, on
both sides of every size at which the mapping changes.  A small edge system
(ragged blocks, all parts of the range, an empty atom, an invalid type) is
repeated up to the wanted number of atoms, so that the oracle runs once."""
import numpy as np
import pytest

from parity import TOL, normwise, oracle_fwd_bwd
from synth.edge import edge_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE = 43          # atoms repeated: odd, so that copies start anywhere in a workgroup
BAD, EMPTY = 7, 11


@pytest.mark.parametrize("sel,m1,m2,dtype", [((40, 33), 100, 16, "f64"), ((700,), 17, 4, "f64"),
                                             ((30, 20, 14), 128, 15, "f64"), ((50,), 129, 8, "f64"),
                                             ((3, 70), 100, 16, "f32"), ((64,), 100, 16, "f32acc64"),
                                             ((40, 33), 200, 16, "f32acc64"),
                                             ((40, 33), 200, 16, "f64"), ((70,), 256, 16, "f64"),
                                             ((20, 30), 137, 8, "f32acc64"), ((40,), 241, 5, "f32"),
                                             ((20, 31), 161, 8, "f32acc64"), ((30, 241), 208, 8, "f32acc64"),
                                             ((30, 241), 209, 8, "f32acc64"), ((70,), 256, 16, "f32acc64")])
def test_every_mapping_matches_the_oracle(sel, m1, m2, dtype):
    import paper_2107_02103_amd as P
    x = edge_inputs(BASE, sel, m1, m2, seed=sum(sel) + m1 + 29)
    x.nlist[EMPTY] = -1
    x.em[EMPTY] = 0
    good = np.array([i for i in range(BASE) if i != BAD])
    ref = oracle_fwd_bwd(x, good, dtype)
    x.atype[BAD] = -1
    c = x.cfg
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[dtype]
    op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=mode)
    base = [torch.from_numpy(v).cuda() for v in (x.em, x.nlist, x.atype, x.dT)]
    for k in (0, 3):
        base[k] = base[k].to(op.t_in)
    for n in (1, 512, 513, 640, 641, 1024, 1025, 1280, 1281, 1536, 1537, 2048, 2049, 3072, 3073, 6144, 6145, 6161,
              8192, 8193, 10240, 10241):
        em, nl, at, dT = (t.repeat((n // BASE + 1,) + (1,) * (t.dim() - 1))[:n].contiguous() for t in base)
        out = (*op.forward(em, nl, at), op.backward(em, nl, at, dT))
        out = [t.cpu().numpy().astype(np.float64) for t in out]
        rows = np.arange(n)
        ok = rows[rows % BASE != BAD]
        pick = np.searchsorted(good, ok % BASE)
        err = [normwise(g[ok], r[pick]) for g, r in zip(out, ref)]
        print(f"[gpu-split] sel {sel} m1 {m1} {dtype} n {n}: {err}", flush=True)
        assert max(err) <= TOL[dtype], (n, err)
        assert all(np.isnan(g[rows % BASE == BAD]).all() for g in out)
        assert np.all(out[2][ok][x.nlist[ok % BASE] < 0] == 0)


def test_from_dD_in_every_mapping():
    import paper_2107_02103_amd as P
    from oracle import cref
    from oracle.se_a import descriptor_backward
    from oracle.table import build_tables
    for sel, m1, m2 in (((40, 33), 100, 16), ((70,), 17, 2), ((50,), 113, 10)):
        x = edge_inputs(BASE, sel, m1, m2, seed=m1)
        rng = np.random.default_rng(m1)
        T, dD = rng.normal(size=(BASE, m1, 4)), rng.normal(size=(BASE, m1, m2))
        ref = cref.Problem(x.em, x.nlist, x.atype, build_tables(x), x.cfg.sel, m2).backward(descriptor_backward(T, dD))
        c = x.cfg
        op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2)
        base = [torch.from_numpy(v).cuda() for v in (x.em, x.nlist, x.atype, T, dD)]
        for n in (2, 1280, 1281, 6144, 6145):
            args = [t.repeat((n // BASE + 1,) + (1,) * (t.dim() - 1))[:n].contiguous() for t in base]
            got = op.backward_from_dD(*args).cpu().numpy()
            err = normwise(got, ref[np.arange(n) % BASE])
            print(f"[gpu-split] from dD, m1 {m1} n {n}: {err:.2e}", flush=True)
            assert err <= TOL["f64"], (m1, n, err)


@pytest.mark.parametrize("sel,m1,dtype", [((63,), 100, "f64"), ((64,), 60, "f64"), ((200, 55), 100, "f64"),
                                          ((256,), 100, "f64"), ((63,), 100, "f32"), ((64,), 100, "f32"),
                                          ((40,), 200, "f64"), ((40,), 200, "f32acc64"), ((40,), 256, "f32acc64"),
                                          ((90,), 256, "f32acc64"), ((40, 20), 60, "f32acc64"), ((90,), 200, "f32")])
def test_sharing_by_the_length_of_the_list(sel, m1, dtype):
    # both sides of the atom counts at which short, middle and long lists change how atoms are shared
    import paper_2107_02103_amd as P
    x = edge_inputs(BASE, sel, m1, 8, seed=sum(sel) + m1)
    good = np.array([i for i in range(BASE) if i != BAD])
    ref = oracle_fwd_bwd(x, good, dtype)
    x.atype[BAD] = -1
    c = x.cfg
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[dtype]
    op = P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=mode)
    base = [torch.from_numpy(v).cuda() for v in (x.em, x.nlist, x.atype, x.dT)]
    for k in (0, 3):
        base[k] = base[k].to(op.t_in)
    for n in (1024, 1025, 1536, 1537, 2048, 2049, 3072, 3073, 4096, 4097, 6144, 6145, 8192, 8193):
        em, nl, at, dT = (t.repeat((n // BASE + 1,) + (1,) * (t.dim() - 1))[:n].contiguous() for t in base)
        out = (*op.forward(em, nl, at), op.backward(em, nl, at, dT))
        out = [t.cpu().numpy().astype(np.float64) for t in out]
        rows = np.arange(n) % BASE
        err = [normwise(g[rows != BAD], r[np.searchsorted(good, rows[rows != BAD])]) for g, r in zip(out, ref)]
        assert max(err) <= TOL[dtype], (n, err)
        assert all(np.isnan(g[rows == BAD]).all() for g in out)
