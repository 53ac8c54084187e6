"""Timed cases: the calls a user of this library makes, over the sizes, types and options it is used at.

Three paths, all through the public entry points:

* "step"     one forward (T, D) and one backward (dE/dR~) pass of the compressed descriptor, inputs resident on
             the GPU (what training-free inference costs, and the benchmark's step);
* "forces"   positions to energies, forces and virials: environment matrix, forward, fitting net, backward from
             dE/dD, force assembly (one MD force evaluation between neighbour-list rebuilds);
* "rebuild"  neighbour list and its reverse slots from positions (what an MD code repeats every few steps).

Structures are fcc lattices with thermal displacements (one species, or a random alloy) and a cubic lattice of
rigid water molecules in random orientations at 1 g/cm^3; embedding and fitting nets have random weights.  All
inputs come from the seed alone and are made by this file in plain torch.
"""
import math

import numpy as np
import torch

DEV = "cuda" if torch.cuda.is_available() else "cpu"
FIT = 240                          # width of the three fitting layers
WATER_EDGE = (18.015 / 6.02214076e23 * 1e24) ** (1.0 / 3.0)   # Angstrom per molecule at 1 g/cm^3

CU = dict(kind="fcc", a=3.634, jitter=0.1, probs="1")
AL = dict(kind="fcc", a=4.05, jitter=0.1, probs="0.9,0.05,0.05")
WATER = dict(kind="water", a=WATER_EDGE, jitter=0.0, probs="")


def listed():
    cu6 = dict(CU, rc=6.0, rcs=0.5, sel="128", m1=100, m2=16)
    cu8 = dict(CU, rc=8.0, rcs=2.0, sel="512", m1=100, m2=16)
    al8 = dict(AL, rc=8.0, rcs=2.0, sel="300,60,60", m1=100, m2=16)
    h2o = dict(WATER, rc=6.0, rcs=0.5, sel="46,92", m1=100, m2=16)
    return [
        # the smallest useful cell: a unit-cell study or one replica of many; latency counts
        dict(cu6, name="step_cu256_f64", path="step", ncell=4, dtype="f64"),
        # an ordinary liquid box, two types, half-filled lists
        dict(h2o, name="step_water12288_f64", path="step", ncell=16, dtype="f64"),
        # an alloy: three types, nine tables, most neighbours of one type
        dict(al8, name="step_alcumg32000_f64", path="step", ncell=20, dtype="f64"),
        # a wider embedding net than the usual 100 channels, an odd lattice
        dict(cu6, name="step_cu8788_m200_f64", path="step", ncell=13, m1=200, dtype="f64"),
        # a large liquid in the two single-precision modes
        dict(h2o, name="step_water331776_f32", path="step", ncell=48, dtype="f32"),
        dict(h2o, name="step_water331776_f32acc64", path="step", ncell=48, dtype="f32acc64"),
        # the headline workload: a million atoms on one GPU, long lists with much padding
        dict(cu8, name="step_cu1m_f64", path="step", ncell=64, dtype="f64"),
        # MD force evaluations: the smallest cell, an ordinary one, a large one
        dict(cu6, name="forces_cu256", path="forces", ncell=4, dtype="f64"),
        dict(h2o, name="forces_water12288", path="forces", ncell=16, dtype="f64"),
        dict(cu8, name="forces_cu131072", path="forces", ncell=32, dtype="f64"),
        # neighbour-list rebuilds: an ordinary liquid box, the large crystal
        dict(h2o, name="rebuild_water12288", path="rebuild", ncell=16, dtype="f64"),
        dict(cu8, name="rebuild_cu1m", path="rebuild", ncell=64, dtype="f64"),
    ]


def draw(rng):
    """A case of the same ranges: 256 to 500,000 atoms, other lattices, cutoffs, widths and modes."""
    path = rng.choice(["step", "step", "step", "forces", "forces", "rebuild"])
    mat = rng.choice(["cu", "al", "water"])
    if mat == "water":
        rc = rng.choice([5.0, 5.5, 6.0])
        ncell = int(round(math.exp(rng.uniform(math.log(6), math.log(50)))))
        c = dict(WATER, rc=rc, rcs=0.5, sel=rng.choice(["46,92", "48,96", "60,110"]))
    else:
        rc = rng.choice([5.5, 6.0, 7.0, 8.0])
        lo = 4 if mat == "cu" and rc <= 6 else 5
        ncell = int(round(math.exp(rng.uniform(math.log(lo), math.log(50)))))
        if mat == "cu":
            sel = rng.choice(["128", "150"]) if rc <= 6 else rng.choice(["256", "300", "512"])
        else:
            sel = rng.choice(["120,40,40", "160,30,30"]) if rc <= 6 else rng.choice(["300,60,60", "400,80,80"])
        c = dict(CU if mat == "cu" else AL, rc=rc, rcs=rng.choice([0.5, 2.0]), sel=sel)
    # the box holds two cutoffs and the displacements of both atoms
    while ncell * c["a"] < 2.0 * (rc + 2.2):
        ncell += 1
    c.update(path=path, ncell=ncell, m1=100, m2=16, dtype="f64")
    if path == "step":
        c["dtype"] = rng.choice(["f64", "f64", "f32", "f32acc64"])
        c["m1"] = rng.choice([100, 100, 64, 120, 128, 99, 200, 256])
        c["m2"] = rng.choice([16, 16, 8, 12, 15])
        if c["m1"] > 128:              # wide nets are used on smaller systems
            c["ncell"] = min(c["ncell"], 24)
    elif path == "forces":
        c["m1"] = rng.choice([100, 100, 64, 128, 80])
        c["m2"] = rng.choice([16, 16, 8])
        c["ncell"] = min(c["ncell"], 32)
    return c


# ---------------------------------------------------------------------------
# structures and lists
# ---------------------------------------------------------------------------
def _sel(case):
    return [int(v) for v in case["sel"].split(",")]


def _natoms(case):
    return (4 if case["kind"] == "fcc" else 3) * case["ncell"] ** 3


def _box(case):
    return case["ncell"] * case["a"]


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) % (1 << 62))
    return g


def _positions(case, seed):
    """(site vectors of the basis [nb, 3], types [n] int32, displacements [n, 3], coordinates [n, 3])."""
    N, a, n = case["ncell"], case["a"], _natoms(case)
    g = _gen(seed, 1)
    if case["kind"] == "fcc":
        basis = a * torch.tensor([[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]], dtype=torch.float64, device=DEV)
        # thermal displacements, at most four standard deviations per component
        disp = (torch.randn((n, 3), dtype=torch.float64, device=DEV, generator=g) * case["jitter"]).clamp(
            -4 * case["jitter"], 4 * case["jitter"])
        cum = np.cumsum([float(v) for v in case["probs"].split(",")])
        u = torch.rand(n, dtype=torch.float64, device=DEV, generator=g)
        types = sum((u >= float(c)).to(torch.int32) for c in cum[:-1]) if len(cum) > 1 else torch.zeros(
            n, dtype=torch.int32, device=DEV)
    else:
        basis = torch.zeros((3, 3), dtype=torch.float64, device=DEV)
        h, d = math.radians(104.52) / 2, 0.9572
        ref = torch.tensor([[0, 0, 0], [d * math.sin(h), 0, d * math.cos(h)], [-d * math.sin(h), 0, d * math.cos(h)]],
                           dtype=torch.float64, device=DEV)
        q = torch.randn((N ** 3, 4), dtype=torch.float64, device=DEV, generator=g)
        w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
        R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                         2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                         2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 1, 3, 3)
        disp = (R * ref.reshape(1, 3, 1, 3)).sum(-1).reshape(n, 3).contiguous()
        types = torch.tensor([0, 1, 1], dtype=torch.int32, device=DEV).repeat(N ** 3)
    nb = len(basis)
    c = torch.arange(n, device=DEV) // nb
    cell = torch.stack([c // (N * N), (c // N) % N, c % N], 1).to(torch.float64)
    coord = cell * a + basis[torch.arange(n, device=DEV) % nb] + disp
    return basis, types.to(torch.int32), disp, coord


def _offsets(basis, a, cut, b):
    """Site offsets (dx, dy, dz, basis index) within `cut` of basis site b, the atom itself left out."""
    K = int(math.ceil(cut / a)) + 1
    r = torch.arange(-K, K + 1, device=DEV)
    d = torch.stack(torch.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    rows = []
    for bp in range(len(basis)):
        keep = (d.double() * a + basis[bp] - basis[b]).norm(dim=1) < cut
        if bp == b:
            keep &= (d != 0).any(1)
        s = d[keep]
        rows.append(torch.cat([s, torch.full((len(s), 1), bp, device=DEV)], 1))
    return torch.cat(rows)


def _weight(r, rc, rcs):
    """s(r) and ds/dr of the smooth 1/r weighting."""
    u = ((r - rcs) / (rc - rcs)).clamp(0.0, 1.0)
    sw = u ** 3 * (-6 * u * u + 15 * u - 10) + 1
    dsw = -30 * u * u * (u - 1) ** 2 / (rc - rcs)
    return sw / r, (dsw - sw / r) / r


def _system(case, seed):
    """Positions, types, neighbour lists, the environment matrix and its statistics, table ranges; float64."""
    basis, types, disp, coord = _positions(case, seed)
    N, a, n, sel = case["ncell"], case["a"], _natoms(case), _sel(case)
    nt, nb, nnei = len(sel), len(basis), sum(sel)
    rc, rcs = case["rc"], case["rcs"]
    dmax = float(disp.norm(dim=1).max())
    off = torch.tensor([0] + list(np.cumsum(sel)), device=DEV)
    sel_t = torch.tensor(sel, device=DEV)
    nlist = torch.full((n, nnei), -1, dtype=torch.int32, device=DEV)
    em = torch.zeros((n, nnei, 4), dtype=torch.float64, device=DEV)
    acc = torch.zeros((nt, 5), dtype=torch.float64, device=DEV)
    smax = torch.full((nt, nt), -math.inf, dtype=torch.float64, device=DEV)
    step = 16384
    for b in range(nb):
        cand = _offsets(basis, a, rc + 2 * dmax + 1e-9, b)
        site = cand[:, :3].double() * a + basis[cand[:, 3]] - basis[b]
        for c0 in range(0, N ** 3, step):
            cell = torch.arange(c0, min(N ** 3, c0 + step), device=DEV)
            cx, cy, cz = cell // (N * N), (cell // N) % N, cell % N
            j = ((((cx[:, None] + cand[:, 0]) % N) * N + (cy[:, None] + cand[:, 1]) % N) * N
                 + (cz[:, None] + cand[:, 2]) % N) * nb + cand[:, 3]
            i = cell * nb + b
            vec = site + disp[j] - disp[i][:, None]
            r = vec.square().sum(-1).sqrt()
            tj, ti = types[j].long(), types[i].long()
            key, order = torch.where(r < rc, tj * (4.0 * rc) + r, torch.full_like(r, 1e9)).sort(1)
            ok = key < 1e8
            ts = tj.gather(1, order)
            cnt = torch.stack([((r < rc) & (tj == t)).sum(1) for t in range(nt)], 1)
            start = torch.cat([torch.zeros_like(cnt[:, :1]), cnt.cumsum(1)[:, :-1]], 1)
            rank = torch.arange(key.shape[1], device=DEV) - start.gather(1, ts)
            ok &= rank < sel_t[ts]                       # the nearest sel of each type are kept
            col = torch.where(ok, off[ts] + rank, torch.full_like(ts, nnei))
            rs, vs = r.gather(1, order), vec.gather(1, order[..., None].expand(-1, -1, 3))
            s = torch.where(ok, _weight(rs, rc, rcs)[0], torch.zeros_like(rs))
            val = torch.cat([s[..., None], s[..., None] * vs], 2)
            nl = torch.full((len(cell), nnei + 1), -1, dtype=torch.int32, device=DEV)
            nl.scatter_(1, col, torch.where(ok, j.gather(1, order), torch.full_like(j, -1)).to(torch.int32))
            e = torch.zeros((len(cell), nnei + 1, 4), dtype=torch.float64, device=DEV)
            e.scatter_(1, col[..., None].expand(-1, -1, 4), val)
            nlist[i], em[i] = nl[:, :nnei], e[:, :nnei]
            row = torch.stack([s.sum(1), s.square().sum(1), ok.sum(1).double(), val[..., 1:].sum((1, 2)),
                               val[..., 1:].square().sum((1, 2))], 1)
            for t in range(nt):
                acc[t] += row[ti == t].sum(0)
                for u in range(nt):
                    first = e[:, int(off[u]), 0][(ti == t) & (nl[:, int(off[u])] >= 0)]
                    if len(first):
                        smax[t, u] = torch.maximum(smax[t, u], first.max())
    acc, smax = acc.cpu().numpy(), smax.cpu().numpy()
    mean, sigma, sall = np.zeros(nt), np.ones(nt), np.ones(nt)
    for t in range(nt):
        ss, sq, k, vs, vq = acc[t]
        if k > 1:
            mean[t] = ss / k
            sigma[t] = math.sqrt(max(sq / k - mean[t] ** 2, 1e-12))
            sall[t] = math.sqrt(max(vq / (3 * k) - (vs / (3 * k)) ** 2, 1e-12))
    m_t, s_t, a_t = (torch.tensor(v, device=DEV) for v in (mean, sigma, sall))
    for i0 in range(0, n, 65536):
        sl = slice(i0, min(n, i0 + 65536))
        t = types[sl].long()
        em[sl, :, 0] = torch.where(nlist[sl] >= 0, (em[sl, :, 0] - m_t[t][:, None]) / s_t[t][:, None], 0.0)
        em[sl, :, 1:] /= a_t[t][:, None, None]
    lo, L1, L2 = np.zeros(nt * nt), np.ones(nt * nt, np.int64), np.ones(nt * nt, np.int64)
    for t in range(nt):
        for u in range(nt):
            p = t * nt + u
            lo[p] = -mean[t] / sigma[t]
            if np.isfinite(smax[t, u]):
                L1[p] = int(math.floor(((smax[t, u] - mean[t]) / sigma[t] - lo[p]) / 0.01)) + 1
            L2[p] = max(1, int(math.ceil(L1[p] * 0.01 / 0.1)))
    return dict(types=types, coord=coord, nlist=nlist, em=em, mean=mean, sigma=sigma, sall=sall, lo=lo, L1=L1, L2=L2)


def _nets(case, seed):
    """Random embedding nets, one per ordered type pair, widths 1 -> m1/4 -> m1/2 -> m1."""
    rng, m1 = np.random.default_rng([int(seed), 7]), case["m1"]
    w = (1, max(1, m1 // 4), max(1, m1 // 2), m1)
    return [{"W": [rng.normal(0, 1 / math.sqrt(w[k]), (w[k], w[k + 1])) for k in range(3)],
             "b": [rng.normal(0, 1, w[k + 1]) for k in range(3)]} for _ in range(len(_sel(case)) ** 2)]


def _neighbours(case):
    """Mean number of neighbours within the cutoff."""
    density = (4 if case["kind"] == "fcc" else 3) / case["a"] ** 3
    return min(sum(_sel(case)), 4.0 / 3.0 * math.pi * case["rc"] ** 3 * density)


def _fit_net(case, seed):
    """Random fitting net.  The first layer is scaled so that its pre-activations are of order one, as a trained
    model's are (D grows with the square of the number of neighbours)."""
    rng, fan, W, b = np.random.default_rng([int(seed), 8]), case["m1"] * case["m2"], [], []
    for _ in range(3):
        W.append(rng.normal(0, 1 / math.sqrt(fan), (fan, FIT)))
        b.append(rng.normal(0, 1, FIT))
        fan = FIT
    W[0] *= 4.0 / _neighbours(case) ** 2
    return {"W": W, "b": b, "w_out": rng.normal(0, 1 / math.sqrt(fan), fan), "b_out": float(rng.normal())}


def _grad(case, seed, dtype):
    return torch.randn((_natoms(case), case["m1"], 4), dtype=torch.float64, device=DEV,
                       generator=_gen(seed, 2)).to(dtype)


# ---------------------------------------------------------------------------
# the timed calls
# ---------------------------------------------------------------------------
def prepare(case, seed):
    import paper_2107_02103_amd as P
    sel, n, nt = _sel(case), _natoms(case), len(_sel(case))
    nnei, m1, m2 = sum(sel), case["m1"], case["m2"]

    def empty(*shape, dtype=torch.float64):
        return torch.empty(shape, dtype=dtype, device=DEV)

    if case["path"] == "rebuild":
        _, types, _, coord = _positions(case, seed)
        nb = P.dpc_nlist_workspace_bytes(n, _box(case), case["rc"])
        return dict(case=case, sel=sel, n=n, coord=coord, types=types, ws_bytes=nb,
                    ws=empty(nb, dtype=torch.uint8), nlist=empty(n, nnei, dtype=torch.int32),
                    rev=empty(n, nnei, dtype=torch.int32))
    s = _system(case, seed)
    mode = {"f64": P.DPC_F64, "f32": P.DPC_F32, "f32acc64": P.DPC_F32_ACC64}[case["dtype"]]
    store = torch.float64 if case["dtype"] == "f64" else torch.float32
    out = torch.float32 if case["dtype"] == "f32" else torch.float64
    op = P.SeATab(_nets(case, seed), s["lo"], s["L1"], s["L2"], 0.01, 0.1, sel, m2, dtype=mode)
    st = dict(case=case, sel=sel, n=n, op=op, types=s["types"], nlist=s["nlist"], T=empty(n, m1, 4, dtype=out),
              D=empty(n, m1, m2, dtype=out), dR=empty(n, nnei, 4, dtype=out))
    if case["path"] == "step":
        st.update(em=s["em"].to(store), dT=_grad(case, seed, store))
        return st
    net = _fit_net(case, seed)
    keep = [torch.from_numpy(v).to(DEV) for v in net["W"] + net["b"] + [net["w_out"]]]
    c = P.dpc_fitting_net()
    c.n_in, c.width, c.b_out, c.w_out = m1 * m2, FIT, net["b_out"], keep[6].data_ptr()
    for k in range(3):
        c.W[k], c.b[k] = keep[k].data_ptr(), keep[3 + k].data_ptr()
    nb = P.dpc_fitting_workspace_bytes(n, FIT)
    rev = empty(n, nnei, dtype=torch.int32)
    P.dpc_nlist_reverse(torch.cuda.current_stream(), n, nt, sel, _box(case), s["coord"], s["types"], s["nlist"], rev)
    st.update(em=empty(n, nnei, 4), coord=s["coord"], rev=rev, mean=s["mean"], sigma=s["sigma"], sall=s["sall"],
              net=c, keep=keep, ws=empty(nb // 8), ws_bytes=nb, blas=P.RocblasHandle(), E=empty(n),
              dD=empty(n, m1, m2), F=empty(n, 3), V=empty(n, 9))
    return st


def run(st):
    import paper_2107_02103_amd as P
    case, n, sel = st["case"], st["n"], st["sel"]
    nt, nnei, stream = len(sel), sum(sel), torch.cuda.current_stream()
    if case["path"] == "rebuild":
        P.dpc_nlist_build(stream, n, nt, sel, _box(case), case["rc"], st["coord"], st["types"], st["ws"],
                          st["ws_bytes"], st["nlist"], wait=False)
        P.dpc_nlist_reverse(stream, n, nt, sel, _box(case), st["coord"], st["types"], st["nlist"], st["rev"])
        return {"nlist": st["nlist"], "rev": st["rev"]}
    op = st["op"]
    if case["path"] == "step":
        op.forward(st["em"], st["nlist"], st["types"], st["T"], st["D"])
        op.backward(st["em"], st["nlist"], st["types"], st["dT"], st["dR"])
        return {"T": st["T"], "D": st["D"], "dR": st["dR"]}
    P.dpc_env_mat_a(stream, P.DPC_F64, n, nt, nnei, _box(case), case["rc"], case["rcs"], st["mean"], st["sigma"],
                    st["sall"], st["coord"], st["types"], st["nlist"], st["em"])
    op.forward(st["em"], st["nlist"], st["types"], st["T"], st["D"])
    P.dpc_fitting_fwd_bwd(stream, st["blas"].value, n, st["net"], st["D"], st["ws"], st["ws_bytes"], st["E"],
                          st["dD"])
    op.backward_from_dD(st["em"], st["nlist"], st["types"], st["T"], st["dD"], st["dR"])
    P.dpc_force_a(stream, P.DPC_F64, n, nt, nnei, _box(case), case["rc"], case["rcs"], st["sigma"], st["sall"],
                  st["coord"], st["types"], st["nlist"], st["rev"], st["dR"], st["F"], st["V"])
    return {"E": st["E"], "F": st["F"], "V": st["V"], "D": st["D"], "dD": st["dD"], "dR": st["dR"]}


def work(case):
    """Inputs read once, outputs written once; FLOP of the method (one quintic per neighbour and channel)."""
    n, sel, m1, m2 = _natoms(case), _sel(case), case["m1"], case["m2"]
    nnei, pairs = sum(sel), n * _neighbours(case)
    es, eo = 8 if case["dtype"] == "f64" else 4, 4 if case["dtype"] == "f32" else 8
    if case["path"] == "rebuild":
        # positions and types in, the list out; the list in, the reverse slots out; one distance per neighbour
        return {"bytes": 28.0 * n + 12.0 * n * nnei, "flops": 20.0 * pairs}
    desc = pairs * 54.0 * m1 + n * 8.0 * m1 * m2
    if case["path"] == "step":
        fwd = 4 * n * nnei + 4 * es * pairs + n * (4 * m1 + m1 * m2) * eo
        bwd = 4 * n * nnei + 4 * es * pairs + n * 4 * m1 * es + 4 * eo * n * nnei
        return {"bytes": float(fwd + bwd), "flops": desc}
    fit = 4.0 * n * (m1 * m2 * FIT + 2 * FIT * FIT)
    env = 28 * n + 4 * n * nnei + 32 * n * nnei
    fwd = 4 * n * nnei + 32 * pairs + 8 * n * (4 * m1 + m1 * m2)
    mid = 8 * n * (2 * m1 * m2 + 1)
    bwd = 4 * n * nnei + 32 * pairs + 8 * n * (4 * m1 + m1 * m2) + 32 * n * nnei
    frc = 28 * n + 8 * n * nnei + 32 * n * nnei + 32 * pairs + 96 * n
    return {"bytes": float(env + fwd + mid + bwd + frc), "flops": desc + fit + n * 16.0 * m1 * m2 + 150.0 * pairs}


def tolerance(case):
    """About four times the distance to the same path in plain float64 (float32 tables and inputs in the
    single-precision modes; forces of a crystal near its lattice sites cancel to a few parts in 1e13)."""
    if case["path"] == "rebuild":
        return "exact"
    if case["path"] == "forces":
        return {"rel": 6e-12, "max": 4e-11}
    return {"f64": {"rel": 2e-13, "max": 2e-11}, "f32": {"rel": 1.2e-6, "max": 2e-5},
            "f32acc64": {"rel": 1.6e-7, "max": 3e-6}}[case["dtype"]]


# ---------------------------------------------------------------------------
# the same values in plain float64
# ---------------------------------------------------------------------------
def _net_jet(net, x):
    """Value, first and second derivative of an embedding net at the points x."""
    y, d, e = x[:, None], np.ones((len(x), 1)), np.zeros((len(x), 1))
    for W, b in zip(net["W"], net["b"]):
        t, u, v = np.tanh(y @ W + b), d @ W, e @ W
        g = 1 - t * t
        t, u, v = t, g * u, g * v - 2 * t * g * u * u
        if W.shape[1] == 2 * W.shape[0]:
            t, u, v = t + np.hstack([y, y]), u + np.hstack([d, d]), v + np.hstack([e, e])
        elif W.shape[1] == W.shape[0]:
            t, u, v = t + y, u + d, v + e
        y, d, e = t, u, v
    return y, d, e


def _table(net, lo, L1, L2):
    """Quintic Hermite coefficients [L1 + L2, 6, m1] on the main range (0.01) and the band (0.1)."""
    parts = []
    for org, h, k in ((lo, 0.01, L1), (lo + L1 * 0.01, 0.1, L2)):
        y, d, e = _net_jet(net, org + h * np.arange(k + 1))
        dy, d0, d1, e0, e1 = y[1:] - y[:-1], d[:-1], d[1:], e[:-1], e[1:]
        parts.append(np.stack([
            y[:-1], d0, e0 / 2, (20 * dy - (8 * d1 + 12 * d0) * h - (3 * e0 - e1) * h * h) / (2 * h ** 3),
            (-30 * dy + (14 * d1 + 16 * d0) * h + (3 * e0 - 2 * e1) * h * h) / (2 * h ** 4),
            (12 * dy - 6 * (d1 + d0) * h + (e1 - e0) * h * h) / (2 * h ** 5)], 1))
    return np.concatenate(parts)


class _Exact:
    """The descriptor of one system, evaluated neighbour by neighbour in float64."""

    def __init__(self, case, seed, s):
        self.case, self.sel = case, _sel(case)
        nt, nets = len(self.sel), _nets(case, seed)
        self.s = s
        tabs = [_table(nets[p], s["lo"][p], int(s["L1"][p]), int(s["L2"][p])) for p in range(nt * nt)]
        self.base = torch.tensor(np.concatenate([[0], np.cumsum([len(t) for t in tabs])[:-1]]), device=DEV)
        self.coef = torch.from_numpy(np.concatenate(tabs)).to(DEV)
        self.lo, self.L1, self.L2 = (torch.from_numpy(s[k]).to(DEV) for k in ("lo", "L1", "L2"))
        self.blk = torch.tensor(np.repeat(np.arange(nt), self.sel), device=DEV)

    def chunks(self, size=4096):
        n = len(self.s["types"])
        for i0 in range(0, n, size):
            sl = slice(i0, min(n, i0 + size))
            ok = self.s["nlist"][sl] >= 0
            yield sl, ok.any(0).nonzero()[:, 0]

    def values(self, em, sl, cols):
        """R~ rows of the valid columns, g and g' of every row and channel (zero where there is no neighbour)."""
        R, ok = em[sl][:, cols].double(), (self.s["nlist"][sl][:, cols] >= 0)
        p = self.s["types"][sl].long()[:, None] * len(self.sel) + self.blk[cols]
        x = R[..., 0]
        up = self.lo[p] + self.L1[p] * 0.01
        main = x < up
        q = torch.where(main, (x - self.lo[p]) / 0.01, (x - up) / 0.1).floor()
        q = torch.minimum(q.clamp(min=0), torch.where(main, self.L1[p], self.L2[p]) - 1.0)
        t = x - torch.where(main, self.lo[p] + q * 0.01, up + q * 0.1)
        row = self.base[p] + q.long() + torch.where(main, torch.zeros_like(p), self.L1[p])
        t, okf = t[..., None], ok[..., None].double()
        v = d = self.coef[:, 5][row]
        for k in (4, 3, 2, 1):
            v = v * t + self.coef[:, k][row]
            d = d * t + v
        v = v * t + self.coef[:, 0][row]
        return R, v * okf, d * okf

    def forward(self, em):
        n, m1, m2 = len(self.s["types"]), self.case["m1"], self.case["m2"]
        T = torch.empty((n, m1, 4), dtype=torch.float64, device=DEV)
        D = torch.empty((n, m1, m2), dtype=torch.float64, device=DEV)
        for sl, cols in self.chunks():
            R, g, _ = self.values(em, sl, cols)
            t = torch.bmm(g.transpose(1, 2).contiguous(), R)
            T[sl] = t
            D[sl] = torch.bmm(t, t[:, :m2].transpose(1, 2).contiguous())
        return T, D

    def backward(self, em, dT):
        n, nnei = len(self.s["types"]), sum(self.sel)
        dR = torch.zeros((n, nnei, 4), dtype=torch.float64, device=DEV)
        for sl, cols in self.chunks():
            R, g, d = self.values(em, sl, cols)
            dt = dT[sl].double()
            out = torch.bmm(g, dt)
            out[..., 0] += (d * torch.bmm(R, dt.transpose(1, 2).contiguous())).sum(-1)
            out *= (self.s["nlist"][sl][:, cols] >= 0)[..., None]
            full = torch.zeros((out.shape[0], nnei, 4), dtype=torch.float64, device=DEV)
            full[:, cols] = out
            dR[sl] = full
        return dR


def _exact_forces(case, seed, s):
    ex = _Exact(case, seed, s)
    T, D = ex.forward(s["em"])
    net, n, m2 = _fit_net(case, seed), _natoms(case), case["m2"]
    W, b = [torch.from_numpy(v).to(DEV) for v in net["W"]], [torch.from_numpy(v).to(DEV) for v in net["b"]]
    wo = torch.from_numpy(net["w_out"]).to(DEV)
    E, dT, dDs = torch.empty(n, dtype=torch.float64, device=DEV), torch.empty_like(T), torch.empty_like(D)
    Wt = [w.t().contiguous() for w in W]
    for i0 in range(0, n, 16384):
        sl = slice(i0, min(n, i0 + 16384))
        t1 = torch.tanh(D[sl].reshape(-1, W[0].shape[0]) @ W[0] + b[0])
        t2 = torch.tanh(t1 @ W[1] + b[1])
        h2 = t1 + t2
        t3 = torch.tanh(h2 @ W[2] + b[2])
        E[sl] = (h2 + t3) @ wo + net["b_out"]
        g = wo + ((1 - t3 * t3) * wo) @ Wt[2]
        g = g + ((1 - t2 * t2) * g) @ Wt[1]
        dD = (((1 - t1 * t1) * g) @ Wt[0]).reshape(-1, case["m1"], m2)
        t, dDs[sl] = T[sl], dD
        dt = torch.bmm(dD, t[:, :m2].contiguous())
        dt[:, :m2] += torch.bmm(dD.transpose(1, 2).contiguous(), t)
        dT[sl] = dt
    dR = ex.backward(s["em"], dT)
    F = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    V = torch.zeros((n, 9), dtype=torch.float64, device=DEV)
    L, sg, sa = _box(case), torch.from_numpy(s["sigma"]).to(DEV), torch.from_numpy(s["sall"]).to(DEV)
    for sl, cols in ex.chunks(16384):
        nl, lam = s["nlist"][sl][:, cols].long(), dR[sl][:, cols]
        ok = nl >= 0
        i = torch.arange(sl.start, sl.stop, device=DEV)
        j = torch.where(ok, nl, i[:, None])
        d = s["coord"][j] - s["coord"][sl][:, None]
        d = d - L * (d / L).round()
        r = torch.where(ok, d.square().sum(-1).sqrt(), torch.ones((), dtype=torch.float64, device=DEV))
        w, dw = _weight(r, case["rc"], case["rcs"])
        t = s["types"][sl].long()
        c1 = dw / r * (lam[..., 0] / sg[t][:, None] + (lam[..., 1:] * d).sum(-1) / sa[t][:, None])
        g = (c1[..., None] * d + (w / sa[t][:, None])[..., None] * lam[..., 1:]) * ok[..., None]
        F[sl] += g.sum(1)
        F.index_add_(0, j.reshape(-1), -g.reshape(-1, 3))
        V[sl] = -(d[..., :, None] * g[..., None, :]).sum(1).reshape(-1, 9)
    return {"E": E, "F": F, "V": V, "D": D, "dD": dDs, "dR": dR}


def exact(case, seed):
    if case["path"] == "rebuild":
        return None
    s = _system(case, seed)
    if case["path"] == "forces":
        return _exact_forces(case, seed, s)
    store = torch.float64 if case["dtype"] == "f64" else torch.float32
    em = s["em"] = s["em"].to(store)
    ex = _Exact(case, seed, s)
    T, D = ex.forward(em)
    return {"T": T, "D": D, "dR": ex.backward(em, _grad(case, seed, store))}
