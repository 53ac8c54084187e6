"""The fitting net of width 240 on the matrix cores: both sides of every atom
count at which its kernels change (16, 48 or 240 channels per workgroup, one
launch per product or one for the middle of the net), input widths that end
inside a chunk of 16, energies alone, and the plain-GEMM path for what the
kernels do not take (other widths, n_in not a multiple of 4, buffers 8 bytes
off), against the numpy oracle."""
import numpy as np
import pytest

import oracle.fitting as fn
from synth.system import random_fitting_net

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


class Net:
    def __init__(self, n_in, width, seed):
        import paper_2107_02103_amd as P
        self.net = random_fitting_net(np.random.default_rng(seed), n_in, (width,) * 3)
        self.keep = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
                     for a in self.net["W"] + self.net["b"] + [self.net["w_out"]]]
        self.c = P.dpc_fitting_net()
        self.c.n_in, self.c.width, self.c.b_out = n_in, width, self.net["b_out"]
        for k in range(3):
            self.c.W[k], self.c.b[k] = self.keep[k].data_ptr(), self.keep[3 + k].data_ptr()
        self.c.w_out = self.keep[6].data_ptr()
        self.blas = P.RocblasHandle()

    def run(self, D, grad=True, shift=0):
        import paper_2107_02103_amd as P
        n, (m1, m2) = len(D), D.shape[1:]
        buf = torch.empty(D.size + shift, dtype=torch.float64, device="cuda")
        Dg = buf[shift:].view(D.shape)
        Dg.copy_(torch.from_numpy(D))
        nb = P.dpc_fitting_workspace_bytes(n, self.c.width)
        # NaN in the workspace and past the outputs: nothing is read before it is written, nothing written past
        ws = torch.full((nb // 8 + 64,), float("nan"), dtype=torch.float64, device="cuda")
        E = torch.full((n + 8,), 7.0, dtype=torch.float64, device="cuda")
        G = torch.full((n + 1, m1, m2), 7.0, dtype=torch.float64, device="cuda")
        P.dpc_fitting_fwd_bwd(torch.cuda.current_stream(), self.blas.value, n, self.c, Dg, ws, nb, E,
                              G if grad else None)
        torch.cuda.synchronize()
        assert torch.isnan(ws[nb // 8:]).all() and (E[n:] == 7.0).all() and (G[n:] == 7.0).all()
        return E[:n].cpu().numpy(), G[:n].cpu().numpy()


def _errors(net, D, E, G):
    Er, _ = fn.forward(D, net)
    Gr = fn.backward(D, net)
    scale = np.abs(Gr).reshape(len(Gr), -1).max(1)
    return np.max(np.abs(E - Er)) / np.max(np.abs(Er)), np.max(np.abs(G - Gr).reshape(len(Gr), -1).max(1) / scale)


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65, 512, 513, 2048, 2049, 4096, 4097, 8200, 12289])
def test_atom_counts(n):
    net = Net(100 * 4, 240, 3)
    D = np.random.default_rng(n).standard_normal((n, 100, 4))
    E, G = net.run(D)
    eE, eG = _errors(net.net, D, E, G)
    print(f"[gpu-fitting] n={n} E {eE:.2e} dE/dD {eG:.2e}", flush=True)
    assert eE <= TOL and eG <= TOL
    E2, _ = net.run(D, grad=False)
    np.testing.assert_array_equal(E, E2)
    E3, G3 = net.run(D)
    np.testing.assert_array_equal(E, E3)
    np.testing.assert_array_equal(G, G3)


@pytest.mark.parametrize("m1,m2", [(1, 4), (5, 4), (3, 12), (15, 16), (61, 4), (99, 12), (256, 16)])
def test_input_widths(m1, m2):
    net = Net(m1 * m2, 240, m1)
    for n in (70, 530, 2100, 12300):
        D = np.random.default_rng(n + m1).standard_normal((n, m1, m2))
        D[n // 2, 0, 0] = np.nan               # stays in its atom
        E, G = net.run(D)
        ok = np.arange(n) != n // 2
        assert np.isnan(E[~ok]).all() and np.isnan(G[~ok]).all()
        pick = np.flatnonzero(ok)[:: max(1, n // 500)]
        eE, eG = _errors(net.net, D[pick], E[pick], G[pick])
        print(f"[gpu-fitting] n_in={m1 * m2} n={n} E {eE:.2e} dE/dD {eG:.2e}", flush=True)
        assert eE <= TOL and eG <= TOL and np.isfinite(E[ok]).all() and np.isfinite(G[ok]).all()


@pytest.mark.parametrize("n", [3841, 4000, 4096, 7700, 8000])
@pytest.mark.parametrize("m1,m2", [(5, 4), (100, 16)])
def test_layer_of_four_tiles(n, m1, m2):
    # atom counts whose first layer runs in four groups of channel tiles, of which the last has three
    net = Net(m1 * m2, 240, n + m1)
    D = np.random.default_rng(n).standard_normal((n, m1, m2))
    E, G = net.run(D)
    pick = np.r_[0:n:max(1, n // 400), n - 65:n]
    eE, eG = _errors(net.net, D[pick], E[pick], G[pick])
    assert eE <= TOL and eG <= TOL and np.isfinite(E).all() and np.isfinite(G).all()


@pytest.mark.parametrize("m1,m2,width,shift", [(7, 3, 240, 0), (9, 6, 240, 0), (20, 4, 240, 1), (20, 4, 256, 0),
                                               (20, 4, 48, 0)])
def test_general_path(m1, m2, width, shift):
    net = Net(m1 * m2, width, 11)
    D = np.random.default_rng(5).standard_normal((77, m1, m2))
    E, G = net.run(D, shift=shift)
    eE, eG = _errors(net.net, D, E, G)
    assert eE <= TOL and eG <= TOL
