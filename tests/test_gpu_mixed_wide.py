"""The mixed mode's backward above 128 channels: up to 208 it is float64
arithmetic on float32 inputs whatever the length of the list, as the header
says, so it equals the float64 mode on the same (widened) table and inputs to
float64 rounding, which float32 polynomials miss by six orders of magnitude;
above 208 the polynomial is float32."""
import numpy as np
import pytest

from parity import TOL, normwise
from synth.edge import edge_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE = 43


@pytest.mark.parametrize("m1", [129, 160, 161, 176, 208, 209, 256])
@pytest.mark.parametrize("sel", [(40, 33), (200,), (256,), (257,), (30, 241)])
def test_float64_up_to_208_channels(m1, sel):
    import paper_2107_02103_amd as P
    x = edge_inputs(BASE, sel, m1, 8, seed=m1 + sum(sel))
    c = x.cfg
    mixed, f64 = (P.SeATab(x.nets, x.lo, x.L1, x.L2, c.d1, c.d2, c.sel, c.m2, dtype=d)
                  for d in (P.DPC_F32_ACC64, P.DPC_F64))
    f64.coeff.copy_(mixed.coeff)                  # the same layout in elements: the float32 table, widened
    em, nl, at, dT = (torch.from_numpy(v).cuda() for v in (x.em, x.nlist, x.atype, x.dT))
    em, dT = em.float(), dT.float()
    for n in (BASE, 2100, 10300):                 # runs shared out, and not
        a = [t.repeat((n // BASE + 1,) + (1,) * (t.dim() - 1))[:n].contiguous() for t in (em, nl, at, dT)]
        got = mixed.backward(*a).cpu().numpy()
        ref = f64.backward(a[0].double(), a[1], a[2], a[3].double()).cpu().numpy()
        err = normwise(got, ref)
        print(f"[gpu-mixed-wide] m1 {m1} sel {sel} n {n}: {err:.2e}", flush=True)
        assert err <= (TOL["f64"] if m1 <= 208 else TOL["f32acc64"]), (n, err)
        assert m1 <= 208 or err > 1e-10           # (and the header's float32 is what runs)
