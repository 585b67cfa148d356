"""The vector-ALU transport kernel at the edges of its shapes: species per wave
(4, 8, 16), a last wave with one species, chunks of 32 species with an odd
remainder, tile remainders, other fit orders, both fit kinds."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2411_02640_amd import inputs as I

from . import parity as PM

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ns,kind,order,n", [(9, 1, 5, 64), (17, 1, 5, 65), (23, 1, 3, 1),
                                             (33, 0, 5, 63), (64, 0, 4, 66), (65, 0, 5, 5),
                                             (129, 0, 5, 3), (200, 0, 5, 2)])
def test_shapes_against_the_oracle(ns, kind, order, n):
    from paper_2411_02640_amd import kx
    print("[gpu-case] transport rows", ns, kind, order, n, flush=True)
    if ns == 9:
        spec = I.MechSpec(9, 17, 3, 0, 1, seed=9021, diff_fit_kind=kind, fit_order=order)
    else:
        spec = I.MechSpec(ns, 5 * ns, ns // 2, 0, 2, seed=9000 + ns, diff_fit_kind=kind,
                          fit_order=order)
    mech = I.make_mechanism(spec)
    T, p, Y = I.make_states(ns, I.StateSpec(n, seed=81, p_atm_range=(1.0, 40.0), dirichlet_alpha=0.3))
    Y[:, 0] = 0.0
    Y[ns - 1, 0] = 1.0  # a pure species: D_km -> D_kk
    ref = O.OracleMech(mech).transport(T, p, Y)
    dm = kx.Mechanism(mech, 0)
    d = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]
    for prec, tol in (("fp64", PM.REL_FP64), ("mixed", PM.REL_MIXED)):
        out = kx.transport(dm, *d, precision=prec)
        for g, r in zip(out, ref):
            assert PM.rel_report(g.cpu().numpy(), r, tol)["ok"], (prec, PM.rel_report(g.cpu().numpy(), r, tol))
    dm.close()
