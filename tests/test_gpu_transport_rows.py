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


@pytest.mark.parametrize("ns,order,n", [(24, 5, 65), (33, 4, 64), (48, 5, 63), (49, 5, 1),
                                        (129, 5, 33), (200, 4, 17)])
def test_matrix_core_shapes_against_the_oracle(ns, order, n):
    """The matrix-core kernel at the edges of its tile shapes (512 threads below
    four row blocks; above 128 species 16 points in FP64, 32 in the mixed path)."""
    from paper_2411_02640_amd import kx
    print("[gpu-case] transport mfma", ns, order, n, flush=True)
    mech = I.make_mechanism(I.MechSpec(ns, 5 * ns, ns // 2, 0, 2, seed=9000 + ns, fit_order=order))
    T, p, Y = I.make_states(ns, I.StateSpec(n, seed=82, p_atm_range=(1.0, 40.0), dirichlet_alpha=0.3))
    Y[:, 0] = 0.0
    Y[ns - 1, 0] = 1.0
    ref = O.OracleMech(mech).transport(T, p, Y)
    dm = kx.Mechanism(mech, 0)
    d = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]
    for prec, tol in (("fp64", PM.REL_FP64), ("mixed", PM.REL_MIXED)):
        for g, r in zip(kx.transport(dm, *d, precision=prec), ref):
            rep = PM.rel_report(g.cpu().numpy(), r, tol)
            assert rep["ok"], (prec, rep)
    dm.close()
