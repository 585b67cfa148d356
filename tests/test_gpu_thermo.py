"""Mixture thermo at the remainders of its tiles (64 points, four waves over the
species, four rows a trip) and with each output left out, against the oracle."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as O
from paper_2411_02640_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ns,nr,n", [(9, 21, 1), (17, 119, 64), (53, 325, 129), (200, 1500, 63)])
def test_tiles_and_optional_outputs(ns, nr, n):
    from paper_2411_02640_amd import kx
    spec = {9: I.MECH_9, 53: I.MECH_53, 200: I.MECH_200}.get(
        ns, I.MechSpec(17, 98, 12, 2, 7, seed=9017))
    mech = I.make_mechanism(spec)
    print("[gpu-case] thermo", ns, n, flush=True)
    T, p, Y = I.make_states(ns, I.StateSpec(n, seed=80, dirichlet_alpha=0.3))
    Td, Yd = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, Y)]
    dm = kx.Mechanism(mech, 0)
    cpk, hk, cp = kx.thermo(dm, Td, Yd)
    R, W = 8.31446261815324e7, np.asarray(mech["composition"] @ mech["elem_mass"], float)
    for i in {0, n // 2, n - 1}:
        c, h = [np.asarray(a) for a in O.OracleMech(mech).thermo(T[i])[:2]]
        rc, rh = c * R / W, h * R * T[i] / W
        # about ten roundings of terms up to four times the sum
        assert np.allclose(cpk[:, i].cpu().numpy(), rc, rtol=1e-14, atol=0)
        assert np.all(np.abs(hk[:, i].cpu().numpy() - rh) <= 1e-14 * np.abs(rh).max())
        assert abs(cp[i].item() - (Y[:, i] * rc).sum()) <= 1e-14 * abs((Y[:, i] * rc).sum())
    only = torch.full_like(cp, float("nan"))
    vp = lambda t: C.c_void_p(t.data_ptr()) if t is not None else None
    for outs, want in (((None, None, only), cp), ((torch.full_like(cpk, 0), None, None), cpk),
                       ((None, torch.full_like(hk, 0), None), hk)):
        kx.check(kx.lib().kx_thermo(dm.handle, n, vp(Td), vp(Yd), *[vp(t) for t in outs],
                                    C.c_void_p(torch.cuda.current_stream().cuda_stream)))
        got = next(t for t in outs if t is not None)
        assert torch.equal(got, want)
    dm.close()
