"""Calls of more workgroups than one launch takes (HIP: fewer than 2^32 threads per
grid dimension): the points come in a pattern of 1024, so every output row repeats
what a call of 1024 points gives."""
import ctypes as C

import numpy as np
import pytest

from paper_2411_02640_amd import inputs as I

from . import tiny_mechs as TM

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
PERIOD = 1024


def _states(ns, n):
    T, p, Y = I.make_states(ns, I.StateSpec(PERIOD, seed=93, p_atm_range=(1.0, 40.0),
                                            dirichlet_alpha=0.3))
    small = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]

    def tiled(a):
        out = torch.empty(a.shape[:-1] + (n,), dtype=a.dtype, device=a.device)
        full = n // PERIOD * PERIOD
        for row, src in zip(out.view(-1, n), a.view(-1, PERIOD)):
            row[:full].view(-1, PERIOD).copy_(src)
            row[full:].copy_(src[:n - full])
        return out

    return small, [tiled(a) for a in small]


def _repeats(big, small):
    n = big.shape[-1]
    full = n // PERIOD * PERIOD
    for row, src in zip(big.view(-1, n), small.view(-1, PERIOD)):
        if not torch.equal(row[:full].view(-1, PERIOD), src.expand(full // PERIOD, PERIOD)):
            return False
        if not torch.equal(row[full:], src[:n - full]):
            return False
    return True


def _free():
    torch.cuda.empty_cache()


def _call(kx, dm, name, d, out):
    """One call through the C entry point, into `out` (thermo: cp only)."""
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    n, (T, p, Y) = d[0].shape[0], [t.data_ptr() for t in d]
    if name == "thermo":
        kx.check(kx.lib().kx_thermo(dm.handle, n, T, Y, None, None, out.data_ptr(), st))
    elif name == "rates":
        kx.check(kx.lib().kx_production_rates(dm.handle, n, T, p, Y, out.data_ptr(), st))
    else:
        kx.check(kx.lib().kx_qss_concentrations(dm.handle, n, T, p, Y, out.data_ptr(), st))


@pytest.mark.parametrize("name", ["thermo", "rates", "qss"])
def test_beyond_2_30_points(name):
    """Five species (four waves a tile, or 256 threads): at most 103 GB."""
    from paper_2411_02640_amd import kx
    n = (1 << 30) + 65
    mech = TM.qss_chain_mechanism((TM.Q1_, TM.Q2_))
    if name != "qss":
        mech["qss"] = None
    dm = kx.Mechanism(mech, 0)
    print("[gpu-case] beyond 2^30 points", name, flush=True)
    small, big = _states(5, n)
    rows = {"thermo": (), "rates": (5,), "qss": (2,)}[name]
    ref = torch.empty(rows + (PERIOD,), dtype=torch.float64, device="cuda:0")
    out = torch.empty(rows + (n,), dtype=torch.float64, device="cuda:0")
    _call(kx, dm, name, small, ref)
    _call(kx, dm, name, big, out)
    assert _repeats(out, ref)
    dm.close()
    del big, out
    _free()
