"""The one-lane-per-point rates kernel at the edges of its shapes: waves per
workgroup (4, 8, 12, 16 by species count), the last species count it takes, tile
remainders, and the switch from one tile per CU to shared CUs."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2411_02640_amd import inputs as I

from . import parity as PM

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mech(ns):
    nr = 7 * ns
    fall, three, lind = max(1, nr * 6 // 100), nr // 10, nr // 50
    return I.make_mechanism(I.MechSpec(ns, nr - fall - three - lind, three, lind, fall, seed=9000 + ns))


def _run(kx, dm, T, p, Y, prec):
    d = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]
    return kx.production_rates(dm, *d, precision=prec).cpu().numpy()


@pytest.mark.parametrize("ns,n", [(17, 63), (32, 64), (33, 65), (56, 16385), (57, 129),
                                  (128, 70), (129, 5), (24, 1)])
def test_shapes_against_the_oracle(ns, n):
    from paper_2411_02640_amd import kx
    print("[gpu-case] wide rates", ns, n, flush=True)
    mech = _mech(ns)
    T, p, Y = I.make_states(ns, I.StateSpec(n, seed=77, p_atm_range=(1.0, 40.0), dirichlet_alpha=0.3))
    ref, s = O.OracleMech(mech).production_rates(T, p, Y)
    dm = kx.Mechanism(mech, 0)
    for prec in ("fp64", "mixed"):
        w = _run(kx, dm, T, p, Y, prec)
        if prec == "fp64":
            r = PM.wdot_report(w, ref, s)
            assert r["ok"], r
        else:
            assert np.all(np.abs(w - ref) <= 1e-5 * s + 1e-300)
        # a call of few tiles (16 waves a tile) gives the same bits
        m = min(n, 100)
        assert np.array_equal(_run(kx, dm, T[:m], p[:m], Y[:, :m], prec), w[:, :m])
    dm.close()


@pytest.mark.parametrize("spec,n", [(I.MECH_53Q, 16385 + 7), (I.MECH_53XQ, 16385)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_qss_kernels_agree(spec, n):
    """C_Q and the rates of a QSS mechanism: the same bits from calls of few tiles
    (16 waves a tile) and of many; one wave per point (small calls) against the
    oracle's bound through the rates' own term sizes."""
    from paper_2411_02640_amd import kx
    print("[gpu-case] wide qss", spec.name, n, flush=True)
    mech = I.make_mechanism(spec)
    T, p, Y = I.make_states(53, I.StateSpec(n, seed=79, p_atm_range=(1.0, 40.0), dirichlet_alpha=0.3))
    dm = kx.Mechanism(mech, 0)
    d = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]

    def first(m):
        return d[0][:m].clone(), d[1][:m].clone(), d[2][:, :m].contiguous()

    C, w = kx.qss_concentrations(dm, *d), kx.production_rates(dm, *d)
    s = first(4097)
    assert torch.equal(kx.qss_concentrations(dm, *s), C[:, :4097])
    assert torch.equal(kx.production_rates(dm, *s), w[:, :4097])
    assert bool((w[np.flatnonzero(mech["qss"]).tolist()] == 0).all())
    # two evaluations of one balance differ by rounding times its condition, at
    # most 2e6 for these states, of terms good to 3e-13
    c1 = kx.qss_concentrations(dm, *first(4096))
    assert bool(((c1 - C[:, :4096]).abs() <= 6e-7 * C[:, :4096].abs()).all())
    assert float(((c1 - C[:, :4096]).abs() / C[:, :4096].abs()).median()) <= 1e-12
    dm.close()


@pytest.mark.parametrize("ns", [9, 53, 128])
def test_no_reactions(ns):
    """A mechanism without reactions: wdot is 0."""
    from paper_2411_02640_amd import kx
    print("[gpu-case] wide rates without reactions", ns, flush=True)
    dm = kx.Mechanism(I.make_mechanism(I.MechSpec(ns, 0, 0, 0, 0, seed=1)), 0)
    T, p, Y = I.make_states(ns, I.StateSpec(70, seed=77, p_atm_range=(1.0, 40.0), dirichlet_alpha=0.3))
    for prec in ("fp64", "mixed"):
        assert np.all(_run(kx, dm, T, p, Y, prec) == 0.0)
    dm.close()
