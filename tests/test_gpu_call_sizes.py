"""A point's results do not depend on how many points a call has: the forms that a
call's size selects (one point per workgroup, one lane per point with every tile on
a CU of its own or with several to a CU) give the same bits."""
import numpy as np
import pytest

from paper_2411_02640_amd import inputs as I

from . import tiny_mechs as TM

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mech(ns, nq=0, seed=0, nr=0, **kw):
    nr = nr or 7 * ns
    fall, three, lind = max(1, nr * 6 // 100), nr // 10, nr // 50
    return I.make_mechanism(I.MechSpec(ns, nr - fall - three - lind, three, lind, fall,
                                       seed=seed or 9000 + ns, n_qss=nq, **kw))


def _states(ns, n, seed=91):
    s = I.make_states(ns, I.StateSpec(n, seed=seed, p_atm_range=(0.2, 40.0), dirichlet_alpha=0.3))
    return [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in s]


def _first(d, m):
    return d[0][:m].clone(), d[1][:m].clone(), d[2][:, :m].contiguous()


QSS = {"chain2": lambda: TM.qss_chain_mechanism((TM.Q1_, TM.Q2_)),  # 4 waves
       "24sp-4": lambda: _mech(24, 4, 9031),                        # 8 waves
       "53Q": lambda: I.make_mechanism(I.MECH_53Q),                 # 12 waves
       "53XQ": lambda: I.make_mechanism(I.MECH_53XQ),
       "56sp-7": lambda: _mech(56, 7),                              # every column of [A | b]
       "80sp-7": lambda: _mech(80, 7)}                              # 16 waves


@pytest.mark.parametrize("name", list(QSS))
def test_qss(name):
    from paper_2411_02640_amd import kx
    mech = QSS[name]()
    n = 16384 + 70
    dm = kx.Mechanism(mech, 0)
    d = _states(mech["n_species"], n)
    print("[gpu-case] qss call sizes", name, flush=True)
    C, w = kx.qss_concentrations(dm, *d), kx.production_rates(dm, *d)
    for m in (1, 512, 513, 1025, 2049, 4096, 4097, 16384):
        s = _first(d, m)
        assert torch.equal(kx.qss_concentrations(dm, *s), C[:, :m]), m
        assert torch.equal(kx.production_rates(dm, *s), w[:, :m]), m
    dm.close()


def _repeated(mech, times):
    """The mechanism with every reaction listed `times` times."""
    m, nr = dict(mech), mech["n_reactions"]
    for key in ("reac", "prod", "eff"):
        cnt = np.diff(m[key + "_ptr"])
        m[key + "_ptr"] = np.concatenate([[0], np.cumsum(np.tile(cnt, times))]).astype(np.int32)
        for part in ("_sp", "_nu", "_val"):
            if key + part in m:
                m[key + part] = np.tile(m[key + part], times)
    for key, v in mech.items():
        if isinstance(v, np.ndarray) and v.shape[:1] == (nr,) and key not in ("qss", "t_mid") \
                and not key.endswith(("_sp", "_nu", "_val", "fit")) and "nasa" not in key \
                and key != "composition":
            m[key] = np.tile(v, (times,) + (1,) * (v.ndim - 1))
    m["n_reactions"] = nr * times
    return m


def test_qss_mechanism_too_large():
    """A mechanism whose reaction terms exceed one workgroup's LDS is refused whatever
    the number of points."""
    from paper_2411_02640_amd import kx
    mech = _repeated(TM.qss_chain_mechanism((TM.Q1_, TM.Q2_)), 2500)
    assert mech["n_reactions"] * 16 > 160 * 1024
    dm = kx.Mechanism(mech, 0)
    for n in (10, 5000):
        print("[gpu-case] qss too large", n, flush=True)
        with pytest.raises(kx.KxError) as e:
            kx.production_rates(dm, *_states(5, n))
        assert e.value.code == kx.KX_EUNSUPPORTED
    dm.close()


RATES = {"17sp": lambda: _mech(17),                    # 8 waves a tile, 119 reactions
         "24sp": lambda: _mech(24),
         "53X": lambda: I.make_mechanism(I.MECH_53X),  # 12 waves, every reaction form
         "53O": lambda: I.make_mechanism(I.MECH_53O),
         "57sp": lambda: _mech(57),                    # 16 waves
         "128sp": lambda: _mech(128),
         "128sp-1231": lambda: _mech(128, nr=1231),    # one wave per point: not all resident
         "53sp-2000": lambda: _mech(53, nr=2000)}


# the ends of the ranges of 4, 8 and 12 waves a tile
ENDS = {f"{ns}sp": (lambda ns=ns: _mech(ns)) for ns in (16, 32, 33, 56)}


@pytest.mark.parametrize("name", ["9sp", "200sp"] + list(RATES) + list(ENDS))
def test_rates(name):
    """Also the points past the first tile of every CU, and the batched call."""
    from paper_2411_02640_amd import kx
    mech = {"9sp": lambda: I.make_mechanism(I.MECH_9),
            "200sp": lambda: I.make_mechanism(I.MECH_200), **RATES, **ENDS}[name]()
    ns, n = mech["n_species"], 16384 + 4097
    dm = kx.Mechanism(mech, 0)
    d = _states(ns, n)
    d[2][:, 3] = 0.0
    d[2][ns - 1, 3] = 1.0  # a pure species, and an absent one
    d[2][0, 5] = 0.0
    for prec in ("fp64", "mixed"):
        print("[gpu-case] rates call sizes", name, prec, flush=True)
        w = kx.production_rates(dm, *d, precision=prec)
        assert bool(torch.isfinite(w).all())
        for m in (1, 512, 513, 1025, 2048, 2049, 3500, 4096, 4097, 5121, 6144, 6145, 16384, 16385,
                  16384 + 2048, 16384 + 4096, n - 1):
            assert torch.equal(kx.production_rates(dm, *_first(d, m), precision=prec), w[:, :m]), m
        for sizes in ((1, 700, 0, 65), (2048, 2049), (6143, 1)):
            sets = [_first(d, m) for m in sizes]
            for out, m in zip(kx.batch_noalloc(dm, sets, precision=prec), sizes):
                assert torch.equal(out[0], w[:, :m]), m
    dm.close()


@pytest.mark.parametrize("name", list(RATES) + list(ENDS))
def test_small_calls_against_the_oracle(name):
    """One point per workgroup (the oracle checks the first 70 of 700 points)."""
    from oracle import oracle as O
    from paper_2411_02640_amd import kx

    from . import parity as PM
    mech = {**RATES, **ENDS}[name]()
    T, p, Y = I.make_states(mech["n_species"], I.StateSpec(700, seed=92, p_atm_range=(1.0, 40.0),
                                                           dirichlet_alpha=0.3))
    ref, s = O.OracleMech(mech).production_rates(T[:70], p[:70], np.ascontiguousarray(Y[:, :70]))
    dm = kx.Mechanism(mech, 0)
    d = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (T, p, Y)]
    print("[gpu-case] rates small calls", name, flush=True)
    r = PM.wdot_report(kx.production_rates(dm, *d)[:, :70].cpu().numpy(), ref, s)
    assert r["ok"], r
    w = kx.production_rates(dm, *d, precision="mixed")[:, :70].cpu().numpy()
    assert np.all(np.abs(w - ref) <= 1e-5 * s + 1e-300)
    dm.close()


TRANSPORT = {"48sp": dict(ns=48),   # three row blocks: 512 or 256 threads (mixed)
             "144sp": dict(ns=144), "200sp": dict(ns=200), "256sp": dict(ns=256),
             # the vector-ALU forms: 5, 9, 14, 9 and 9 waves, an odd last species
             "17sp-Dkj": dict(ns=17, diff_fit_kind=0), "23sp": dict(ns=23),
             "33sp-Dkj": dict(ns=33, diff_fit_kind=0), "53sp-Dkj": dict(ns=53, diff_fit_kind=0),
             "65sp-Dkj": dict(ns=65, diff_fit_kind=0), "129sp-Dkj": dict(ns=129, diff_fit_kind=0)}


@pytest.mark.parametrize("name", list(TRANSPORT))
def test_transport(name):
    """The matrix-core tile shapes that a call's size selects (mixed path), the
    vector-ALU kernel's form for very many points, and the batched calls of the same
    sizes."""
    from paper_2411_02640_amd import kx
    kw = dict(TRANSPORT[name])
    ns = kw.pop("ns")
    dm = kx.Mechanism(I.make_mechanism(I.MechSpec(ns, 5 * ns, ns // 2, 0, 2, seed=9000 + ns, **kw)), 0)
    vector = "diff_fit_kind" in kw or ns < 24
    n = 900001 if vector and ns <= 53 else 450001 if vector else 160001 if ns <= 64 else 50001
    base = _states(ns, 1024)
    d = [t.repeat(*([1] * (t.dim() - 1)), n // 1024 + 1)[..., :n].contiguous() for t in base]
    d[2][:, 3] = 0.0
    d[2][ns - 1, 3] = 1.0
    for prec in ("fp64", "mixed"):
        print("[gpu-case] transport call sizes", name, prec, flush=True)
        out = kx.transport(dm, *d, precision=prec)
        for m in (1, 65, 4096, 4097, 8193, 10241, 16385, n // 2, n - 1):
            for a, b in zip(kx.transport(dm, *_first(d, m), precision=prec), out):
                assert torch.equal(a, b[..., :m]), m
        for sizes in ((1, 65), (4097,), (5000, 5000), (16384, 30000), (63, n - 1)):
            sets = [_first(d, m) for m in sizes]
            for got, m in zip(kx.batch_noalloc(dm, sets, transport=True, precision=prec), sizes):
                for a, b in zip(got[1:], out):
                    assert torch.equal(a, b[..., :m]), (sizes, m)
    dm.close()


@pytest.mark.parametrize("name", list(QSS))
def test_qss_forms_against_the_oracle(name):
    """C_Q and wdot at sampled points of a call with several tiles to a CU, of one with a
    CU to each tile and of one with a point per workgroup; the QSS rows of Y hold NaN."""
    from paper_2411_02640_amd import kx

    from . import test_gpu_qss as Q
    mech = QSS[name]()
    ns, n = mech["n_species"], 16384 + 70
    T, p, Y = I.make_states(ns, I.StateSpec(n, seed=94, p_atm_range=(0.2, 40.0), dirichlet_alpha=0.3))
    hidden = Y.copy()
    hidden[np.flatnonzero(mech["qss"])] = np.nan
    dm = kx.Mechanism(mech, 0)
    for m in (n, 5000, 700):
        print("[gpu-case] qss forms", name, m, flush=True)
        w, C = Q.run_qss(kx, dm, T[:m], p[:m], np.ascontiguousarray(hidden[:, :m]))
        i = np.unique(np.concatenate([np.arange(0, m, max(1, m // 90)), [63, 64, m - 1]]))
        Q.compare(mech, w[:, i], C[:, i], T[i], p[i], np.ascontiguousarray(Y[:, i]), name)
    dm.close()


@pytest.mark.parametrize("ns", [24, 57])
def test_served_rates(ns):
    """The work-stealing and the one-tile-per-workgroup batches with 8 and 16 waves a
    tile against direct calls."""
    from paper_2411_02640_amd import kx
    dm = kx.Mechanism(_mech(ns), 0)
    d = _states(ns, 140000)
    srv = kx.Server(0, hbm_budget=1 << 30, max_slots=16)
    for sizes in ((1, 65, 700, 3000), (140000,)):
        for prec in ("fp64", "mixed"):
            print("[gpu-case] served rates", ns, sizes, prec, flush=True)
            sets = [_first(d, m) for m in sizes]
            torch.cuda.synchronize()
            tickets = [srv.submit(dm, *s, precision=prec) for s in sets]
            for t, s in zip(tickets, sets):
                assert srv.wait(t)["state"] == "done"
                assert torch.equal(srv.outputs(t)[0], kx.production_rates(dm, *s, precision=prec))
                srv.release(t)
    srv.close()
    dm.close()
