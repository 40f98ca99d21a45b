"""Work splits at the sizes where they can go wrong, against the CPU FP64 oracle: tiles narrower than
their neighbours, PEs cut along z, threads with two halo points, grids smaller than one tile.  FP64
bars as in the parity tests: relative L2 <= 1e-12 per component (a ghost value carries the rounding
of its terms times at most 31)."""
import numpy as np
import pytest

from oracle import Oracle, OracleConfig
from paper_2003_10561_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2003_10561_amd import atns  # noqa: E402

TOL64 = 1e-12


def smooth_levels(n, nlev, seed, form):
    """Smooth periodic states that drift in time: (rho, m, E) or (rho, m, rho e)."""
    rng = np.random.default_rng(seed)
    x, y, z = (2 * np.pi * np.arange(m) / m for m in n)
    Z, Y, X = np.meshgrid(z, y, x, indexing="ij")
    ph = rng.uniform(0, 2 * np.pi, (5, 3))
    out = np.empty((nlev, 5) + X.shape)
    for lv in range(nlev):
        s = 0.05 * lv
        f = [np.sin(X + ph[i, 0] + s) * np.cos(Y + ph[i, 1]) + 0.5 * np.sin(Z + ph[i, 2] - s) for i in range(5)]
        rho, t = 1 + 0.1 * f[0], 1 + 0.1 * f[4]
        u = [0.3 * g for g in f[1:4]]
        out[lv, 0] = rho
        for i in range(3):
            out[lv, 1 + i] = rho * u[i]
        out[lv, 4] = rho * 2.5 * t + (0.5 * rho * sum(v * v for v in u) if form == 0 else 0)
    return out


def check(n, p, order=4, form=0, steps=2, precision="fp64", tol=TOL64, tune=None):
    nlev = 7 if order == 6 else 6
    q = smooth_levels(n, nlev, sum(n), form)
    kw = dict(n=n, p=p, dt=2e-3, mu_ref=0.02, max_delay=3, order=order, form=form)
    g = atns.Sim(atns.Config(precision=precision, **kw))
    o = Oracle(OracleConfig(**kw))
    g.init_field(q, nlev)
    o.init_field(q, nlev)
    tab = np.random.default_rng(sum(p)).integers(0, 4, (nlev + steps, p[0] * p[1] * p[2], 6)).astype(np.int8)
    tab[:nlev - 1] = 0
    g.set_delay_schedule(atns.EXPLICIT, table=tab)
    o.set_schedule(atns.EXPLICIT, table=tab)
    if tune:
        g.set_stage_tuning(*tune)

    def same(a, b, what):
        err = max(float(np.linalg.norm(a[c] - b[c]) / np.linalg.norm(b[c])) for c in range(5))
        print(f"case n={n} p={p} order={order} form={form} {precision} {what}: rel-L2 {err:.2e}", flush=True)
        assert err <= tol, (what, err)

    if precision == "fp64":
        same(g.rhs().cpu().numpy(), o.rhs(), "rhs")
    g.rk_step(steps)
    o.rk_step(steps)
    same(g.get_field(), o.field(), "fields")
    gs, os_ = g.stats(), o.stats()
    for k in ("mass", "energy", "mass_rk", "K", "eps", "enstrophy", "Mt", "umax"):
        assert abs(gs[k] - os_[k]) <= max(tol, 1e-12) * abs(os_[k]), (k, gs[k], os_[k])
    g.close()


# edges: 6 (the smallest PE: 36 columns, two halo points a thread), 7 (two halo points a thread), 40 along z
# (cut into chunks of 8), 21 x 25 (rows of 9 + 9 + 7; z chunks of 9 + 9 + 9 + 6), 33 x 21 (one column of
# tiles 33 wide, rows of 7), 65 (columns of 22 + 22 + 21)
@pytest.mark.parametrize("n,p", [((6, 6, 6), (1, 1, 1)), ((12, 14, 40), (2, 2, 1)), ((42, 25, 33), (2, 1, 1)),
                                 ((33, 21, 24), (1, 1, 3)), ((130, 9, 12), (2, 1, 1))])
def test_order6_tiles(n, p):
    check(n, p, order=6)


# the paper's form: edges 5 (the smallest PE), 9 x 11 (99 of 256 threads: a point per thread), 12 x 11
# (132: a partial tile), 17 x 33 (9 + 8 by 11 + 11 + 11: 99 again, a point per thread), 33 x 16 (three
# equal tiles, chunks of 8 planes that start inside z-PEs of 20), grids of fewer columns than a brick
@pytest.mark.parametrize("n,p", [((10, 5, 15), (2, 1, 3)), ((18, 22, 10), (2, 2, 1)), ((12, 22, 30), (1, 2, 2)),
                                 ((34, 33, 18), (2, 1, 3)), ((66, 16, 40), (2, 1, 2))])
def test_paper_form_tiles(n, p):
    check(n, p, form=1)


def test_paper_form_tiles_fp32():
    check((34, 30, 36), (2, 2, 3), form=1, precision="fp32", tol=2e-6)


@pytest.mark.parametrize("n,prec", [((1024, 8, 16), "fp64"), ((8, 1024, 32), "fp64"), ((64, 16, 1024), "fp64"),
                                    ((256, 128, 8), "fp32"), ((16, 256, 128), "fp64"), ((8, 8, 512), "fp32"),
                                    ((32, 512, 8), "fp64")])
def test_diagnostics_line_lengths(n, prec):
    """Every length of a transformed line (one to four stages, the last of radix 8, 4 or 2) in x, y and
    z, fewer columns than a tile and shells beyond the last; bars as in test_gpu_diag.py."""
    from oracle.diagnostics import diagnostics as oracle_diagnostics
    from tests.test_gpu_diag import cfg_pair, check
    q = smooth_levels(n, 1, 3, 0)[0]
    q[:, ::3] *= 1.01  # (energy beyond the lowest shells)
    dq = torch.from_numpy(q).to("cuda", torch.float32 if prec == "fp32" else torch.float64).contiguous()
    nshell, nb = max(n) // 3, 20
    gc, oc = cfg_pair(n, 4 if n[0] > 16 else 6, prec)
    got = atns.field_diagnostics(gc, dq.data_ptr(), nshell, nb, 6.0, 6.0)
    check(got, oracle_diagnostics(oc, dq.double().cpu().numpy(), nshell, nb, 6.0, 6.0), nb, 6.0, 6.0, f"{n} {prec}")


@pytest.mark.parametrize("prec,shape", [("fp32", (1, 64)), ("fp64", (5, 64))])
def test_serve_default_shape(prec, shape):
    """The z chunk that the server derives from the trace never changes a field: every final state of
    a mixed burst equals that of one long chunk, bit for bit."""
    reqs = []
    for i, (n, p) in enumerate(((16, 2), (48, 3), (32, 2), (64, 2), (40, 4), (16, 1))):
        q = smooth_levels((n,) * 3, 1, 40 + i, 0)[0]
        reqs.append(dict(arrival_s=0.0, n=n, p=p, steps=5 + i, mode=(atns.CAA, atns.SAA, atns.SYNC)[i % 3], L=1 + i % 2,
                         seed=i, dt=0.2 * 2 * np.pi / n / 2.0, mu_ref=0.01, q0=q, q_final=np.empty_like(q)))
    for r in reqs:
        r["L"] = 0 if r["mode"] == atns.SYNC else r["L"]
    got = {}
    for k in ("default", "long"):
        kw = {} if k == "default" else dict(tile=shape[0], zchunk=shape[1])
        res, _ = atns.serve(reqs, precision=prec, max_active=4, **kw)
        assert [o["status"] for o in res] == [0] * len(reqs)
        got[k] = [r["q_final"].copy() for r in reqs]
    for i, (a, b) in enumerate(zip(got["default"], got["long"])):
        assert np.isfinite(a).all() and np.array_equal(a, b), i


# FP32 marches with two alternating flux planes and one barrier a plane, FP64 with one plane: edges 6 and
# 6 x 7 (two halo points a thread), 21 x 25 (rows of 9 + 9 + 7, z chunks of 9 + 9 + 9 + 6), 65 x 9 (columns
# of 22 + 22 + 21), 37 x 19 (19 + 18 by 10 + 9), 59 x 13 (30 + 29 by 7 + 6, two halo points a thread).
# FP32 bar as in test_gpu_order6.py (a ghost value carries the rounding of its terms, 6e-8, times at most
# 200, and enters a field through dt / h < 0.05: 6e-7)
@pytest.mark.parametrize("n,p", [((6, 6, 6), (1, 1, 1)), ((12, 14, 40), (2, 2, 1)), ((42, 25, 33), (2, 1, 1)),
                                 ((130, 9, 12), (2, 1, 1)), ((37, 19, 18), (1, 1, 2)), ((59, 13, 17), (1, 1, 1))])
@pytest.mark.parametrize("precision,tol", [("fp32", 2e-6), ("fp64", TOL64)])
def test_order6_narrower_tiles(n, p, precision, tol):
    check(n, p, order=6, precision=precision, tol=tol)


# edges 30 x 25 (15 + 15 by 13 + 12), 17 x 15 (9 + 8 by 15), 15 x 17 (15 by 9 + 8)
@pytest.mark.parametrize("n,p", [((60, 50, 20), (2, 2, 2)), ((34, 30, 20), (2, 2, 2)), ((30, 34, 18), (2, 2, 3))])
@pytest.mark.parametrize("precision,tol", [("fp64", TOL64), ("fp32", 2e-6)])
def test_paper_form_narrower_tiles(n, p, precision, tol):
    check(n, p, form=1, precision=precision, tol=tol)


@pytest.mark.parametrize("precision,tol", [("fp64", TOL64), ("fp32", 2e-6)])
def test_paper_form_long_marches(precision, tol):
    """256 tiles of 16 x 8 on 130 planes march 32 planes at a time (a smaller grid takes chunks of 8) over
    z-PEs of 5: up to eight of them in a chunk, which starts inside one, with random delays on every
    face of every one."""
    check((256, 128, 130), (16, 16, 26), form=1, steps=1, precision=precision, tol=tol)


@pytest.mark.parametrize("edge", [(10, 10, 10), (9, 11, 5)])
def test_paper_form_ab2_on_small_pes(edge):
    """Adams-Bashforth steps, then Runge-Kutta ones, then Adams-Bashforth again where a point takes a
    thread (10 x 10 and 9 x 11 points fill less than half of a tile)."""
    p = (2, 2, 2)
    n = tuple(2 * e for e in edge)
    q = smooth_levels(n, 6, 71, 1)
    kw = dict(n=n, p=p, dt=2e-3, mu_ref=0.02, max_delay=3, form=1)
    g, o = atns.Sim(atns.Config(precision="fp64", **kw)), Oracle(OracleConfig(**kw))
    tab = np.random.default_rng(72).integers(0, 4, (14, 8, 6)).astype(np.int8)
    g.init_field(q, 6)
    o.init_field(q, 6)
    tab[:5] = 0
    g.set_delay_schedule(atns.EXPLICIT, table=tab)
    o.set_schedule(atns.EXPLICIT, table=tab)
    for s in (g, o):
        s.ab2_step(3)
        s.rk_step(2)
        s.ab2_step(2)
    a, b = g.get_field(), o.field()
    err = max(float(np.linalg.norm(a[c] - b[c]) / np.linalg.norm(b[c])) for c in range(5))
    print(f"case n={n} p={p} form=1 ab2: rel-L2 {err:.2e}", flush=True)
    assert err <= TOL64
    gs, os_ = g.stats(), o.stats()
    for k in ("mass", "energy", "mass_rk", "energy_rk", "K", "eps", "enstrophy"):
        assert abs(gs[k] - os_[k]) <= TOL64 * abs(os_[k]), (k, gs[k], os_[k])
    g.close()


@pytest.mark.parametrize("n,p", [((16, 16, 16), (1, 1, 1)), ((40, 24, 4), (1, 3, 1)), ((33, 20, 57), (1, 1, 3)),
                                 ((72, 60, 40), (2, 2, 2)), ((64, 96, 80), (1, 3, 5)), ((8, 8, 200), (2, 2, 1))])
def test_default_shapes(n, p):
    """The shapes that a run takes by itself, for its synchronous and its delayed stages, against the
    oracle in FP64, and against one long chunk of 32 x 8 tiles bit for bit in FP32."""
    check(n, p)
    q = smooth_levels(n, 4, 5, 0)
    field = []
    for shape in (None, (1, 64, 1, 64)):
        s = atns.Sim(atns.Config(n=n, p=p, dt=2e-3, mu_ref=0.02, max_delay=1, precision="fp32"))
        if shape:
            s.set_stage_tuning(*shape)
        print(f"case default shapes n={n} p={p} fp32: {s.get_stage_tuning()}", flush=True)
        s.init_field(q, 4)
        s.set_delay_schedule(atns.SAA, L=1, seed=9, n_steps=12)
        s.rk_step(4)
        field.append(s.get_field())
        s.close()
    assert np.isfinite(field[0]).all() and np.array_equal(field[0], field[1])
