"""Which demag passes a plan runs, and the passes behind each choice.

A 3-D grid of up to 8 layers whose y lines fit a block's LDS runs y and z as
one pass unless its plan asks for two: by xy_cols = 0, or by launch shapes that
only the separate passes have.  The kernel classes of the profile tell the two
apart.  Fields against the oracle: max |dB| over max |B_ref|, FP64 <= 1e-12,
FP32 <= 2e-6 on the FP32-rounded state.
"""
import itertools

import numpy as np
import pytest

from oracle.system import Problem
from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu

TOL = {mmp.FP64: 1e-12, mmp.FP32: 2e-6}


_ref = {}


def _case(n, prec, seed=101):
    p = inputs.base_params(n, (2e-9, 3e-9, 2.5e-9))
    p.update(Ms=[9e5], A11=[1.3e-11], alpha=[0.1], demag=True)
    m = inputs.smoothed_random_unit(inputs.rng(seed), 1, n, sigma=1.5)
    if prec == mmp.FP32:
        m = np.asarray(m, np.float32).astype(np.float64)
    g = mmp.Grid(p, prec)
    g.set_state(m)
    if (n, prec) not in _ref:
        _ref[n, prec] = Problem(p).demag_field(m)
    return g, _ref[n, prec]


def _run(g, ref):
    """(y and z are one pass, error) of one field."""
    g.prof_enable(True)
    g.prof_reset()
    b = g.eval_heff(mmp.T_DEMAG)[0]
    g.synchronize()
    launches = {k: v[1] for k, v in g.prof_read().items()}
    g.prof_enable(False)
    assert launches["fftz_mul"] == 1 and launches["ffty_fwd"] == launches["ffty_inv"]
    return launches["ffty_fwd"] == 0, np.abs(b - ref).max() / np.abs(ref).max()


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("n", [(24, 16, 8), (37, 23, 5)])
def test_route_follows_the_plan(n, prec):
    g, ref = _case(n, prec)

    def route(fused, **kw):
        pl = g.set_plan(**kw) if kw else g.plan()
        one, err = _run(g, ref)
        assert one == fused and (pl["xy_cols"] != 0) == fused, (kw, pl)
        assert err <= TOL[prec], (kw, err)
        # the same plan says the same to a grid that has never held another
        h, _ = _case(n, prec)
        assert h.set_plan(**pl) == pl
        assert _run(h, ref)[0] == fused, (kw, pl)
        h.close()
        return pl

    pl = route(True)
    route(False, xy_cols=0)
    assert route(True, xy_cols=1) == dict(pl, xy_cols=1)
    route(True, **pl)
    y = [2 if v == 1 else v // 2 for v in pl["y_lines"]]
    assert route(False, y_lines=y)["y_lines"] == y
    route(False, x_rows=[2, 4])
    route(True, **pl)
    route(True, field_zplanes=1, x_rows=[2, 4])
    route(False, z_cols=max(1, pl["z_cols"] // 2))
    route(True, **pl)
    route(True, lds_axes=7, y_lines=[1, 1], z_cols=1)     # of the LDS kernels
    route(False, xy_cols=0)
    route(True, **pl)
    route(True, pad=[80, 48, 16])
    if g.plan()["kinds"] & 4:
        route(False, z_threads=64)
    route(True, **pl)
    # a refused plan changes nothing
    with pytest.raises(mmp.MMPError):
        g.set_plan(xy_cols=0, y_lines=[128, 1])
    assert g.plan() == pl and _run(g, ref)[0]
    g.close()


# pads of 4, 8 and 16, one of them over a y pad that leaves part of a block empty
@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("n,pad", [((8, 16, 2), [16, 32, 4]), ((9, 12, 4), [20, 24, 8]),
                                   ((8, 16, 8), [16, 32, 16]), ((37, 23, 5), [80, 50, 16])])
def test_register_z_shapes(n, pad, prec):
    g, ref = _case(n, prec)
    tried = set()
    for q, w, t, k in itertools.product((1, 2, 4), (1, 2, 4), (64, 128, 256), (0, 1)):
        try:
            pl = g.set_plan(pad=pad, xy_cols=0, z_lanes=q, z_waves=w, z_threads=t, z_mode=k)
        except mmp.MMPError as e:
            assert e.code == -1
            continue
        assert pl["kinds"] & 4 and pl["z_lanes"] == q
        one, err = _run(g, ref)
        assert not one and err <= TOL[prec], (q, w, t, k, err)
        tried.add((q, w, k))
    g.close()
    assert {q for q, _, _ in tried} >= {1, 2} and {k for _, _, k in tried} == (
        {0, 1} if prec == mmp.FP32 else {0}), tried


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
def test_separate_lds_passes(prec):
    """y lines and z columns of the mixed-radix kernels, layers up to 8."""
    g, ref = _case((37, 23, 5), prec)
    for lines, cols in itertools.product(((1, 4), (8, 2), (4, 16)), (1, 4, 16, 32)):
        pl = g.set_plan(xy_cols=0, y_lines=list(lines), z_cols=cols)
        assert pl["kinds"] == 0
        one, err = _run(g, ref)
        assert not one and err <= TOL[prec], (lines, cols, err)
    g.close()


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
def test_fused_limit_is_met(prec):
    """Eight layers of a y length that fills the LDS with one pass over y and
    z, of a longer one with two."""
    g, ref = _case((4, 6, 8), prec, 61)
    per = 131072 // (24 * (8 if prec == mmp.FP32 else 16))
    seen = set()
    for L in range(int(0.7 * per) // 2 * 2, int(1.3 * per), 2):
        q = L
        for f in (2, 3, 5, 7):
            while q % f == 0:
                q //= f
        if q != 1:
            continue
        g.set_plan(pad=[8, L, 16], x_rows=[2, 2], y_lines=[1, 1], lds_axes=6)
        one, err = _run(g, ref)
        assert err <= TOL[prec], L
        seen.add(one)
    g.close()
    assert seen == {True, False}


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
def test_tuner_keeps_its_choice(prec):
    g, ref = _case((24, 200, 8), prec)
    pl = g.autotune()
    one, err = _run(g, ref)
    # (of the pads the tuner may pick, one is too long for a pass over both)
    assert err <= TOL[prec] and (pl["xy_cols"] != 0 or not one)
    h, _ = _case((24, 200, 8), prec)
    assert h.plan() == pl and _run(h, ref)[0] == one
    assert h.set_plan(**pl)["xy_cols"] == pl["xy_cols"] and _run(h, ref)[0] == one
    g.close()
    h.close()


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
def test_batch_of_every_route(prec):
    """One batch of 2-D grids, of fused ones with short and long z columns and
    of ones whose y and z are separate passes: each result bitwise as served
    alone, and as the grid run alone on the LDS kernels (FP64 the same steps and
    <m> to 1e-12, energy to 1e-12 of its terms; FP32 the trajectory bar 1e-4)."""
    sizes = [((12, 10, 1), True), ((9, 11, 3), True), ((10, 8, 7), True), ((11, 9, 8), True),
             ((8, 10, 12), False), ((5, 600, 8), False)]
    reqs = []
    for i, (n, _) in enumerate(sizes):
        p = inputs.base_params(n, (2e-9, 2e-9, 2e-9))
        p.update(Ms=[1.0e6], A11=[1.4e-11], Ku1=[4e5], alpha=[0.1], B_ext=(0.0, 0.0, 0.05),
                 demag=True)
        reqs.append((p, inputs.smoothed_random_unit(inputs.rng(141 + i), 1, n, sigma=1.5)))
    t = 1e-11

    def serve(rs):
        srv = mmp.Server(hbm_budget=8 << 30, max_active=8, precision=prec)
        out = [srv.wait(k) for k in [srv.submit(p, m, t) for p, m in rs]]
        srv.close()
        assert all(r.status == 0 for r in out)
        return out

    mixed = serve(reqs)
    assert max(r.t_admit for r in mixed) < min(r.t_done for r in mixed)
    for (p, m), (n, fused), r in zip(reqs, sizes, mixed):
        alone = serve([(p, m)])[0]
        assert (r.steps, r.rejects, r.energy) == (alone.steps, alone.rejects, alone.energy), n
        assert np.array_equal(np.array(r.m_avg), np.array(alone.m_avg)), n
        g = mmp.Grid(p, prec)
        g.set_plan(lds_axes=7)
        g.set_state(m)
        if n[2] > 1:
            assert _run(g, 1.0)[0] == fused, n
        info, _, _ = g.run(t)
        avg = g.get_state()[0].mean(axis=(0, 2, 3, 4))
        _, e = g.eval_heff(mmp.T_ALL, want_b=False)
        g.close()
        bar = 1e-12 if prec == mmp.FP64 else 1e-4
        assert prec == mmp.FP32 or (r.steps, r.rejects) == (info.steps, info.rejects), n
        assert np.abs(np.array([r.m_avg[0][c] for c in range(3)]) - avg).max() <= bar, n
        assert abs(r.energy - sum(e.values())) <= bar * sum(abs(v) for v in e.values()), n
