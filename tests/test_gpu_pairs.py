"""The pairs of few stages with several sublattices: their field kernels hold
two and three stage slopes per cell instead of six.

Against the oracle as the other pair checks: fixed steps max |dm| <= 1e-12,
adaptive runs (whose last stage sums every slope for the error) the same
accepted and rejected steps and the final state within 1e-10 (FP64); a run
resumed from a saved state is bitwise the run it continues.
"""
import numpy as np
import pytest

from oracle.system import Problem
from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu


def _case(nsub, kind, solver):
    n = (13, 6, 3)
    p = inputs.base_params(n, (1.5e-9, 1.5e-9, 2e-9), nsub=nsub)
    p.update(Ms=[4e5, 3e5, 3.5e5][:nsub], A11=[1e-11, 8e-12, 9e-12][:nsub],
             alpha=[0.05, 0.02, 0.03][:nsub], A0=-2e-12, A12=-4e-12, latcon=0.4e-9,
             Ku1=[6e4, 5e4, 4e4][:nsub], B_ext=(0.0, 0.02, 0.05), zl_P=[0.5] * nsub,
             zl_xi=[0.1] * nsub, j=(2e11, 0.0, 0.0), solver=solver)
    if "grains" in kind:
        g = inputs.rng(111)
        ids, _ = inputs.voronoi_grains(g, n, p["cell"], 5)
        ax = g.standard_normal((5, 3))
        p.update(grain=ids, grain_axes=ax / np.linalg.norm(ax, axis=1, keepdims=True),
                 grain_exchange_scale=0.25)
    if "eq6" in kind:
        D = 1.5e-3
        p.update(bc="eq6", dmi_W=[[[0.0, D, 0.0], [-D, 0.0, 0.0], [0.0, 0.0, 0.0]]] * nsub)
    m = inputs.smoothed_random_unit(inputs.rng(112), nsub, n, sigma=1.5)
    return p, m


CASES = [(2, ""), (3, ""), (2, "grains"), (3, "grains"), (2, "eq6"), (2, "eq6 grains")]


@pytest.mark.parametrize("solver", ["heun", "bs23"])
@pytest.mark.parametrize("nsub,kind", CASES)
def test_short_pairs(nsub, kind, solver):
    p, m = _case(nsub, kind, solver)
    P = Problem(p)   # (its stepper keeps the last slope: another for the second run)
    g = mmp.Grid(p, mmp.FP64, tol=1e-5, dt0=1e-15)
    g.set_state(m)
    g.run_fixed(2e-15, 5)
    mg = g.get_state()[0]
    y, _ = P.run_fixed(P.initial_state(m), 0.0, 2e-15, 5)
    assert np.abs(mg - y[0]).max() < 1e-12
    g.set_state(m)
    info, _, _ = g.run(5e-14)
    mg = g.get_state()[0]
    g.close()
    y, _, oinfo, _ = Problem(p).run([m.copy()], 0.0, 5e-14, tol=1e-5, dt0=1e-15)
    assert info.steps > 3 and (info.steps, info.rejects) == (oinfo["steps"], oinfo["rejects"])
    assert np.abs(mg - y[0]).max() < 1e-10


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("solver", ["heun", "bs23", "dp45"])
@pytest.mark.parametrize("nsub", [2, 3])
def test_resume_is_bitwise(nsub, solver, prec):
    p, m = _case(nsub, "", solver)
    out = []
    for parts in ((12,), (5, 7)):
        for k in parts:
            g = mmp.Grid(p, prec)
            g.set_state(out_m if k == 7 else m)
            g.run_fixed(2e-15, k)
            out_m = g.get_state()[0]
            g.close()
        out.append(out_m)
    assert np.array_equal(out[0], out[1])
