"""The tuner times whole attempts in the grid's own stage buffers: neither a
state nor the slope that a run left may notice, before a first state or between
two halves of a run.  Bars: bitwise, every run on one and the same plan."""
import numpy as np
import pytest

from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("n,nsub", [((24, 17, 1), 1), ((16, 12, 9), 1), ((20, 9, 3), 2)])
def test_tuning_leaves_runs_alone(n, nsub, prec):
    p = inputs.base_params(n, (2e-9, 2e-9, 2e-9), nsub=nsub)
    p.update(Ms=[9e5] * nsub, A11=[1.3e-11] * nsub, alpha=[0.1] * nsub, demag=True)
    m = inputs.smoothed_random_unit(inputs.rng(94), nsub, n, sigma=1.5)
    dt = 2e-14

    def end(g):
        out = g.get_state()[0]
        g.close()
        return out

    a = mmp.Grid(p, prec)
    pl = a.plan()
    a.set_state(m)
    a.run_fixed(dt, 8)
    ref = end(a)
    assert np.isfinite(ref).all()
    b = mmp.Grid(p, prec)
    b.autotune()
    b.set_plan(**pl)
    b.set_state(m)
    b.run_fixed(dt, 8)
    assert np.array_equal(end(b), ref)
    c = mmp.Grid(p, prec)
    c.set_plan(**pl)
    c.set_state(m)
    c.run_fixed(dt, 4)
    c.autotune()
    c.set_plan(**pl)
    c.run_fixed(dt, 4)
    assert np.array_equal(end(c), ref)
