"""The two ways the strain and force kernels deal cells to blocks: 64x4 tiles,
and 256 consecutive cells where tiles would leave lanes idle (tracks narrower
than a tile, planes of few rows).  Fixed steps and energies against the oracle:
FP64 <= 1e-12 of the largest value, m absolute.
"""
import numpy as np
import pytest

from oracle.system import Problem
from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu


# (more than 256 tiles each; the last two keep their tiles)
@pytest.mark.parametrize("n", [(3, 150, 9), (70, 9, 60), (1, 1100, 1), (17, 33, 32), (130, 2, 90),
                               (5, 1, 300), (64, 8, 150), (20, 9, 3)])
@pytest.mark.parametrize("beta", [0.0, 5e-14])
def test_linear_blocks(n, beta):
    p, _ = inputs.config_c4_crop()
    p = dict(p, n=n, elastic=dict(p["elastic"], rayleigh=beta))
    nx, ny, nz = n
    r = inputs.rng(121)
    m = inputs.smoothed_random_unit(r, 1, n, sigma=1.5)
    m = np.concatenate([m, -m])
    u = 1e-12 * r.standard_normal((3, nz, ny, nx))
    v = 1e-3 * r.standard_normal((3, nz, ny, nx))
    P = Problem(p)
    g = mmp.Grid(p, mmp.FP64)
    g.set_state(m, u, v)
    _, e = g.eval_heff(mmp.T_ALL, want_b=False)
    ref = P.energies(m, u, v)
    scale = sum(abs(x) for x in ref.values())
    for k in mmp.ENERGY_NAMES:
        assert abs(e[k] - ref[k]) <= 1e-12 * scale, k
    assert abs(e["elastic"] - ref["elastic"]) <= 1e-12 * abs(ref["elastic"])
    g.run_fixed(1e-15, 3)
    mg, ug, vg, _, _ = g.get_state()
    g.close()
    y, _ = P.run_fixed([m, u, v], 0.0, 1e-15, 3)
    assert np.abs(mg - y[0]).max() < 1e-12
    assert np.abs(ug - y[1]).max() <= 1e-12 * np.abs(y[1]).max()
    assert np.abs(vg - y[2]).max() <= 1e-12 * np.abs(y[2]).max()


# one displacement that is not finite, where the schemes of the axis leave it
# out: two cells from a face, one cell from it, on it, and on axes of one cell
@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("n,at", [((9, 7, 6), (2, 4, 3)), ((9, 7, 6), (8, 5, 1)),
                                  ((9, 7, 6), (4, 0, 5)), ((1, 8, 1), (0, 3, 0)),
                                  ((6, 1, 5), (2, 0, 2)), ((2, 3, 4), (1, 1, 2)),
                                  ((3, 150, 9), (1, 75, 4))])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite_displacement_reaches_its_scheme_only(n, at, bad, prec):
    p, _ = inputs.config_c4_crop()
    p = dict(p, n=n)
    nx, ny, nz = n
    r = inputs.rng(122)
    m = inputs.random_unit(r, 1, n)
    m = np.concatenate([m, -m])
    u = 1e-12 * r.standard_normal((3, nz, ny, nx))
    u[:, at[2], at[1], at[0]] = bad
    v = np.zeros_like(u)
    g = mmp.Grid(p, prec)
    g.set_state(m, u, v)
    b, _ = g.eval_heff(mmp.T_MEL)
    g.close()
    with np.errstate(invalid="ignore"):
        P = Problem(p)
        ref = np.stack([P.term_field("mel", m, s, u) for s in range(2)])
    assert np.array_equal(np.isfinite(b), np.isfinite(ref))
