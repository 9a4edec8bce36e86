"""The mixed-radix line transforms and the fused y-z pass against the oracle.

Any even 7-smooth pad >= 2n - 1 gives the same linear convolution, so one
small grid runs on every line length the passes have (191 of them, up to
4096) along x and y, and grids of 2..8 layers run the fused pass with every
z length it is built for, at its LDS limit and just past it.  Bars as for
the other demag plans: max |dB| over max |B_ref|, FP64 <= 1e-12, FP32 <=
2e-6 on the FP32-rounded state.
"""
import numpy as np
import pytest

from oracle.system import Problem
from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu

TOL = {mmp.FP64: 1e-12, mmp.FP32: 2e-6}


def _smooth(L):
    for f in (2, 3, 5, 7):
        while L % f == 0:
            L //= f
    return L == 1


LENGTHS = [L for L in range(12, 4097, 2) if _smooth(L)]


def _case(n, prec, seed, pbc=(0, 0, 0)):
    p = inputs.base_params(n, (2e-9, 3e-9, 2.5e-9))
    p.update(Ms=[9e5], A11=[1.3e-11], alpha=[0.1], demag=True, pbc=pbc)
    m = inputs.smoothed_random_unit(inputs.rng(seed), 1, n, sigma=1.5)
    if prec == mmp.FP32:
        m = np.asarray(m, np.float32).astype(np.float64)
    g = mmp.Grid(p, prec)
    g.set_state(m)
    return g, Problem(p).demag_field(m)


def _err(g, ref):
    return np.abs(g.eval_heff(mmp.T_DEMAG)[0] - ref).max() / np.abs(ref).max()


@pytest.mark.parametrize("prec", [mmp.FP32, mmp.FP64])
@pytest.mark.parametrize("axis,pz", [("x", 4), ("y", 4), ("y", 18)])
def test_every_line_length(axis, pz, prec):
    """x lines; y lines in the fused pass (z pad 4, unless one line of the
    length fills the LDS) and on their own (z pad 18)."""
    g, ref = _case((6, 5, 2), prec, 51)
    bad = {}
    for L in LENGTHS:
        pad = [L, 12, pz] if axis == "x" else [12, L, pz]
        g.set_plan(pad=pad, x_rows=[2, 2], y_lines=[1, 1], z_cols=1, lds_axes=7)
        e = _err(g, ref)
        if not e <= TOL[prec]:
            bad[L] = e
    g.close()
    assert not bad, bad


@pytest.mark.parametrize("prec", [mmp.FP32, mmp.FP64])
@pytest.mark.parametrize("nz,pzs", [(2, (4, 6, 16)), (3, (6, 8)), (4, (8, 10)), (5, (10, 16)),
                                    (6, (12, 14)), (7, (14,)), (8, (16,))])
def test_fused_columns(nz, pzs, prec):
    """Every z length of the fused pass over an odd number of rows, alone and
    with the columns of the last block past the spectrum."""
    g, ref = _case((9, 11, nz), prec, 52 + nz)
    for pz in pzs:
        for py in (22 + 2, 32, 50):
            g.set_plan(pad=[20, py, pz], lds_axes=7)
            assert _err(g, ref) <= TOL[prec], (pz, py)
    g.close()


@pytest.mark.parametrize("prec", [mmp.FP32, mmp.FP64])
def test_fused_limit(prec):
    """A y line length whose 3 nz lines fill the LDS of a block, and the
    next one, which takes the separate y and z passes."""
    g, ref = _case((4, 6, 8), prec, 61)
    per = 131072 // (24 * (8 if prec == mmp.FP32 else 16))
    for L in [x for x in LENGTHS if 0.7 * per < x < 1.3 * per]:
        g.set_plan(pad=[8, L, 16], x_rows=[2, 2], y_lines=[1, 1], lds_axes=6)
        assert _err(g, ref) <= TOL[prec], L
    g.close()


@pytest.mark.parametrize("prec", [mmp.FP32, mmp.FP64])
@pytest.mark.parametrize("n,pbc", [((12, 10, 3), (1, 1, 0)), ((14, 9, 2), (2, 0, 0)),
                                   ((9, 18, 4), (0, 1, 0)), ((30, 14, 1), (1, 1, 0))])
def test_periodic_lines(n, pbc, prec):
    """Lines without a zero half."""
    g, ref = _case(n, prec, 71, pbc)
    g.set_plan(lds_axes=7)
    assert _err(g, ref) <= TOL[prec]
    g.close()


@pytest.mark.parametrize("prec", [mmp.FP32, mmp.FP64])
@pytest.mark.parametrize("n", [(1, 1, 1), (1, 7, 1), (7, 1, 1), (1, 1, 3), (1, 5, 2), (5, 1, 2)])
def test_single_cell_axes(n, prec):
    g, ref = _case(n, prec, 81)
    g.set_plan(lds_axes=7)
    assert _err(g, ref) <= TOL[prec]
    g.close()


# Several lanes per column in the z pass of power-of-two pads: the lanes' own
# planes all, partly or not there, on pads of 16 (too long in y for the fused
# pass), 32 and 64.
@pytest.mark.parametrize("prec", [mmp.FP64, mmp.FP32])
@pytest.mark.parametrize("n,lanes", [((6, 256, 8), 4), ((6, 250, 5), 4), ((6, 250, 7), 2),
                                     ((17, 24, 9), 4), ((9, 33, 13), 2), ((16, 20, 16), 4),
                                     ((7, 12, 17), 4), ((5, 9, 32), 4)])
def test_z_column_lanes(n, lanes, prec):
    g, ref = _case(n, prec, 93)
    pads = [1 << (2 * k - 2).bit_length() for k in n]
    pl = g.set_plan(pad=pads, z_lanes=lanes, z_waves=1)
    assert pl["z_lanes"] == lanes and pl["kinds"] & 4
    assert _err(g, ref) <= TOL[prec]
    g.close()
