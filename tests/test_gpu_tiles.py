"""Edges of the FP64 matrix-product tiles: the stray field (16x16 targets, 4
sources at a time) and the kernel spectrum (64x64 outputs, sums of 16), against
the oracle.  Bars as in the other comparisons of these results: FP64 fields of
near-cubic cells 1e-12 of the largest value.
"""
import numpy as np
import pytest

from oracle import stray
from oracle.system import Problem
from paper_2411_18194_amd import inputs, mmp

pytestmark = pytest.mark.gpu


def _case(n, nsub, seed, cell=(2e-9, 2.2e-9, 1.9e-9)):
    p = inputs.base_params(n, cell, nsub=nsub)
    p.update(Ms=[9e5, 5e5, 3e5][:nsub], A11=[1.3e-11] * nsub, alpha=[0.1] * nsub, demag=True)
    return p, inputs.smoothed_random_unit(inputs.rng(seed), nsub, n, sigma=1.5)


@pytest.mark.parametrize("n,nsub", [((16, 16, 1), 1), ((17, 15, 2), 1), ((33, 1, 1), 1),
                                    ((1, 40, 3), 1), ((3, 5, 1), 1), ((1, 1, 1), 1),
                                    ((48, 50, 1), 1), ((21, 18, 2), 2), ((18, 21, 1), 3)])
def test_stray_tiles(n, nsub):
    p, m = _case(n, nsub, 91)
    g = mmp.Grid(p, mmp.FP64)
    g.set_state(m)
    M = sum(p["Ms"][s] * m[s] for s in range(nsub))
    for height in (0.95e-9, 7e-9):
        b = g.stray_field(height)
        ref = stray.stray_field(M, p["cell"], height)
        assert np.abs(b - ref).max() <= 1e-12 * np.abs(ref).max(), height
    g.close()


@pytest.mark.parametrize("n,pbc", [((64, 33, 1), (0, 0, 0)), ((65, 31, 2), (0, 0, 0)),
                                   ((17, 130, 1), (0, 0, 0)), ((5, 4, 17), (0, 0, 0)),
                                   ((70, 48, 1), (1, 2, 0))])
def test_spectrum_tiles(n, pbc):
    p, m = _case(n, 1, 92)
    p["pbc"] = pbc
    g = mmp.Grid(p, mmp.FP64)
    g.set_state(m)
    ref = Problem(p).demag_field(m)
    b, _ = g.eval_heff(mmp.T_DEMAG)
    g.close()
    assert np.abs(b - ref).max() <= 1e-12 * np.abs(ref).max()


def test_stray_tensor_in_pieces():
    """A tensor whose offsets need more threads than one launch holds: 64x64
    offsets within reach of tall cells, 4097 layers, of which the top ones are
    magnetised.  The same layers on a grid of their own give the same field."""
    torch = pytest.importorskip("torch")
    cell, top, height = (1e-9, 1e-9, 2e-9), 8, 3e-9
    m = inputs.smoothed_random_unit(inputs.rng(95), 1, (64, 64, top), sigma=1.5)
    out = []
    for nz in (4097, top):
        p = inputs.base_params((64, 64, nz), cell)
        p.update(Ms=[9e5], A11=[1.3e-11], alpha=[0.1])
        full = torch.zeros((1, 3, nz, 64, 64), dtype=torch.float64, device="cuda")
        full[:, :, nz - top:] = torch.from_numpy(m).to("cuda")
        torch.cuda.synchronize()
        g = mmp.Grid(p, mmp.FP64)
        g.set_state_device(full)
        out.append(g.stray_field(height))
        g.close()
    assert np.abs(out[0] - out[1]).max() <= 1e-12 * np.abs(out[1]).max()
