"""Table design at the edges of its kernel's tiling, against the FP64 oracle: odd and
even coefficient counts at the ends of each padded size, one and two entries per
workgroup with an odd table end, grids that end inside a chunk of 64 points.

Tolerance: both sides evaluate the same formulas in the same order; what differs is
the last bit of cos, sin, exp and sqrt, which the fit amplifies by its own
conditioning.  So four times the oracle's change under 1-ulp changes of dx and dz,
plus 1e-10 of the table's largest value."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import dev

pytestmark = pytest.mark.gpu

CASES = [
    # dims, ntaps, nk, ngrid, ncheck
    (1, 1, 2, 8, 8), (1, 3, 1025, 31, 77), (1, 23, 5, 64, 9), (1, 25, 1026, 65, 64),
    (1, 35, 3, 127, 100), (1, 37, 514, 128, 33), (1, 47, 515, 96, 65), (1, 49, 3, 200, 33),
    (1, 63, 343, 100, 64), (1, 63, 2, 2048, 8),
    (2, 1, 2, 8, 9), (2, 7, 4, 33, 30), (2, 9, 1025, 17, 32), (2, 11, 513, 13, 16), (2, 11, 3, 64, 20),
]


@pytest.mark.parametrize("dims,ntaps,nk,ngrid,ncheck", CASES)
def test_design_tiling_edges(dims, ntaps, nk, ngrid, ncheck):
    make = synth.table_for if dims == 1 else synth.table2d_for
    desc = make(ntaps, nk, 5.0, 40.0, 750.0, 2000.0, 10.0, 10.0, ngrid=ngrid, ncheck=ncheck, nreweight=3)
    design = oracle.design_table if dims == 1 else oracle.design_table_2d
    ot, omg, ope = design(desc)[:3]
    near = design(dataclasses.replace(desc, dx=np.nextafter(desc.dx, np.inf), dz=np.nextafter(desc.dz, np.inf)))[0]
    scale = np.abs(ot).max()
    tol = 1e-10 + 4.0 * np.abs(near - ot).max() / scale
    g = (mig.design_table if dims == 1 else mig.design_table_2d)(desc, dev())
    err = np.abs(g["tab64"].cpu().numpy() - ot).max() / scale
    print("dims %d N %d nk %d grid %d: %.2e (tol %.2e)" % (dims, ntaps, nk, ngrid, err, tol), flush=True)
    assert err <= tol
    assert np.abs(g["maxgain"].cpu().numpy() - omg).max() <= 10 * tol
    assert np.abs(g["passerr"].cpu().numpy() - ope).max() <= 10 * tol
    assert torch.equal(g["tab32"], g["tab64"].to(torch.complex64))
