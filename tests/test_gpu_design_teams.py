"""Table design with one to four teams of waves per workgroup, which share the check of the
designed filters: numbers of entries that take each number of teams on 256 CUs, with a last
workgroup that is not full, one and two entries per team, check grids of odd sizes, against
the FP64 oracle.  Tolerance as in the tests of the tiling: four times the oracle's change
under 1-ulp changes of dx and dz, plus 1e-10 of the table's largest value."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,ntaps,nk,ngrid,ncheck", [
    (1, 19, 259, 40, 97), (1, 25, 601, 33, 131), (1, 35, 1021, 40, 1025), (1, 35, 1603, 70, 515), (1, 23, 2041, 64, 64),
    (1, 45, 300, 50, 129), (1, 45, 1031, 50, 127), (1, 63, 345, 70, 193),
    (2, 9, 700, 9, 17), (2, 9, 1801, 9, 16), (2, 11, 1031, 11, 13), (2, 11, 300, 64, 15)])
def test_design_teams(dims, ntaps, nk, ngrid, ncheck):
    make = synth.table_for if dims == 1 else synth.table2d_for
    desc = make(ntaps, nk, 5.0, 40.0, 750.0, 2000.0, 10.0, 10.0, ngrid=ngrid, ncheck=ncheck, nreweight=2)
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
