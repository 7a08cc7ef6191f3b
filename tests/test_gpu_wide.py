"""Depth stepping of wide sections and long filters at the edges of its runs of outputs
(two and four per thread, one to three runs), and image rows formed after the launch,
against the FP64 oracle.  Tolerance: relative L2 1e-5 after a few steps (FP32 taps and
arithmetic: about 1e-7 per operation, 2 N operations per output and step)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import data64, dev, rel_l2, upload

pytestmark = pytest.mark.gpu


def _check(sec, nsteps):
    tab = mig.design_table(sec.desc, dev())
    t = upload(sec)
    vel = t["vel"][:nsteps].contiguous()
    plane, rows = mig.extrapolate(t["data"], vel, t["omega"], tab["tab32"], sec.desc, nsteps)
    ot = tab["tab64"].cpu().numpy()
    ref_plane, ref_rows = oracle.extrapolate(sec.desc, ot, sec.omega, sec.vel[:nsteps], data64(sec), nsteps)
    assert rel_l2(plane.cpu().numpy(), ref_plane) <= 1e-5
    assert rel_l2(rows.cpu().numpy(), ref_rows) <= 1e-5
    only, none = mig.extrapolate(t["data"], vel, t["omega"], tab["tab32"], sec.desc, nsteps, rows=False)
    assert none is None and torch.equal(only, plane)


@pytest.mark.parametrize("nx,nw,nsteps,ntaps,layered", [
    (2049, 2, 5, 1, True), (3072, 2, 4, 35, True), (3073, 2, 3, 35, False), (8192, 1, 3, 3, True),
    (6145, 1, 2, 63, False), (1536, 2, 36, 37, True), (1537, 2, 3, 45, False), (1, 1, 3, 63, False),
    (6, 2, 2, 39, True), (2500, 3, 66, 11, True)])
def test_wide_and_long_filters(nx, nw, nsteps, ntaps, layered):
    print("wide nx=%d N=%d" % (nx, ntaps), flush=True)
    _check(synth.random_case(8000 + nx, nx, nsteps + 1, nw, ntaps=ntaps, nk=128, layered=layered), nsteps)


@pytest.mark.parametrize("nx,nw,nsteps", [(65, 224, 70), (65, 225, 70), (258, 257, 33), (1026, 226, 34)])
def test_rows_beside_and_after_the_launch(nx, nw, nsteps):
    """224 frequencies leave 32 of 256 CUs to reducers; one more and all rows are
    summed after the launch."""
    print("rows nx=%d nw=%d" % (nx, nw), flush=True)
    _check(synth.random_case(8300 + nx + nw, nx, nsteps + 1, nw, ntaps=25, nk=128), nsteps)
