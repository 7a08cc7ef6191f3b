"""Adjoint of wide sections and long filters at the edges of its kernels (two and four
outputs per thread, several runs, one to four taps of products at a time; the folded
kernel up to 1536 points and its fallback), element by element against the FP64
oracle's adjoint.  Tolerance 2e-5 of the largest value: FP32 taps and arithmetic over a
few steps, as for the other adjoint kernels."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import assert_rows_close, dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,nw,ntaps,layered", [
    (1025, 12, 3, 35, True), (1536, 9, 2, 33, True), (1536, 6, 2, 35, False), (1537, 8, 2, 35, True),
    (3072, 4, 2, 25, False), (3073, 4, 1, 35, True), (8192, 3, 1, 63, True), (6700, 3, 1, 63, False),
    (1, 3, 2, 63, False), (63, 5, 2, 37, True), (128, 4, 2, 1, True), (129, 1, 2, 45, True),
    (1500, 5, 2, 3, False)])
def test_demigrate_wide_and_long_filters(nx, nz, nw, ntaps, layered):
    print("adjoint nx=%d N=%d" % (nx, ntaps), flush=True)
    sec = synth.random_case(9100 + nx, nx, nz, nw, ntaps=ntaps, nk=128, layered=layered)
    tab = mig.design_table(sec.desc, dev())
    t = upload(sec)
    img = np.random.default_rng(nx).standard_normal((nz, nx))
    got = mig.demigrate(torch.from_numpy(img).to(dev()), t["vel"], t["omega"], tab["tab32"], sec.desc)
    ref = oracle.demigrate(sec.desc, tab["tab64"].cpu().numpy(), sec.omega, sec.vel, img)
    assert_rows_close(got.cpu().numpy(), ref, 2e-5, "adjoint nx=%d" % nx, axis=1)
    again = mig.demigrate(torch.from_numpy(img).to(dev()), t["vel"], t["omega"], tab["tab32"], sec.desc)
    assert torch.equal(again, got)
