"""The folded adjoint kernel in both its forms (up to 1024 points and up to 1536) for every
filter length that it takes, element by element against the FP64 oracle's adjoint: two
velocity changes along each row, which move with depth across the edges of the waves'
outputs, so that no row has more than the kernel handles.  Tolerance 2e-5 of the largest
value: FP32 taps and arithmetic over a few steps, as for the other adjoint kernels."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import assert_rows_close, dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntaps", range(3, 36, 2))
@pytest.mark.parametrize("nx", [131, 1027])
def test_folded_adjoint_every_length(nx, ntaps):
    print("fold nx=%d N=%d" % (nx, ntaps), flush=True)
    nz, nw = 9, 3
    sec = synth.random_case(9700 + ntaps, nx, nz, nw, ntaps=ntaps, nk=64)
    vel = np.empty((nz, nx), np.float32)
    for k in range(nz):
        a, b = 120 + 2 * k, nx - 1 - 3 * k
        vel[k, :a], vel[k, a:b], vel[k, b:] = 900.0 + 40 * k, 1300.0 - 20 * (k // 2), 1700.0
    tab = mig.design_table(sec.desc, dev())
    img = np.random.default_rng(ntaps).standard_normal((nz, nx))
    got = mig.demigrate(torch.from_numpy(img).to(dev()), torch.from_numpy(vel).to(dev()), upload(sec)["omega"],
                        tab["tab32"], sec.desc)
    ref = oracle.demigrate(sec.desc, tab["tab64"].cpu().numpy(), sec.omega, vel, img)
    assert_rows_close(got.cpu().numpy(), ref, 2e-5, "fold nx=%d N=%d" % (nx, ntaps), axis=1)
