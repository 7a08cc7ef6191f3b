"""Image partials of volumes at the edges of the numbers of groups that are summed together
(8, 16, 32 and more), and grids of any remainder modulo 8.  Groups change only the order
of the FP64 sum over frequencies: 40 terms, a few 1e-16 each, against 1e-12 of the image's
largest value; planes are the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nw", [(33, 70, 8), (20, 65, 9), (40, 30, 16), (33, 129, 17), (12, 64, 32), (35, 66, 33),
                                      (31, 63, 40), (65, 10, 7)])
def test_partials_of_any_number_of_groups(nx, ny, nw):
    print("volume %d x %d, %d groups" % (nx, ny, nw), flush=True)
    vol = synth.random_volume(900 + nw, nx, ny, 4, nw, ntaps=7, nk=64)
    tab = torch.from_numpy(oracle.design_table_2d(vol.desc)[0].astype(np.complex64)).to(dev())
    data = torch.from_numpy(np.ascontiguousarray(np.moveaxis(vol.data.astype(np.complex64), 2, 0))).to(dev())
    vel = torch.from_numpy(np.ascontiguousarray(vol.vel)).to(dev())
    om = torch.from_numpy(vol.omega).to(dev())
    planes, imgs = [], []
    for wpg in (1, nw):
        planes.append(torch.empty_like(data))
        imgs.append(mig.migrate3d(data, vel, om, tab, vol.desc, omegas_per_group=wpg, plane_out=planes[-1]))
    assert torch.equal(planes[0], planes[1])
    assert float((imgs[0] - imgs[1]).abs().max()) <= 1e-12 * float(imgs[1].abs().max())
