"""Image partials of volumes around the 24 groups from which 32 are summed at a time, and
around one and two times 32 with 0 to 23 groups left: against a run with all frequencies
in one group.  Groups change only the order of the FP64 sum over frequencies: under 100
terms, a few 1e-16 each, against 1e-12 of the image's largest value; planes are the same
bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntaps,nw", [(1, 23), (3, 24), (5, 25), (7, 31), (9, 33), (11, 55), (11, 56), (3, 64), (5, 65)])
def test_partials_of_many_groups(ntaps, nw):
    print("volume %d taps, %d groups" % (ntaps, nw), flush=True)
    vol = synth.random_volume(950 + nw, 34, 67, 4, nw, ntaps=ntaps, nk=64)
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
