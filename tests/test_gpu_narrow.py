"""Depth stepping with one output per thread (up to 512 points) against two outputs per
thread (the batched form): planes of both are the same sums in the same order, so images
are the same bits.  Refills of every width against the FP64 oracle where every output
changes its filter at every step.  Tolerance: relative L2 1e-5 after a few steps (FP32
taps and arithmetic: about 1e-7 per operation, 2 N operations per output and step).  Batches whose
image rows are summed after the launch."""
import pytest
import torch

import oracle
from paper_1912_05529_amd import mig, synth
from gpu_helpers import data64, dev, rel_l2, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,nw,ntaps,layered", [
    (1, 3, 2, 35, True), (63, 70, 3, 1, True), (64, 68, 2, 35, False), (65, 36, 5, 3, True), (128, 2, 4, 25, False),
    (256, 35, 260, 35, True), (257, 34, 7, 33, False), (257, 5, 257, 25, True), (511, 67, 3, 19, True),
    (512, 4, 5, 35, False), (513, 4, 5, 35, True)])
def test_one_and_two_outputs_per_thread(nx, nz, nw, ntaps, layered):
    print("narrow nx=%d N=%d" % (nx, ntaps), flush=True)
    sec = synth.random_case(9300 + nx, nx, nz, nw, ntaps=ntaps, nk=128, layered=layered)
    tab = mig.design_table(sec.desc, dev())["tab32"]
    t = upload(sec)
    one = mig.migrate(t["data"], t["vel"], t["omega"], tab, sec.desc)
    two = mig.migrate_batched([dict(t, image=torch.empty_like(one)) for _ in range(2)], tab, sec.desc)
    assert torch.equal(one, two[0]) and torch.equal(one, two[1])


@pytest.mark.parametrize("nx,nw,nsteps,ntaps,layered", [
    (255, 3, 7, 35, False), (600, 2, 6, 33, False), (1024, 2, 5, 35, False), (1025, 2, 5, 35, False),
    (1536, 2, 4, 33, False), (1537, 2, 4, 35, False), (2048, 2, 4, 33, False), (2047, 2, 40, 35, True),
    (1400, 3, 40, 25, True), (900, 1, 1, 3, False), (1100, 1, 2, 1, False), (1600, 1, 1, 5, False)])
def test_refills(nx, nw, nsteps, ntaps, layered):
    print("refills nx=%d N=%d" % (nx, ntaps), flush=True)
    sec = synth.random_case(9400 + nx, nx, nsteps + 1, nw, ntaps=ntaps, nk=128, layered=layered)
    tab = mig.design_table(sec.desc, dev())
    t = upload(sec)
    vel = t["vel"][:nsteps].contiguous()
    plane, rows = mig.extrapolate(t["data"], vel, t["omega"], tab["tab32"], sec.desc, nsteps)
    ref_plane, ref_rows = oracle.extrapolate(sec.desc, tab["tab64"].cpu().numpy(), sec.omega, sec.vel[:nsteps],
                                             data64(sec), nsteps)
    assert rel_l2(plane.cpu().numpy(), ref_plane) <= 1e-5
    assert rel_l2(rows.cpu().numpy(), ref_rows) <= 1e-5


@pytest.mark.parametrize("nxs,nw,nz,ntaps", [
    ((300, 129, 512, 1000), 70, 40, 25), ((1100, 1501), 120, 5, 35), ((1600, 2048, 1537), 90, 4, 35),
    ((2049, 100, 3000), 90, 3, 37), ((64,), 300, 3, 11), ((64, 65, 1024, 1200, 2000, 2100), 60, 35, 35)])
def test_batch_rows_after_the_launch(nxs, nw, nz, ntaps):
    """Batches with more workgroups than CUs (sections of unequal depths and frequencies):
    the same bits as each section by itself."""
    print("batch nx=%s N=%d" % (nxs, ntaps), flush=True)
    secs = [synth.random_case(9500 + nx, nx, nz + i, nw + 3 * i, ntaps=ntaps, nk=128) for i, nx in enumerate(nxs)]
    tab = mig.design_table(secs[0].desc, dev())["tab32"]
    batch, want = [], []
    for sec in secs:
        t = upload(sec)
        want.append(mig.migrate(t["data"], t["vel"], t["omega"], tab, secs[0].desc))
        batch.append(dict(t, image=torch.full_like(want[-1], float("nan"))))
    for got, ref in zip(mig.migrate_batched(batch, tab, secs[0].desc), want):
        assert torch.equal(got, ref)
