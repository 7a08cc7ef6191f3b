"""Image rows of batches, summed after the launch, where one section is far wider and
another far deeper than the rest: the same bits as each section by itself."""
import pytest
import torch

from paper_1912_05529_amd import mig, synth
from gpu_helpers import dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [((8192, 2, 1), (1, (1 << 21) + 2, 1)), ((2049, 3, 2), (1, 5000, 1), (7, 2, 5))])
def test_uneven_batch(sizes):
    print("uneven batch", sizes, flush=True)
    base = synth.random_case(77, 64, 4, 5, ntaps=37, nk=64)
    tab = mig.design_table(base.desc, dev())["tab32"]
    gen = torch.Generator().manual_seed(5)
    batch, want = [], []
    for nx, nz, nw in sizes:
        t = dict(data=torch.randn(nx, nw, dtype=torch.complex64, generator=gen).to(dev()),
                 vel=(1000.0 + 500.0 * torch.rand(nz, nx, generator=gen)).to(dev()),
                 omega=upload(base)["omega"][:nw].contiguous())
        want.append(mig.migrate(t["data"], t["vel"], t["omega"], tab, base.desc))
        batch.append(dict(t, image=torch.full_like(want[-1], float("nan"))))
    for got, ref in zip(mig.migrate_batched(batch, tab, base.desc), want):
        assert torch.equal(got, ref)
