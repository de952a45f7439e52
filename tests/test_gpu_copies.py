"""Padded and masked copies either side of the sizes at which a thread takes
several rows, against the scalar reference and plain torch."""
import pytest
import torch

from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t", [(1000, 32764), (1000, 32765), (1000, 32769), (257, 65533), (2047, 16387)])
def test_padded_copies(n, t):
    g = torch.Generator(device="cuda").manual_seed(n + t)
    x = torch.randint(0, 256, (t, n), dtype=torch.uint8, device="cuda", generator=g)
    c = xeng.Correlator(n, 1)
    c.correlate(0, x)
    assert torch.equal(c.dump(0), xeng.correlate_reference(x))
    c.close()


@pytest.mark.parametrize("n,t,block", [(1000, 16380, 64), (1000, 16387, 100), (40, 262143, 256), (2047, 8195, 2)])
def test_masked_copies(n, t, block):
    g = torch.Generator(device="cuda").manual_seed(n + t)
    x = torch.randint(0, 256, (t, n), dtype=torch.uint8, device="cuda", generator=g)
    f = (torch.rand((-(-t // block), n), device="cuda", generator=g) < 0.3).to(torch.uint8)
    masked = torch.where(f.repeat_interleave(block, dim=0)[:t] != 0, torch.full_like(x, 0x88), x)
    c = xeng.Correlator(n, 1, counts=True)
    c.correlate_flagged(0, x, f, block)
    assert torch.equal(c.dump(0), xeng.correlate_reference(masked))
    c.close()
