"""Batched exports past the caches: launches whose resetting exports hold 192
MiB of accumulators and 768 MiB, of equal and of different tile counts, with
inputs that end inside a tile; an export that keeps the sums before, two
integrations with their exports.  Against the scalar reference."""
import pytest
import torch

from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(1000, 46)], [(2048, 46)], [(1000, 90), (2047, 28)], [(130, 500), (2000, 8), (1, 5)]])
def test_exports_match_reference(sizes):
    g = torch.Generator(device="cuda").manual_seed(sizes[0][0])
    jobs = []
    for n, slots in sizes:
        c = xeng.Correlator(n, slots)
        jobs += [(c, k, torch.randint(0, 256, (33, n), dtype=torch.uint8, device="cuda", generator=g))
                 for k in range(slots)]
    want = [xeng.correlate_reference(x) for _, _, x in jobs]
    xeng.correlate_batch(jobs)
    kept = xeng.dump_batch([(c, k, None, False) for c, k, _ in jobs])
    for rep in (1, 2):
        outs = xeng.dump_batch([(c, k) for c, k, _ in jobs])
        for o, w, x in zip(outs, want, kept):
            assert torch.equal(o, rep * w) and torch.equal(x, w)
        xeng.correlate_batch(jobs)
        xeng.correlate_batch(jobs)
    for c in {j[0] for j in jobs}:
        c.close()
