"""The DMA kernels' shapes on the GPU at sizes where each is chosen: the
region kernel (64 x 64 regions, time split over eight waves), the tile kernel
(128 x 128 tiles, two time groups), the wide kernel, each with whole units
and with shared ones, at the edges of half stages, stages, regions and tiles.
Small cases against the oracle, larger ones against the scalar reference
kernel; repeated integrations and both nibble orders."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


def host(t):
    return t.cpu().numpy().astype(np.int64)


@pytest.mark.parametrize("n", [80, 112, 128, 144, 192, 208, 320])
@pytest.mark.parametrize("t", [1, 31, 32, 33, 64, 65, 127, 129, 255, 257, 700])
def test_small_jobs_match_oracle(n, t):
    x = synth.uniform_bytes(n, t, seed=[n, t])
    d = torch.from_numpy(x).cuda()
    ref = oracle.correlate(x)
    for re_low in (False, True):
        c = xeng.Correlator(n, 1, re_low=re_low)
        want = oracle.correlate(x, re_low=re_low) if re_low else ref
        c.correlate(0, d)
        assert np.array_equal(host(c.dump(0, reset=False)), want)
        c.correlate(0, d)              # into a slot that no longer holds zeros
        xeng.correlate_batch([(c, 0, d)])
        assert np.array_equal(host(c.dump(0)), 3 * want)
        c.close()


@pytest.mark.parametrize("n,t", [(512, 8192), (768, 3000), (1008, 4100), (1024, 20000), (1024, 33000), (1280, 1500),
                                 (1536, 5000), (1536, 9000), (2048, 100), (2048, 512), (2048, 1025), (2048, 3000),
                                 (2064, 9000), (3072, 700), (1000, 33000), (777, 6000)])
def test_larger_jobs_match_reference(n, t):
    g = torch.Generator(device="cuda").manual_seed(n * 7 + t)
    x = torch.randint(0, 256, (t, n), dtype=torch.uint8, device="cuda", generator=g)
    for re_low in (False, True):
        ref = xeng.correlate_reference(x, re_low=re_low)
        c = xeng.Correlator(n, 1, re_low=re_low)
        c.correlate(0, x)
        assert torch.equal(c.dump(0, reset=False), ref)
        c.correlate(0, x)
        assert torch.equal(c.dump(0), 2 * ref)
        b = xeng.Batch([(c, 0, x)])
        b.launch()
        assert torch.equal(c.dump(0), ref)
        b.close()
        c.close()


@pytest.mark.parametrize("n,slots,t", [(2048, 11, 96), (2048, 12, 200), (1000, 46, 64), (8192, 1, 64)])
def test_launches_past_the_caches(n, slots, t):
    """Launches whose accumulators stay just under, and pass, what goes past
    the caches: fresh slots, slots that hold sums, a resetting export between."""
    g = torch.Generator(device="cuda").manual_seed(n + slots + t)
    x = torch.randint(0, 256, (slots, t, n), dtype=torch.uint8, device="cuda", generator=g)
    c = xeng.Correlator(n, slots)
    jobs = [(c, k, x[k]) for k in range(slots)]
    for launches in (2, 1):
        for _ in range(launches):
            xeng.correlate_batch(jobs)
        outs = xeng.dump_batch([(c, k) for k in range(slots)])
        for k in range(slots):
            assert torch.equal(outs[k], launches * xeng.correlate_reference(x[k]))
    for k in range(slots):
        c.correlate(k, x[k])
        c.correlate_presum(k, x[k])
        assert torch.equal(c.dump(k), 2 * xeng.correlate_reference(x[k]))
    c.close()


@pytest.mark.parametrize("sizes", [
    [(128, 64), (320, 700)],                                       # a few regions
    [(512, 4096), (256, 1), (512, 4097), (80, 65)],                # regions in shares, a tiny job
    [(512, 1024)] * 7 + [(1000, 333)],                             # about as many regions as compute units
    [(1024, 2000)] * 6,                                            # tiles
    [(768, 12000), (1024, 5000), (64, 300), (200, 31), (777, 900)],
    [(1536, 300)] * 6,                                             # windows just past the compute units
    [(640, 900), (48, 2000), (17, 64)],                            # one job beside narrow ones
])
def test_batches_match_reference(sizes):
    g = torch.Generator(device="cuda").manual_seed(len(sizes) + sizes[0][0])
    jobs, want = [], []
    for k, (n, t) in enumerate(sizes):
        c = xeng.Correlator(n, 1, re_low=bool(k % 2))
        x = torch.randint(0, 256, (t, n), dtype=torch.uint8, device="cuda", generator=g)
        jobs.append((c, 0, x))
        want.append(xeng.correlate_reference(x, re_low=bool(k % 2)))
    xeng.correlate_batch(jobs)                 # into fresh slots
    xeng.correlate_batch(jobs)                 # and slots that hold sums
    b = xeng.Batch(jobs)
    b.launch()
    outs = xeng.dump_batch([(c, 0) for c, _, _ in jobs])
    for o, w in zip(outs, want):
        assert torch.equal(o, 3 * w)
    b.launch()
    b.close()
    for (c, _, _), w in zip(jobs, want):
        assert torch.equal(c.dump(0), w)
        c.close()
