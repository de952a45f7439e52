"""The bias bases in the diagonal tiles' words below the diagonal: exports
with and without reset between integrations by every kernel that flushes a
diagonal tile, whole and in shared pieces, leave them as they are."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu

KERNELS = [xeng.XENG_KERNEL_AUTO, xeng.XENG_KERNEL_GENERAL, xeng.XENG_KERNEL_DMA4, xeng.XENG_KERNEL_FP8]


@pytest.fixture
def tuning():
    yield
    xeng.set_tuning(2, 4, xeng.XENG_KERNEL_AUTO)


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("n", [16, 33, 64, 96, 97, 112, 128, 129, 144, 256, 257, 272])
@pytest.mark.parametrize("t,min_stages", [(90, 4), (700, 1)])
def test_exports_between_integrations(n, t, min_stages, kernel, tuning):
    xeng.set_tuning(2, min_stages, kernel)
    xs = [synth.uniform_bytes(n, t + k, seed=[n, t, k]) for k in range(3)]
    ref = [oracle.correlate(x) for x in xs]
    d = [torch.from_numpy(x).cuda() for x in xs]
    c = xeng.Correlator(n, 2)
    try:
        total = 0
        for rep in range(3):
            # biases that differ from integration to integration
            k = rep % 3
            c.correlate(1, d[k])                       # into zeros
            total = ref[k].copy()
            assert np.array_equal(c.dump(1, reset=False).cpu().numpy(), total)
            xeng.correlate_batch([(c, 1, d[(k + 1) % 3])])   # and onto sums
            total += ref[(k + 1) % 3]
            c.correlate_presum(1, d[k])
            total += ref[k]
            if rep == 1:
                xeng.set_tuning(2, min_stages, xeng.XENG_KERNEL_AUTO)
                c.correlate(1, d[2])
                total += ref[2]
                xeng.set_tuning(2, min_stages, kernel)
            got = xeng.dump_batch([(c, 1)])[0] if rep % 2 else c.dump(1)
            assert np.array_equal(got.cpu().numpy(), total)
            assert not c.dump(1).any()
            assert not c.dump(0, reset=False).any()
    finally:
        c.close()
