"""Every DMA kernel over the same sizes, at the edges of half stages, stages,
regions and tiles, whatever the model would choose there: a tune-cache file
names the kernel, and a process of its own reads it.  Against the oracle."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NS = [80, 112, 128, 144, 192, 208, 256, 320]
TS = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, 700]
SHAPES = {"wide": 1, "tile": 3, "region": 4}

CHILD = r"""
import sys
sys.path.insert(0, sys.argv[1])
import numpy as np, torch, oracle, synth
from paper_2005_09481_amd import xeng
for n in %r:
    for t in %r:
        x = synth.uniform_bytes(n, t, seed=[n, t, 3])
        d, want = torch.from_numpy(x).cuda(), oracle.correlate(x)
        c = xeng.Correlator(n, 2)
        for jobs in ([(c, 0, d)], [(c, 0, d), (c, 1, d)]):
            assert xeng.tuning_lookup(jobs).source == xeng.XENG_TUNE_CACHE_FILE, (n, t)
            for k, s, y in jobs:
                k.correlate(s, y)              # into zeros
            xeng.correlate_batch(jobs)         # onto sums
            b = xeng.Batch(jobs)
            b.launch()
            b.close()
            for o in xeng.dump_batch([(k, s) for k, s, _ in jobs]):
                assert np.array_equal(o.cpu().numpy(), 3 * want), (n, t, len(jobs))
        c.close()
    print(n, flush=True)
""" % (NS, TS)


@pytest.mark.parametrize("min_stages", [1, 4])
@pytest.mark.parametrize("shape", SHAPES)
def test_kernel_matches_oracle(shape, min_stages, tmp_path):
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    lines = ['  {"n": %d, "t_class": %d, "jobs_class": %d, "dma": 1, "kernel": 0, "shape": %d, "wgs_per_cu": 2, '
             '"min_stages": %d, "plan_order": 1, "us_per_launch": 1.000000}' % (n, tc, jc, SHAPES[shape], min_stages)
             for n in NS for tc in range(10) for jc in (0, 1)]
    (tmp_path / f"xeng_tune_{arch}.json").write_text(
        '{"arch": "%s", "format": 2, "entries": [\n%s\n]}\n' % (arch, ",\n".join(lines)))
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=dict(os.environ, XENG_TUNE_DIR=str(tmp_path)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-200:] + r.stderr[-2000:]
