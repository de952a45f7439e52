"""Beamforming at the edges of its kernel's forms: times either side of the
row-block and dispatch boundaries, input counts either side of a 16-byte
load, a pair of k-steps and a weight chunk, rows at every byte alignment; the
last row ends with the allocation.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle.beams as OB
import synth
from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


def check(x_dev, x, w):
    want = OB.beamform(x, w)
    bm = xeng.Beams(w, device=0)
    got = bm.form(x_dev).cpu().numpy().astype(np.int64)
    assert np.array_equal(got, want)
    assert np.array_equal(bm.form(x_dev, shift=9).cpu().numpy(), OB.quantize(want, 9))
    bm.close()


@pytest.mark.parametrize("n", [15, 17, 31, 33, 63, 65, 129, 1000, 2047, 2049, 2063])
@pytest.mark.parametrize("t", [1, 17, 33])
def test_input_counts(n, t):
    x = synth.uniform_bytes(n, t, seed=[n, t, 7])
    check(torch.from_numpy(x).cuda(), x, synth.beam_weights(5, n, seed=[n, 3]))


@pytest.mark.parametrize("t", [31, 32, 8192, 8193, 16400, 24575, 24576, 24641, 33000])
@pytest.mark.parametrize("n", [48, 70])
def test_times(n, t):
    x = synth.uniform_bytes(n, t, seed=[n, t, 8])
    check(torch.from_numpy(x).cuda(), x, synth.beam_weights(16, n, seed=[n, 4]))


@pytest.mark.parametrize("shift", range(1, 16, 2))
def test_row_alignments(shift):
    n, t = 100, 40
    x = synth.uniform_bytes(n + 16, t, seed=[shift, 9])
    view = torch.from_numpy(x).cuda()[:, shift:shift + n]
    check(view, np.ascontiguousarray(x[:, shift:shift + n]), synth.beam_weights(10, n, seed=[n, 5]))
