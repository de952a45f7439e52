"""The export's edges on the GPU: inputs that end inside a tile, a block or a
lane's pair of columns; repeated exports with and without reset (the
imaginary biases are only ever added to, an export subtracts those of the
last reset); batched exports of jobs with different tile counts; slots of a
live prepared batch, whose device counter a resetting export clears."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


def vis(x):
    return oracle.correlate(x)


def host(t):
    return t.cpu().numpy().astype(np.int64)


def dev(x):
    return torch.from_numpy(x).cuda()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 31, 33, 63, 64, 65, 96, 127, 128, 129, 160, 255, 257, 272])
def test_exports_in_turn(n):
    xs = [synth.uniform_bytes(n, t, seed=[n, t]) for t in (70, 33, 65, 40)]
    ref = [vis(x) for x in xs]
    c = xeng.Correlator(n, 2)
    c.correlate(1, dev(xs[0]))
    assert np.array_equal(host(c.dump(1, reset=False)), ref[0])
    c.correlate(1, dev(xs[1]))
    assert np.array_equal(host(c.dump(1, reset=False)), ref[0] + ref[1])
    assert np.array_equal(host(c.dump(1)), ref[0] + ref[1])
    assert not host(c.dump(1)).any()
    c.correlate(1, dev(xs[2]))
    assert np.array_equal(host(c.dump(1)), ref[2])
    # a reset that is no export, between integrations
    c.correlate(1, dev(xs[0]))
    c.reset(1)
    c.correlate(1, dev(xs[3]))
    assert np.array_equal(host(c.dump(1)), ref[3])
    assert not host(c.dump(0)).any()
    c.close()


@pytest.mark.parametrize("n", [48, 130, 272])
def test_signed_and_unsigned_forms_in_turn(n):
    xs = [synth.uniform_bytes(n, t, seed=[n, t, 1]) for t in (80, 64, 50)]
    ref = [vis(x) for x in xs]
    c = xeng.Correlator(n, 1)
    for batched in (False, True):
        c.correlate(0, dev(xs[0]))
        c.correlate_presum(0, dev(xs[1]))
        assert np.array_equal(host(c.dump(0, reset=False)), ref[0] + ref[1])
        c.correlate_presum(0, dev(xs[2]))
        got = xeng.dump_batch([(c, 0)])[0] if batched else c.dump(0)
        assert np.array_equal(host(got), sum(ref))
    c.close()


def test_batched_exports_of_mixed_sizes():
    ns = [64, 300, 1, 129, 2048, 272, 64]
    cs = [xeng.Correlator(n, 2) for n in ns]
    for rep in range(3):
        xs = [synth.uniform_bytes(n, 40 + k, seed=[n, k, rep]) for k, n in enumerate(ns)]
        xeng.correlate_batch([(c, 1, dev(x)) for c, x in zip(cs, xs)])
        keep = xeng.dump_batch([(c, 1, None, False) for c in cs])
        outs = xeng.dump_batch([(c, 1) for c in cs])
        for x, a, b in zip(xs, keep, outs):
            ref = vis(x)
            assert np.array_equal(host(a), ref) and np.array_equal(host(b), ref)
    for c in cs:
        c.close()


@pytest.mark.parametrize("n", [64, 272])
def test_exports_of_a_prepared_batch(n):
    t = 100
    x = synth.uniform_bytes(n, 3 * t, seed=[n, 5])
    parts = [dev(np.ascontiguousarray(x[k * t:(k + 1) * t])) for k in range(3)]
    ref = [vis(x[k * t:(k + 1) * t]) for k in range(3)]
    c = xeng.Correlator(n, 3)
    b = xeng.Batch([(c, k, parts[k]) for k in range(3)])
    for rep in range(3):
        b.launch()
        b.launch()
        assert c.samples_integrated(0) == 2 * t
        outs = xeng.dump_batch([(c, 0), (c, 1)]) + [c.dump(2)]
        assert [c.samples_integrated(k) for k in range(3)] == [0, 0, 0]
        for k in range(3):
            assert np.array_equal(host(outs[k]), 2 * ref[k])
    b.launch()
    c.reset(1)
    assert c.samples_integrated(1) == 0 and c.samples_integrated(2) == t
    assert b.check() == xeng.XENG_OK
    assert not host(c.dump(1)).any()
    assert np.array_equal(host(c.dump(2)), ref[2])
    b.close()
    c.close()
