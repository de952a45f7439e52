"""The row kernels at their edges: RFI flags at input counts and block
lengths either side of a lane row, a chunk and a row quad, at every byte
alignment; padded and masked copies of rows that end at the allocation's end;
sample counts stored by the first flagged call after a reset and added to by
the next.  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import oracle.flags as OF
import synth
from paper_2005_09481_amd import xeng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 63, 64, 65, 255, 257, 511, 513, 1023, 1025, 1040])
@pytest.mark.parametrize("t,bl", [(1, 2), (2, 2), (130, 3), (131, 5), (70, 33), (2100, 1024), (300, 64)])
def test_rfi_flags_edges(n, t, bl):
    x = synth.rfi_channel(n, t, seed=[n, t, bl], block_len=bl, tone_frac=0.2, burst_frac=0.2)
    got = xeng.rfi_flags(torch.from_numpy(x).cuda(), block_len=bl).cpu().numpy()
    assert np.array_equal(got, OF.sk_flags(x, block_len=bl))


def test_rfi_flags_every_power():
    # every byte value, alone in a block and beside every other value
    x = np.arange(256, dtype=np.uint8)[None].repeat(8, axis=0)
    x[4:] = np.arange(256, dtype=np.uint8)[::-1]
    for bl in (2, 5, 8):
        got = xeng.rfi_flags(torch.from_numpy(x).cuda(), block_len=bl).cpu().numpy()
        assert np.array_equal(got, OF.sk_flags(x, block_len=bl))


@pytest.mark.parametrize("off", range(1, 16, 2))
def test_rfi_flags_alignments(off):
    x = synth.rfi_channel(150, 260, seed=off, block_len=50, tone_frac=0.1, burst_frac=0.1)
    view = torch.from_numpy(x).cuda()[:, off:off + 131]
    want = OF.sk_flags(np.ascontiguousarray(x[:, off:off + 131]), block_len=50)
    assert np.array_equal(xeng.rfi_flags(view, n_inputs=131, block_len=50).cpu().numpy(), want)


@pytest.mark.parametrize("n", [256, 257, 271, 300, 383])
@pytest.mark.parametrize("off", [0, 1, 6, 15])
def test_padded_rows(n, off):
    x = synth.uniform_bytes(n + 16, 77, seed=[n, off])
    view = torch.from_numpy(x).cuda()[:, off:off + n]
    want = oracle.correlate(np.ascontiguousarray(x[:, off:off + n]))
    c = xeng.Correlator(n, 1)
    c.correlate(0, view)
    xeng.correlate_batch([(c, 0, view)])
    assert np.array_equal(c.dump(0).cpu().numpy().astype(np.int64), 2 * want)
    c.close()


@pytest.mark.parametrize("n,t,bl", [(7, 50, 3), (48, 300, 64), (130, 257, 32), (300, 100, 1)])
def test_counts_first_call_and_after_resets(n, t, bl):
    rng = np.random.default_rng([n, t])
    c = xeng.Correlator(n, 2, counts=True)
    for rep in range(3):
        want_v, want_c = 0, 0
        for k in range(2):
            x = synth.uniform_bytes(n, t, seed=[n, rep, k])
            fl = (rng.random((OF.n_blocks(t, bl), n)) < 0.4).astype(np.uint8)
            v, cn = OF.correlate_flagged(x, fl, bl)
            c.correlate_flagged(1, torch.from_numpy(x).cuda(), torch.from_numpy(fl).cuda(), bl)
            want_v, want_c = want_v + v, want_c + cn
        assert np.array_equal(c.dump_counts(1).cpu().numpy(), want_c)
        if rep == 1:
            c.reset(1)
            assert not c.dump(1).any()
        else:
            assert np.array_equal(c.dump(1).cpu().numpy().astype(np.int64), want_v)
        assert not c.dump_counts(1).any()
        # unflagged samples alone: every pair counts them
        c.correlate(1, torch.from_numpy(synth.uniform_bytes(n, 10, seed=1)).cuda())
        assert (c.dump_counts(1) == 10).all()
        c.reset(1)
    assert not c.dump_counts(0).any()
    c.close()
