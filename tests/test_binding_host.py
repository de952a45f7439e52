"""The binding's job records on the CPU: a slot may be any integer object
(Python, numpy or a torch scalar), as it may where ctypes converts it, and
what is no integer is refused."""
import ctypes
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2005_09481_amd import xeng

N = 16
SLOTS = [3, True, np.int8(3), np.uint8(3), np.int16(3), np.int32(3), np.uint32(3), np.int64(3), np.uint64(3),
         torch.tensor(3), torch.tensor(3, dtype=torch.int32), torch.tensor(3, dtype=torch.uint8), -1, np.int32(-1)]


def fake_correlator():
    h = ctypes.c_void_p(0x1000)
    return SimpleNamespace(_h=h, handle=h, n_inputs=N, device=0, _vis_numel=2 * xeng.tri(N))


@pytest.mark.parametrize("slot", SLOTS, ids=lambda s: f"{type(s).__name__}-{int(s)}")
def test_any_integer_slot(slot, monkeypatch):
    c = fake_correlator()
    arr = xeng._job_array([(c, slot, torch.empty((0, N), dtype=torch.uint8))])
    assert (arr[0].ctx, arr[0].slot, arr[0].reserved) == (0x1000, int(slot), 0)

    seen = []

    def dump_batch(jobs, n, stream):
        seen.extend((jobs[k].ctx, jobs[k].slot, jobs[k].reset, jobs[k].out, jobs[k].reserved) for k in range(n))
        return 0

    monkeypatch.setattr(xeng, "lib", lambda: SimpleNamespace(xeng_dump_batch=dump_batch))
    monkeypatch.setattr(xeng, "_stream_handle", lambda stream, device: None)
    out = torch.empty((xeng.tri(N), 2), dtype=torch.int32)
    assert xeng.dump_batch([(c, slot, out, False), (c, slot, out)])[0] is out
    assert seen == [(0x1000, int(slot), r, out.data_ptr(), 0) for r in (0, 1)]


@pytest.mark.parametrize("slot", [1.0, "1", None, np.float32(1), np.array([1, 2])])
def test_other_slots_are_refused(slot):
    c = fake_correlator()
    with pytest.raises(TypeError):
        xeng._job_array([(c, slot, torch.empty((0, N), dtype=torch.uint8))])
    with pytest.raises(TypeError):
        xeng.dump_batch([(c, slot, torch.empty((xeng.tri(N), 2), dtype=torch.int32))])
