"""The library's host bookkeeping without a GPU: its HIP calls go to a
stand-in (tests/fake_hip.cpp) that counts allocations and launches and can
make a call fail.  Every test runs in a process of its own, so that the
stand-in reaches no other test."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
F = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
for f in ("fake_device_bytes", "fake_pool_allocs", "fake_pool_bytes", "fake_launches", "fake_workgroups"):
    getattr(F, f).restype = ctypes.c_int64
F.fake_pool_bytes.argtypes = [ctypes.c_int64]
F.fake_launches.argtypes = F.fake_workgroups.argtypes = [ctypes.c_char_p]
from paper_2005_09481_amd import xeng as X
L = X.lib()
P = 1 << 20          # a sample address: never read, kernels do nothing

def create(n, slots=1, flags=0, budget=0):
    h = ctypes.c_void_p()
    assert L.xeng_create(ctypes.byref(X._Config(n, slots, 0, flags, budget)), ctypes.byref(h)) == 0
    return h

def jobs(*js):
    return (X._Job * len(js))(*[X._Job(c, s, 0, P, t, stride) for c, s, t, stride in js]), len(js), None

def dumps(*js):
    return (X._DumpJob * len(js))(*[X._DumpJob(c, s, r, P, 0, 0) for c, s, r in js]), len(js), None
"""


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I",
                    "/opt/rocm/include", os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", out, "-ldl"],
                   check=True, capture_output=True)
    return out


@pytest.fixture
def run(fake_hip, tmp_path):
    def go(body):
        env = dict(os.environ, XENG_TUNE_DIR=str(tmp_path))
        r = subprocess.run([sys.executable, "-c", PRELUDE + body, ROOT, fake_hip], env=env, capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr[-3000:]
        return r.stdout
    return go


def test_stand_in_takes_the_calls(run):
    run(r"""
c = create(130, 2)
assert L.xeng_correlate(c, 0, P, 100, 130, None) == 0
assert L.xeng_samples_integrated(c, 0) == 100
assert L.xeng_dump(c, 0, P, 1, None) == 0
assert F.fake_launches(b"xcorr_mfma") == 1 and F.fake_launches(b"vis_dump") == 1
assert L.xeng_samples_integrated(c, 0) == 0
assert L.xeng_destroy(c) == 0
""")


def test_failed_event_record_after_a_batched_export(run):
    # the export is queued when the event behind it cannot be recorded: its
    # slots are reset on the device, so on the host too, and the staging
    # buffer it reads is not reused while it may still run
    run(r"""
c = create(130, 3)
assert L.xeng_correlate_batch(*jobs((c, 0, 64, 130), (c, 1, 64, 130), (c, 2, 64, 130))) == 0
F.fake_clear()
F.fake_fail_records(1)
assert L.xeng_dump_batch(*dumps((c, 0, 1), (c, 1, 0))) == X.XENG_EDEVICE
assert F.fake_launches(b"vis_dump_batch") == 1
assert [L.xeng_samples_integrated(c, s) for s in range(3)] == [0, 64, 64]
assert F.fake_stream_syncs() == 1
assert L.xeng_dump_batch(*dumps((c, 0, 1), (c, 1, 1))) == 0
assert [L.xeng_samples_integrated(c, s) for s in range(3)] == [0, 0, 64]
""")


def test_failed_event_record_after_a_batched_correlation(run):
    # the call reports the error, after the launch that reads its staging
    # buffer has ended
    run(r"""
c = create(130, 2)
F.fake_fail_records(1)
assert L.xeng_correlate_batch(*jobs((c, 0, 64, 130), (c, 1, 64, 130))) == X.XENG_EDEVICE
assert F.fake_launches(b"xcorr_mfma") == 1 and F.fake_stream_syncs() == 1
""")


def test_padded_batches_fit_the_scratch_they_need(run):
    # N = 257 needs rows of 272 bytes; whole cache lines (384) are taken only
    # where the scratch has room, never instead of the DMA kernel
    run(r"""
c = create(257, 2)
def batch(limit, *ts):
    assert L.xeng_set_pad_chunk_bytes(limit) == 0
    F.fake_clear()
    assert L.xeng_correlate_batch(*jobs(*[(c, k, t, 257) for k, t in enumerate(ts)])) == 0
    copies, general = F.fake_launches(b"copy_rows"), F.fake_launches(b"xcorr_mfma")
    return copies, general, F.fake_pool_bytes(0) if F.fake_pool_allocs() else 0

assert batch(272 * 640, 640) == (1, 0, 272 * 640)            # exactly the tight rows
assert batch(272 * 640 - 1, 640) == (0, 1, 0)
assert batch(384 * 640, 640) == (1, 0, 384 * 640)            # room for whole lines
assert batch(272 * 1280, 640, 640) == (2, 0, 272 * 1280)
assert batch((272 + 384) * 640, 640, 640) == (2, 0, (272 + 384) * 640)
assert batch(0, 640, 640) == (2, 0, 2 * 384 * 640)
""")


def test_padded_calls_take_no_more_chunks_than_they_need(run):
    run(r"""
c, small = create(257), create(7, 1, X.XENG_COUNTS)
def chunks(call, limit):
    assert L.xeng_set_pad_chunk_bytes(limit) == 0
    F.fake_clear()
    assert call() == 0
    assert F.fake_launches(b"copy_rows") == F.fake_launches(b"xcorr_region") + F.fake_launches(b"xcorr_tile")
    return F.fake_launches(b"copy_rows")

one = lambda: L.xeng_correlate(c, 0, P, 640, 257, None)
assert chunks(one, 0) == 1 and F.fake_pool_bytes(0) == 384 * 640
assert chunks(one, 272 * 640) == 1 and F.fake_pool_bytes(0) == 272 * 640
assert chunks(one, 272 * 320) == 2
flagged = lambda: L.xeng_correlate_flagged(small, 0, P, 2048, 7, P, 64, None)
assert chunks(flagged, 0) == 1 and F.fake_pool_bytes(1) == 128 * 2048      # (behind the counts' masks)
assert chunks(flagged, 16 * 2048) == 1 and F.fake_pool_bytes(1) == 16 * 2048
assert chunks(flagged, 16 * 1024) == 2
""")


def test_a_context_allocates_what_is_counted(run):
    # accumulators and biases (xeng_slot_bytes, the memory budget), beside them
    # the pre-sums (16 bytes per input, N rounded up to 4) and a counter per
    # slot, with XENG_COUNTS the pair counts; nothing else per slot
    run(r"""
create(1)                                    # (the device's own set-up)
for n in (1, 64, 100, 128, 130, 1000, 2048):
    for slots in (1, 2, 33):
        for flags in (0, X.XENG_COUNTS):
            before = F.fake_device_bytes()
            counts = -(-X.tri(n) // 4) * 16 if flags else 0
            c = create(n, slots, flags, slots * (X.slot_bytes(n) + counts))
            got = F.fake_device_bytes() - before
            assert got == slots * (X.slot_bytes(n) + 16 * -(-n // 4) * 4 + counts) + 16 * -(-slots // 2), (n, slots, got)
            assert L.xeng_destroy(c) == 0 and F.fake_device_bytes() == before
""")


def test_short_copies_fill_the_chip(run):
    # one row a thread until several leave eight workgroups per compute unit
    run(r"""
c, f = create(1000), create(1000, 1, X.XENG_COUNTS)       # four rows side by side in a workgroup
for t, wgs in ((1, 1), (256, 64), (8192, 2048), (32764, 8191), (32768, 2048), (40000, 2500)):
    assert L.xeng_correlate(c, 0, P, t, 1000, None) == 0
    assert F.fake_workgroups(b"copy_rows") == wgs, (t, F.fake_workgroups(b"copy_rows"))
for t, wgs in ((64, 16), (16380, 4095), (16384, 2048)):
    assert L.xeng_correlate_flagged(f, 0, P, t, 1000, P, 64, None) == 0
    assert F.fake_workgroups(b"copy_rows") == wgs, (t, F.fake_workgroups(b"copy_rows"))
""")


def test_small_flag_blocks_take_the_byte_form(run):
    run(r"""
def form(n, block, t):
    F.fake_clear()
    cfg = X._RfiConfig(block, 1000, 625, 1375, 0)
    assert L.xeng_rfi_flags(P, t, n, n, 0, ctypes.byref(cfg), P, None) == 0
    return "bytes" if F.fake_launches(b"sk_flags_bytes") else "vec" if F.fake_launches(b"sk_flags_vec") else None
for n, block, t, want in ((15, 1024, 4096, "bytes"), (16, 16, 4096, "bytes"), (16, 17, 4096, "vec"),
                          (64, 16, 65536, "bytes"), (64, 32, 4096, "vec"), (749, 4, 32768, "bytes"),
                          (750, 4, 32768, "vec"), (1000, 2, 65536, "bytes"), (1000, 3, 32768, "vec"),
                          (1000, 8, 8192, "bytes"), (1000, 9, 8192, "vec"), (2048, 8, 8192, "bytes"),
                          (2048, 8, 8193, "vec"), (2048, 256, 256, "vec")):
    assert form(n, block, t) == want, (n, block, t)
""")


def test_large_resetting_exports_go_past_the_caches(run):
    # from 192 MiB of accumulators that a launch resets (17 MiB a slot of N =
    # 2048) their output does, from 768 MiB on all they touch
    run(r"""
c = create(2048, 46)
def form(call, name):
    F.fake_clear()
    assert call() == 0
    got = [f for f in range(3) if F.fake_launches(b"%sLi%dE" % (name, f))]
    assert len(got) == 1
    return got[0]
def batch(resets):
    return form(lambda: L.xeng_dump_batch(*dumps(*[(c, k, r) for k, r in enumerate(resets)])), b"vis_dump_batchI")
assert [batch([1] * k) for k in (1, 11, 12, 45, 46)] == [0, 0, 1, 1, 2]
assert batch([1] * 11 + [0] * 10) == 0 and batch([0] * 46) == 0 and batch([1] * 12 + [0] * 34) == 1
big = create(8192)          # 260 MiB
one = lambda reset: lambda: L.xeng_dump(big, 0, P, reset, None)
assert form(one(1), b"vis_dumpILb0E") == 1 and form(one(0), b"vis_dumpILb0E") == 0
assert L.xeng_correlate_presum(big, 0, P, 64, 8192, None) == 0
assert form(one(1), b"vis_dumpILb1E") == 1
small = create(64)
assert form(lambda: L.xeng_dump(small, 0, P, 1, None), b"vis_dumpILb0E") == 0
""")


FORMAT2 = ('{"arch": "gfx950", "format": %d, "entries": [\n'
           '  {"n": 512, "t_class": 10, "jobs_class": 0, "dma": 1, "kernel": %d, %s"wgs_per_cu": 2, "min_stages": 4, '
           '"plan_order": 1, "us_per_launch": 1.000000}\n]}\n')


def tune_file(tmp_path, *args):
    (tmp_path / "xeng_tune_gfx950.json").write_text(FORMAT2 % args)


LOOKUP = r"""
c = create(512)
def lookup(t):
    out = X._Tuning()
    assert L.xeng_tuning_lookup(*jobs((c, 0, t, 512))[:2], ctypes.byref(out)) == 0
    return out.kernel, out.source
def launched(t, batch=False):
    F.fake_clear()
    if batch:
        assert L.xeng_correlate_batch(*jobs((c, 0, t, 512))) == 0
    else:
        assert L.xeng_correlate(c, 0, P, t, 512, None) == 0
    return [k for k in ("xcorr_dmaILi8", "xcorr_dmaILi4", "xcorr_tile", "xcorr_region", "xcorr_mfma")
            if F.fake_launches(k.encode())]
"""


@pytest.mark.parametrize("fast", ["xcorr_dmaILi8", "xcorr_dmaILi4", "xcorr_tile", "xcorr_region", "xcorr_mfma"])
def test_autotuner_times_every_kernel_and_keeps_the_fastest(run, fast):
    # every DMA kernel is a candidate by itself, and the one measured fastest
    # is what later calls of the class launch, here and in a new process
    kernel = {"xcorr_dmaILi4": "DMA4", "xcorr_mfma": "GENERAL"}.get(fast, "AUTO")
    run(LOOKUP + r"""
F.fake_fast_kernel(b"%s")
best = X._Tuning()
F.fake_clear()
assert L.xeng_autotune(*jobs((c, 0, 2000, 512))[:2], 1, None, ctypes.byref(best)) == 0
for k in (b"xcorr_dmaILi8", b"xcorr_dmaILi4", b"xcorr_tile", b"xcorr_region", b"xcorr_mfma"):
    assert F.fake_launches(k) > 0, k
assert best.kernel == X.XENG_KERNEL_%s and best.saved == 1 and best.us_per_launch == 500.0
assert lookup(1500) == (best.kernel, X.XENG_TUNE_MEASURED)
assert launched(1500) == ["%s"] and launched(1500, True) == ["%s"]
assert launched(9000) == ["xcorr_region"]          # another class: the modelled kernel
""" % (fast, kernel, fast, fast))
    run(LOOKUP + r"""
assert lookup(1500) == (X.XENG_KERNEL_%s, X.XENG_TUNE_CACHE_FILE)
assert launched(1500) == ["%s"] and launched(1500, True) == ["%s"]
""" % (kernel, fast, fast))


def test_tune_files_of_the_older_format_are_not_read(run, tmp_path):
    # their kernel 0 does not say which DMA kernel was measured
    for args in ((1, 1, ""), (1, 0, ""), (1, 0, '"shape": 3, '), (2, 1, "")):
        tune_file(tmp_path, *args)
        run(LOOKUP + "assert lookup(1500) == (X.XENG_KERNEL_AUTO, X.XENG_TUNE_SETTINGS)\n"
            "assert launched(1500) == ['xcorr_region']\n")


@pytest.mark.parametrize("kernel,shape,ok", [(0, 0, "xcorr_region"), (0, 1, "xcorr_dmaILi8"), (0, 3, "xcorr_tile"),
                                             (0, 4, "xcorr_region"), (1, 0, "xcorr_mfma"), (2, 0, "xcorr_dmaILi4"),
                                             (0, 2, None), (0, 5, None), (0, -1, None), (1, 3, None), (2, 1, None),
                                             (3, 0, None)])
def test_tune_file_entries_name_their_kernel(run, tmp_path, kernel, shape, ok):
    tune_file(tmp_path, 2, kernel, '"shape": %d, ' % shape)
    if ok:
        run(LOOKUP + "assert lookup(1500) == (%d, X.XENG_TUNE_CACHE_FILE) and launched(1500) == [%r]\n" % (kernel, ok))
    else:
        run(LOOKUP + "assert lookup(1500)[1] == X.XENG_TUNE_SETTINGS\n")
