"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, rejects bad
arguments before touching the GPU, and its scalar quantiser numerics (compiled from the same
header the kernels use) agree bit for bit with the oracle's."""
import ctypes as C
import os
import re
import sys

import numpy as np
import pytest
import torch

import kvtc_oracle as ko
import paper_2511_01815_amd as kv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    inc = os.path.join(ROOT, "include")
    headers = sorted(f for f in os.listdir(inc) if f.endswith(".h"))
    assert headers == ["kvtc.h", "kvtc_probe.h", "kvtc_test_hooks.h"]
    hdr = "\n".join(open(os.path.join(inc, f)).read() for f in headers)
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = sorted(set(re.findall(r"\b(kvtc_[a-z0-9_]+)\s*\(", hdr)))
    assert {"kvtc_plan_create", "kvtc_encode", "kvtc_decode", "kvtc_offsets", "kvtc_encode_batch",
            "kvtc_decode_batch", "kvtc_batch_create", "kvtc_last_error"} <= set(names)
    L = kv.lib()
    for n in names:
        assert hasattr(L, n), n


def _probe():
    rng = np.random.default_rng(2)
    tab = np.arange(65536, dtype=np.uint32).astype(np.uint16).view(np.float16)
    tab = tab[np.isfinite(tab)].astype(np.float32)
    xs = [rng.standard_normal(3000) * s for s in (1e-9, 1e-7, 3e-5, 1e-2, 1.0, 500.0, 8e4)]
    xs += [tab[::7], np.nextafter(tab[::11], np.float32(np.inf)), np.nextafter(tab[::13], np.float32(-np.inf))]
    xs.append(np.array([0.0, -0.0, 65504.0, -65504.0, 65519.9, 1e30, -1e30, np.inf, -np.inf, 5.9e-8, -2.9e-8, 2.98e-8]))
    return np.concatenate(xs).astype(np.float32)


def test_directed_fp16_rounding_matches_oracle_bits():
    L = kv.lib()
    x = _probe()
    want_dn = ko.fp16_floor(x).view(np.uint16)
    want_up = ko.fp16_ceil(x).view(np.uint16)
    got_dn = np.array([L.kvtc_host_f16_round_down(float(v)) for v in x], dtype=np.uint16)
    got_up = np.array([L.kvtc_host_f16_round_up(float(v)) for v in x], dtype=np.uint16)
    np.testing.assert_array_equal(got_dn, want_dn)
    np.testing.assert_array_equal(got_up, want_up)


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 6, 8, 11, 16])
def test_header_and_code_decision_match_oracle(bits):
    L = kv.lib()
    rng = np.random.default_rng(bits)
    d = (rng.standard_normal((400, 16)) * rng.choice([1e-6, 1e-3, 0.3, 5.0, 900.0], (400, 1))).astype(np.float32)
    d[:5] = d[:5, :1]                      # zero-range groups
    d[5, :] = [70000.0, -70000.0] + [1.0] * 14   # saturating
    shift, scale, codes = ko.quantise_group(d, bits)
    sh = C.c_uint16()
    sc = C.c_uint16()
    for t in range(d.shape[0]):
        L.kvtc_host_group_header(float(d[t].min()), float(d[t].max()), bits, C.byref(sh), C.byref(sc))
        assert sh.value == int(shift.view(np.uint16)[t]) and sc.value == int(scale.view(np.uint16)[t]), t
        got = [L.kvtc_host_code(float(v), sh.value, sc.value, bits) for v in d[t]]
        assert got == codes[t].tolist(), t


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_only_arrays_on_whole_cache_lines_pass_the_caches(dtype):
    """Base, row pitch and the gap between blocks: all multiples of 128 bytes, or a piece of a row is two parts of lines."""
    per_line = 64 if dtype == kv.KVTC_BF16 else 32
    base, eb = 1 << 40, 128 // per_line

    def whole(address, layout):
        return kv.lib().kvtc_host_whole_lines(address, dtype, 1024, C.byref(layout))

    for skip in (0, per_line // 8, per_line // 2, per_line, 3 * per_line):                   # elements; multiples of 16 bytes
        on = 1 if skip % per_line == 0 else 0
        assert whole(base + skip * eb, kv.layout(1024)) == on, skip
        assert whole(base, kv.layout(1024 + skip)) == on, skip
        assert whole(base, kv.layout(128 + skip, 128, 5000 * (128 + skip))) == on, skip      # heads-major, rows apart
        assert whole(base, kv.layout(128, 128, 5000 * 128 + skip)) == on, skip               # heads-major, heads apart
        assert whole(base, kv.layout(8 * (128 + skip), 128, 128 + skip)) == on, skip         # heads apart inside a token's row
    assert whole(base + 2, kv.layout(1024)) == -1 and whole(base, kv.layout(1000)) == -1


def test_output_passes_the_caches_where_that_was_measured_faster():
    """Light kernels -- few coordinates, or fp32 -- with the bases of a few plans store a few times the last-level cache's 256 MB through it; with many
    bases, or more matrix work than stores, they pass it by from about half of it."""
    MB, never = 1 << 20, (1 << 64) - 1

    def at(tiles, dtype, plans, single=False):
        return kv.lib().kvtc_host_decode_pass_bytes(tiles, dtype, plans * tiles * 32 * 1024 * 2, single)

    for tiles in (2, 4):
        assert at(tiles, kv.KVTC_BF16, 1, True) > 800 * MB and at(tiles, kv.KVTC_BF16, 2) > 800 * MB and at(tiles, kv.KVTC_BF16, 64) <= 256 * MB
        assert at(tiles, kv.KVTC_F32, 1, True) == at(tiles, kv.KVTC_F32, 2) == never and 300 * MB < at(tiles, kv.KVTC_F32, 64) <= 500 * MB
    assert at(6, kv.KVTC_BF16, 1, True) == 256 * MB and at(6, kv.KVTC_BF16, 2) <= 137 * MB
    for tiles in (6, 8, 10):
        assert at(tiles, kv.KVTC_F32, 1, True) > 1000 * MB and at(tiles, kv.KVTC_F32, 4) > 1000 * MB and at(tiles, kv.KVTC_F32, 64) <= 300 * MB
    for tiles, dtype in ((7, kv.KVTC_BF16), (10, kv.KVTC_BF16), (12, kv.KVTC_BF16), (12, kv.KVTC_F32), (32, kv.KVTC_F32)):
        for single in (False, True):
            assert 128 * MB < at(tiles, dtype, 1, single) <= 137 * MB


def test_input_passes_the_caches_where_that_was_measured_faster():
    """No sooner than the last-level cache's 256 MB; later where a variant's ring for whole lines is short, or the caches keep some of an input of a
    little more; never where a line is asked for at two times."""
    MB, never = 1 << 20, (1 << 64) - 1
    at = kv.lib().kvtc_host_encode_pass_bytes
    for tiles in (2, 8, 10, 12, 16, 20, 24, 32):
        assert at(tiles, kv.KVTC_BF16) == 256 * MB
    assert 325 * MB < at(4, kv.KVTC_BF16) <= 351 * MB and at(6, kv.KVTC_BF16) == never
    for tiles in (2, 4, 24, 32):
        assert at(tiles, kv.KVTC_F32) == 320 * MB
    for tiles in (6, 8, 10, 12, 16, 20):
        assert at(tiles, kv.KVTC_F32) == never


def test_argument_errors_need_no_gpu():
    L = kv.lib()
    p, r = 64, 16
    mu = np.zeros(p, dtype=np.float32)
    v = np.zeros((p, r), dtype=np.uint16)
    with pytest.raises(kv.KvtcError) as e:
        kv.kvtc_plan_create(60, 16, np.zeros(60, np.float32), np.zeros((60, 16), np.uint16), [(16, 4)], stream=0)
    assert e.value.status == 1 and "multiple of 64" in str(e.value)
    with pytest.raises(kv.KvtcError) as e:
        kv.kvtc_plan_create(p, r, mu, v, [(16, 17)], stream=0)
    assert e.value.status == 1
    with pytest.raises(kv.KvtcError) as e:
        kv.kvtc_plan_create(p, r, mu, v, [(16, 0)], stream=0)
    assert e.value.status == 1
    with pytest.raises(kv.KvtcError) as e:
        kv.kvtc_plan_create(p, 32, mu, np.zeros((p, 32), np.uint16), [(16, 4)], stream=0)
    assert e.value.status == 1 and "sum" in str(e.value)
    with pytest.raises(kv.KvtcError) as e:          # group of 1: valid format, not served by the kernels
        kv.kvtc_plan_create(p, 17, mu, np.zeros((p, 17), np.uint16), [(16, 4), (1, 8)], stream=0)
    assert e.value.status == 2
    with pytest.raises(kv.KvtcError) as e:          # record too large for on-chip staging
        kv.kvtc_plan_create(1024, 1024, np.zeros(1024, np.float32), np.zeros((1024, 1024), np.uint16),
                            [(16, 16)] * 64, stream=0)
    assert e.value.status == 2
    # null handles
    assert L.kvtc_record_bytes(None) == 0 and L.kvtc_encoded_bytes(None, 5) == 0
    L.kvtc_plan_destroy(None)
    L.kvtc_batch_destroy(None)
    assert L.kvtc_encode(None, None, 0, 1, 64, None, 0, None) == 1
    assert L.kvtc_decode(None, None, 0, 1, None, 0, 64, None) == 1
    assert "null plan" in kv.kvtc_last_error()
    out = C.c_void_p()
    assert L.kvtc_batch_create(C.byref(out), None, 0, None) == 1


def test_job_struct_layout():
    assert kv.JOB_DTYPE.itemsize == 16
    j = kv.make_jobs([0, 1], [5, 7], [0, 5])
    assert j.tobytes() == (b"\x00\x00\x00\x00\x05\x00\x00\x00" + (0).to_bytes(8, "little") +
                           b"\x01\x00\x00\x00\x07\x00\x00\x00" + (5).to_bytes(8, "little"))


# ---- sinks / sliding window (host-only entry points) ------------------------------------------

def test_window_split_equals_the_replay():
    import kvtc_window as kw
    for s, w, c in [(4, 128, 16), (0, 128, 16), (4, 64, 64), (1, 5, 2), (3, 7, 1), (16, 256, 32)]:
        for ctx in list(range(0, 3 * w + 2 * s + 9)) + [8192, 131072, 10**9 + 7][: (3 if c > 1 else 0)]:
            if ctx > 10**6:
                # the replay is linear in ctx: check the closed form's invariants instead
                n_sink, n_coded, n_window = kv.kvtc_window_split(ctx, s, w, c)
                assert n_sink == s and n_coded % c == 0 and w - c <= n_window < w and n_sink + n_coded + n_window == ctx
            else:
                assert kv.kvtc_window_split(ctx, s, w, c) == kw.window_split(ctx, s, w, c), (ctx, s, w, c)


def test_window_split_and_ratio_reject_and_agree():
    import kvtc_window as kw
    for bad in [(-1, 4, 128, 16), (10, -1, 128, 16), (10, 4, 8, 0), (10, 4, 8, 9)]:
        with pytest.raises(kv.KvtcError) as e:
            kv.kvtc_window_split(*bad)
        assert e.value.status == 1
    st = kv.lib().kvtc_window_split(10, 4, 128, 16, None)
    assert st == 1 and "null" in kv.kvtc_last_error()
    for ctx, w, s, cr in [(8192, 128, 4, 20.0), (1000, 112, 4, 16.0), (131072, 127, 0, 40.0), (300, 128, 4, 8.0)]:
        assert kv.kvtc_cr_with_window(ctx, w, s, cr) == pytest.approx(kw.cr_with_window(ctx, w, s, cr), rel=1e-15)


def test_fp8_entry_points_reject_bad_arguments_before_any_launch():
    L = kv.lib()
    buf = np.zeros(4096, dtype=np.uint8)
    ptr = buf.ctypes.data & ~15
    assert L.kvtc_fp8_pack(None, 0, 0, 1024, 1024, None, 0, None) == 0                 # nothing to do
    assert L.kvtc_fp8_pack(None, 0, 4, 1024, 1024, ptr, 4096, None) == 1               # null input
    assert L.kvtc_fp8_pack(ptr, 0, 4, 1024, 512, ptr, 4096, None) == 1                 # pitch below p
    assert L.kvtc_fp8_pack(ptr, 7, 4, 1024, 1024, ptr, 4096, None) == 1                # unknown dtype
    assert L.kvtc_fp8_pack(ptr + 2, 0, 4, 1024, 1024, ptr, 4096, None) == 1            # misaligned
    assert L.kvtc_fp8_pack(ptr, 0, 4, 1024, 1024, ptr, 4095, None) == 3                # output too small
    assert L.kvtc_fp8_unpack(ptr, 4095, 4, 1024, ptr, 0, 1024, None) == 3
    assert L.kvtc_fp8_unpack(ptr, 4096, -1, 1024, ptr, 0, 1024, None) == 1
    assert L.kvtc_offsets_append(None, None, 0, None, None, None, None) == 1


def test_rope_rejects_bad_arguments_before_any_launch():
    L = kv.lib()
    buf = np.zeros(4096, dtype=np.uint8)
    ptr = buf.ctypes.data & ~15
    ok = dict(dtype=0, T=4, H=8, d=128, ts=1024, hs=128)

    def call(x=ptr, dtype=0, T=4, H=8, d=128, ts=1024, hs=128, base=10000.0, pairing=0, inverse=0):
        return L.kvtc_rope(x, dtype, T, H, d, ts, hs, None, 0, base, pairing, inverse, None)

    assert call(x=None, T=0) == 0                      # nothing to do
    assert call(x=None) == 1                           # null buffer
    assert call(dtype=5) == 1
    assert call(d=127) == 1 and call(d=0) == 1 and call(d=258) == 1
    assert call(H=0) == 1
    assert call(ts=1023) == 1                          # a token's heads would run into the next token
    assert call(ts=128, hs=3 * 128) == 1               # heads-major, but a head's slab is shorter than its tokens
    assert call(base=0.0) == 1 and call(base=float("inf")) == 1
    assert call(pairing=2) == 1 and call(inverse=2) == 1
    assert call(T=-1) == 1
    assert "kvtc_rope" in kv.kvtc_last_error()
    del ok


def test_later_entry_points_reject_bad_arguments_before_any_launch():
    """Sectioned plans, the lossless stage and the calibration passes: every argument error below is found on the host,
    before any allocation or launch, so it needs no GPU."""
    L = kv.lib()
    h = C.c_void_p()
    mu = np.zeros(256, np.float32)
    V = np.zeros((256, 64), np.uint16)
    grp = (kv.binding._Group * 2)(kv.binding._Group(32, 4, 0), kv.binding._Group(16, 4, 0))      # sums to 48, not 64
    assert L.kvtc_wide_create(C.byref(h), 256, 64, mu.ctypes.data, V.ctypes.data, 2, C.cast(grp, C.c_void_p), None) == 1
    assert "sum to" in kv.kvtc_last_error()
    assert L.kvtc_wide_create(C.byref(h), 250, 64, mu.ctypes.data, V.ctypes.data, 2, C.cast(grp, C.c_void_p), None) == 1
    assert L.kvtc_wide_create(C.byref(h), 256, 64, None, V.ctypes.data, 2, C.cast(grp, C.c_void_p), None) == 1
    big = (kv.binding._Group * 1)(kv.binding._Group(2048, 4, 0))
    assert L.kvtc_wide_create(C.byref(h), 4096, 2048, mu.ctypes.data, V.ctypes.data, 1, C.cast(big, C.c_void_p), None) == 1
    assert L.kvtc_wide_sections(None) == 0 and L.kvtc_wide_record_bytes(None) == 0 and L.kvtc_wide_encoded_bytes(None, 5) == 0
    lay = kv.layout(256)
    assert L.kvtc_wide_encode(None, 16, 0, 4, C.byref(lay), 16, 64, None) == 1
    assert L.kvtc_wide_decode(None, 16, 64, 4, 16, 0, C.byref(lay), None, None) == 1
    # lossless stage
    good = np.full((8, 256), 8, dtype=np.uint8)
    assert L.kvtc_entropy_create(C.byref(h), 6, 1, good.ctypes.data, None) == 1
    assert L.kvtc_entropy_create(C.byref(h), 580, 1, good.ctypes.data, None) == 2
    assert L.kvtc_entropy_create(C.byref(h), 8, 0, good.ctypes.data, None) == 1
    assert L.kvtc_entropy_create(C.byref(h), 8, 1, None, None) == 1
    bad = good.copy()
    bad[1, :2] = 1
    assert L.kvtc_entropy_create(C.byref(h), 8, 1, bad.ctypes.data, None) == 1 and "prefix code" in kv.kvtc_last_error()
    assert L.kvtc_entropy_bound(None, 100) == 0
    assert L.kvtc_entropy_encode(None, 0, 16, 4, 16, 64, 16, None) == 1
    assert L.kvtc_entropy_decode(None, 0, 16, 64, 4, 16, 64, None) == 1
    assert L.kvtc_entropy_encode_batch(None, 16, 1, 4, 16, 64, 16, 64, 16, None) == 1
    assert L.kvtc_entropy_decode_batch(None, 16, 1, 4, 16, 64, 16, 64, None) == 1
    assert kv.ENTROPY_JOB_DTYPE.itemsize == 32
    # calibration passes
    assert L.kvtc_calib_block_errors(16, 4, 64, 16, 1, 9, 16, None) == 1
    assert L.kvtc_calib_block_errors(None, 4, 64, 16, 1, 8, 16, None) == 1
    assert L.kvtc_calib_block_errors(16, 4, 64, 16, 1, 8, 20, None) == 1          # output not 8-byte aligned
    assert L.kvtc_calib_block_errors(16, 4, 64, 16, 0, 8, 16, None) == 0          # no blocks: nothing to do
    assert L.kvtc_calib_moments(16, 0, 4, 100, C.byref(lay), 16, 16, None) == 1
    assert L.kvtc_calib_moments(16, 0, 4, 256, None, 16, 16, None) == 1
    assert L.kvtc_calib_moments(16, 0, 4, 256, C.byref(kv.layout(128)), 16, 16, None) == 1
    assert L.kvtc_calib_moments(16, 0, 4, 256, C.byref(lay), 16, 20, None) == 1


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr and r.stdout.strip() == ""


def _trace_of(fn, of_code, seen):
    """Runs fn with `seen` called before every line of, and at every exception in, the Python frames whose code is of_code."""
    def local(frame, event, arg):
        seen(event)
        return local

    old = sys.gettrace()
    sys.settrace(lambda frame, event, arg: local if frame.f_code is of_code else None)
    try:
        return fn()
    finally:
        sys.settrace(old)


def test_a_second_thread_finds_the_current_stream_at_any_moment_of_the_first_ones_search(monkeypatch):
    """The first call looks up torch's calls for the current stream; whatever line of it another thread's call comes in at must not matter."""
    from paper_2511_01815_amd import binding
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    monkeypatch.setattr(binding, "_current_stream", binding._first_current_stream)
    first, others = binding._current_stream, []
    found = set(vars(binding))

    def other_thread(event):
        if event == "line":
            before = {k: v for k, v in vars(binding).items() if k in found}
            others.append(binding._current_stream())                 # (untraced: a trace function is not traced itself)
            vars(binding).update(before)                             # (what it found is its own: the first call goes on from where it was)

    assert _trace_of(first, first.__code__, other_thread) == 73
    assert len(others) >= 4 and set(others) == {73}
    assert binding._current_stream() == 73


def test_a_forked_child_asks_torch_before_it_uses_the_gpu(monkeypatch):
    """A child of a process that has made calls must hear torch's refusal, not use a stream of its parent's GPU."""
    from paper_2511_01815_amd import binding
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    monkeypatch.setattr(binding, "_current_stream", binding._first_current_stream)
    assert binding._current_stream() == 73

    def refuse():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")

    monkeypatch.setattr(torch.cuda, "current_device", refuse)
    assert binding._current_stream() == 73
    child = os.fork()
    if child == 0:
        try:
            binding._current_stream()
            os._exit(1)
        except RuntimeError:
            os._exit(0)
        finally:
            os._exit(2)
    assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 0
    assert binding._current_stream() == 73


def test_addresses_of_every_kind_and_no_exception_for_a_plain_integer():
    from paper_2511_01815_amd import binding
    array, tensor, events = np.zeros(3), torch.zeros(3), []
    assert binding._ptr(array) == array.ctypes.data and binding._ptr(tensor) == tensor.data_ptr() and binding._ptr(True) is True
    for t in (1 << 40, 0, None):
        assert _trace_of(lambda: binding._ptr(t), binding._ptr.__code__, events.append) is t
    assert "line" in events and "exception" not in events
    for t in ("address", 1.5, np.int64(8)):
        with pytest.raises(AttributeError):
            binding._ptr(t)


@pytest.mark.skipif(torch.cuda.is_available(), reason="the device has room for the tables")
def test_entropy_tables_are_asked_for_without_the_staged_decoders_before_they_are_refused():
    """The staged decoder's tables, as much again as all others, are left out where they do not fit; what is refused is the memory that records cannot do without."""
    R = 64
    with pytest.raises(kv.KvtcError) as e:
        kv.kvtc_entropy_create(R, np.full((R, 256), 8, dtype=np.uint8), stream=0)
    codes, decoder, limits, lengths = 512, 256 + 256 + 16, 16, 256
    assert f"hipMalloc of {R * (codes + decoder + limits + lengths)} bytes failed" in str(e.value)
