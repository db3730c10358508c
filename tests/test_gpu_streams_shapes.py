"""What goes past the caches in the shapes that one contiguous tensor does not have: feature counts whose slabs end in the middle of the rings' common
period, rows with a pitch, heads apart in memory, batches of ragged jobs, fp32, and the kernels whose outputs pass the caches only with many bases or from
a gigabyte on.  The same bits as in calls of a part of the tokens each, which the caches keep."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _gpu_plan, _manual, _variant_plan

pytestmark = pytest.mark.gpu


def _plan(p, r):
    """r coordinates of p features: 16-coordinate groups of several widths in front, wider groups of 3 bits behind."""
    front = [(16, 7), (16, 5), (16, 8), (16, 4)]
    groups, left = [], r
    while left:
        n, b = front[len(groups)] if len(groups) < 4 else (min(64, left), 3)
        groups.append((min(n, left), b))
        left -= min(n, left)
    return _gpu_plan(_manual(p, groups, p + r))


def _tiles(r):
    return next(t for t in (2, 4, 6, 8, 10, 12, 16, 20, 24, 32) if 32 * t >= r)


def _type(dtype):
    return (torch.bfloat16, 2) if dtype == kv.KVTC_BF16 else (torch.float32, 4)


def _layout(shape, T, p, dtype):
    """(elements, kvtc_layout, view of them as [T][p] or [blocks][T][features])"""
    tdt, _ = _type(dtype)
    if shape == "pitch":                                          # whole lines between the rows' ends
        buf = torch.full((T, p + 64), 7.0, dtype=tdt, device=DEV)
        return buf, kv.layout(p + 64), buf[:, :p]
    if shape == "heads":                                          # heads of 64 features, with whole lines between them
        buf = torch.full((p // 64, T + 2, 64), 7.0, dtype=tdt, device=DEV)
        return buf, kv.layout(64, 64, (T + 2) * 64), buf[:, :T].permute(1, 0, 2)
    buf = torch.full((T, p), 7.0, dtype=tdt, device=DEV)
    return buf, kv.layout(p), buf


def _fill(view, p, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    for t0 in range(0, view.shape[0], 65536):
        n = min(65536, view.shape[0] - t0)
        view[t0:t0 + n] = torch.randn((n, p), generator=gen, device=DEV).reshape(view[t0:t0 + n].shape)


def _parts(T, n):
    return [(t0, min(n, T - t0)) for t0 in range(0, T, n)]


@pytest.mark.parametrize("p,r,dtype,shape", [(320, 48, kv.KVTC_BF16, "pitch"), (320, 128, kv.KVTC_BF16, "plain"), (320, 224, kv.KVTC_BF16, "heads"), (320, 240, kv.KVTC_BF16, "pitch"),
                                             (320, 304, kv.KVTC_BF16, "plain"), (448, 416, kv.KVTC_BF16, "heads"), (960, 112, kv.KVTC_BF16, "heads"),
                                             (960, 256, kv.KVTC_BF16, "plain"), (960, 288, kv.KVTC_BF16, "heads"), (960, 272, kv.KVTC_BF16, "pitch"),
                                             (960, 528, kv.KVTC_BF16, "pitch"), (832, 704, kv.KVTC_BF16, "heads"), (1024, 736, kv.KVTC_F32, "pitch"),
                                             (1024, 1024, kv.KVTC_F32, "heads"), (960, 96, kv.KVTC_F32, "heads"), (320, 32, kv.KVTC_F32, "pitch")])
def test_large_inputs_of_any_shape_are_coded_as_small_ones(p, r, dtype, shape):
    plan, (_, eb) = _plan(p, r), _type(dtype)
    R = plan.record_bytes
    T = kv.lib().kvtc_host_encode_pass_bytes(_tiles(r), dtype) // (p * eb) + 79
    buf, lay, x = _layout(shape, T, p, dtype)
    _fill(x, p, r)
    assert kv.lib().kvtc_host_whole_lines(buf.data_ptr(), dtype, p, lay) == 1
    got = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode_blocked(plan.handle, buf, dtype, T, lay, got, got.numel())
    for t0, n in _parts(T, 50021):
        part = x[t0:t0 + n].reshape(n, p).contiguous()
        want = torch.zeros((n, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, part, dtype, n, p, want, want.numel())
        assert torch.equal(got[t0:t0 + n], want), t0


@pytest.mark.parametrize("r,dtype", [(64, kv.KVTC_BF16), (128, kv.KVTC_BF16), (224, kv.KVTC_BF16), (240, kv.KVTC_BF16), (304, kv.KVTC_BF16), (384, kv.KVTC_BF16), (800, kv.KVTC_BF16),
                                     (64, kv.KVTC_F32), (1024, kv.KVTC_F32)])
def test_large_batches_of_ragged_jobs(r, dtype):
    """Jobs of a token, of a tile and one more, of many tiles; encode and decode against calls of a job each.  64 plans, so that every decode kernel's
    output of this size passes the caches."""
    p, (tdt, eb) = 1024, _type(dtype)
    plan = _gpu_plan(_variant_plan(r))
    R = plan.record_bytes
    batch = kv.Batch([plan] * 64)
    least = max(kv.lib().kvtc_host_encode_pass_bytes(_tiles(r), dtype), kv.lib().kvtc_host_decode_pass_bytes(_tiles(r), dtype, 64 * 2 * p * r, 0))
    lens = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 20011, 5000, 31, 1]
    lens += [7777] * ((least // (p * eb) + 99 - sum(lens)) // 7777 + 1)
    row0 = [int(v) for v in np.concatenate([[0], np.cumsum(lens)[:-1]])]
    T, n = sum(lens), len(lens)
    x = torch.empty((T, p), dtype=tdt, device=DEV)
    _fill(x, p, r)
    jobs = torch.from_numpy(kv.make_jobs([j % 64 for j in range(n)], lens, row0).view(np.uint8)).to(DEV)
    offs = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    status = torch.zeros(2, dtype=torch.int32, device=DEV)
    rec = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_offsets(batch.handle, jobs, n, offs)
    kv.kvtc_encode_batch(batch.handle, jobs, n, x, dtype, p, offs, rec, rec.numel(), status[0:1])
    got = torch.full((T + 1, p), 7.0, dtype=tdt, device=DEV)
    kv.kvtc_decode_batch(batch.handle, jobs, n, rec, rec.numel(), offs, got, dtype, p, status[1:2])
    assert status.tolist() == [0, 0] and bool((got[T] == 7.0).all())
    for j in range(n):
        a, b = row0[j], row0[j] + lens[j]
        want = torch.zeros((lens[j], R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, x[a:b], dtype, lens[j], p, want, want.numel())
        assert torch.equal(rec[a:b], want), j
        back = torch.empty((lens[j], p), dtype=tdt, device=DEV)
        kv.kvtc_decode(plan.handle, want, want.numel(), lens[j], back, dtype, p)
        assert torch.equal(got[a:b], back), j


@pytest.mark.parametrize("p,r,dtype,shape", [(1024, 64, kv.KVTC_BF16, "heads"), (1024, 128, kv.KVTC_BF16, "pitch"), (320, 160, kv.KVTC_BF16, "heads"), (960, 240, kv.KVTC_BF16, "heads"),
                                             (1024, 304, kv.KVTC_BF16, "heads"), (960, 480, kv.KVTC_BF16, "heads"), (1024, 1024, kv.KVTC_BF16, "heads"),
                                             (1024, 160, kv.KVTC_F32, "pitch"), (960, 240, kv.KVTC_F32, "heads"), (1024, 480, kv.KVTC_F32, "heads"),
                                             (960, 800, kv.KVTC_F32, "pitch")])
def test_large_outputs_of_any_shape_hold_what_small_ones_hold(p, r, dtype, shape):
    plan, (tdt, eb) = _plan(p, r), _type(dtype)
    R = plan.record_bytes
    T = kv.lib().kvtc_host_decode_pass_bytes(_tiles(r), dtype, 2 * p * r, 1) // (p * eb) + 79
    some = torch.empty((20011, p), dtype=tdt, device=DEV)
    _fill(some, p, r)
    rec = torch.zeros((20011, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, some, dtype, 20011, p, rec, rec.numel())
    want = torch.empty((20011, p), dtype=tdt, device=DEV)
    kv.kvtc_decode(plan.handle, rec, rec.numel(), 20011, want, dtype, p)
    stream = rec.repeat(T // 20011 + 1, 1)[:T].contiguous()
    buf, lay, out = _layout(shape, T, p, dtype)
    kv.kvtc_decode_blocked(plan.handle, stream, stream.numel(), T, buf, dtype, lay)
    for t0, n in _parts(T, 20011):
        assert torch.equal(out[t0:t0 + n].reshape(n, p), want[:n]), t0
    gaps = buf[:, p:] if shape == "pitch" else buf[:, T:]
    assert bool((gaps == 7.0).all())
