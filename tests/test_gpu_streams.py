"""Tensors beyond the last-level cache, which encode reads and decode stores past the caches from a size on that depends on the kernel
(kvtc_host_encode_pass_bytes, kvtc_host_decode_pass_bytes; the outputs here of plans of up to 4 tiles, of one tensor of 5 and 6, and in fp32 of up to
10, stay in the caches: test_gpu_streams_shapes.py has those beyond).  The same bits as in calls of a part of the tokens each."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _gpu_plan, _manual, _variant_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [64, 160, 224, 240, 272, 480, 1024])
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_large_outputs_hold_what_small_ones_hold(r, dtype):
    plan = _gpu_plan(_variant_plan(r))
    p, R, T, ld = 1024, plan.record_bytes, 70001, 1088
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    x = torch.randn((T, p), generator=torch.Generator(device=DEV).manual_seed(r), device=DEV)
    rec = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, x, kv.KVTC_F32, T, p, rec, rec.numel())
    del x
    want = torch.empty((T, p), dtype=tdt, device=DEV)
    for t0 in range(0, T, 14000):
        n = min(14000, T - t0)
        part = rec[t0:t0 + n].clone()                            # (a tile's records start where they start in a call of their own)
        kv.kvtc_decode(plan.handle, part, part.numel(), n, want[t0:], dtype, p)
    got = torch.full((T + 1, ld), 7.0, dtype=tdt, device=DEV)
    kv.kvtc_decode(plan.handle, rec, rec.numel(), T, got, dtype, ld)
    assert torch.equal(got[:T, :p], want) and bool((got[:, p:] == 7.0).all()) and bool((got[T] == 7.0).all())
    lens = [30000, 1, 255, 39745]
    jobs = torch.from_numpy(kv.make_jobs([0] * 4, lens, [0, 30000, 30001, 30256]).view(np.uint8)).to(DEV)
    offs = torch.zeros(5, dtype=torch.int64, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    batch = kv.Batch([plan])
    got.fill_(7.0)
    kv.kvtc_offsets(batch.handle, jobs, 4, offs)
    kv.kvtc_decode_batch(batch.handle, jobs, 4, rec, rec.numel(), offs, got, dtype, ld, status)
    assert int(status.item()) == 0
    assert torch.equal(got[:T, :p], want) and bool((got[:, p:] == 7.0).all()) and bool((got[T] == 7.0).all())


@pytest.mark.parametrize("r,dtype", [(r, kv.KVTC_BF16) for r in (64, 128, 192, 224, 256, 272, 304, 384, 512, 544, 736, 768, 800, 1024)] +
                         [(r, kv.KVTC_F32) for r in (32, 64, 96, 128)])
def test_large_inputs_are_coded_as_small_ones(r, dtype):
    plan = _gpu_plan(_variant_plan(r) if r >= 64 else _manual(1024, [(16, 4)] * (r // 16), 100 + r))
    p, R, T = 1024, plan.record_bytes, (131072 if dtype == kv.KVTC_BF16 else 81920) + 77      # 256 (fp32: 320) MB and some
    x = torch.randn((T, p), generator=torch.Generator(device=DEV).manual_seed(r), device=DEV)
    x = x.to(torch.bfloat16) if dtype == kv.KVTC_BF16 else x
    got = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, x, dtype, T, p, got, got.numel())
    part = torch.zeros((20001, R), dtype=torch.uint8, device=DEV)
    for t0 in range(0, T, 20001):
        n = min(20001, T - t0)
        kv.kvtc_encode(plan.handle, x[t0:], dtype, n, p, part, part.numel())
        assert torch.equal(got[t0:t0 + n], part[:n]), (r, t0)


def test_a_batch_counts_its_jobs_tokens():
    """Not whole tiles, not one launch's jobs alone, and no job that is not valid: plans of two variants and of two numbers of features, jobs of a
    token more than a tile."""
    plans = [_gpu_plan(_variant_plan(64)), _gpu_plan(_variant_plan(272)), kv.Plan(128, 16, np.zeros(128, np.float32), np.zeros((128, 16), np.uint16), [(16, 4)])]
    p = [1024, 1024, 128]
    batch = kv.Batch(plans)
    which = [j % 3 for j in range(300)] + [7, -1, 0, 1]
    lens = [129 + 64 * (j % 5) for j in range(300)] + [500, 500, -1, 1 << 30]                   # unknown plans, negative, beyond the stream buffer
    jobs = torch.from_numpy(kv.make_jobs(which, lens, [0] * len(lens)).view(np.uint8)).to(DEV)
    elements = sum(n * p[w] for n, w in zip(lens[:300], which))
    offs = torch.zeros(len(lens) + 1, dtype=torch.int64, device=DEV)
    out = torch.full((1,), 9, dtype=torch.int32, device=DEV)
    for at, passes in ((elements, 1), (elements // 2, 1), (elements * 101 // 100, 0), (1 << 60, 0)):
        st = kv.lib().kvtc_test_batch_passes(batch.handle, jobs.data_ptr(), len(lens), offs.data_ptr(), 1 << 22, at, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert st == 0 and int(out.item()) == passes, at
