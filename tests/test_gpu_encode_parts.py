"""Small calls whose tiles' groups are shared out over workgroups, against the bulk kernels: the same bits.  Shares that begin and end inside a
coordinate tile, a dword and a halfword pair of the record, codes of more than 8 bits, many groups, plans of more coordinates than the
short-job kernel takes, one group alone (one share of ten tiles), groups that are too many tiles (no shares); tiles of 1, 31, 32 and 33
tokens, a saturated group in a share beside others, appends between regions that must stay as they are."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_encode_short import bulk_tokens, short_tokens
from test_gpu_parity import DEV, _gpu_plan, _manual

pytestmark = pytest.mark.gpu

PLANS = {"odd blocks": [(16, 3), (48, 5), (16, 1), (80, 7), (16, 2), (96, 3)], "wide codes": [(16, 16), (48, 9), (64, 12), (16, 1)], "small groups": [(16, 1 + k % 7) for k in range(40)],
         "wide plan": [(64, 5), (112, 4), (48, 3)] * 4, "one group": [(320, 3)], "too wide a group": [(336, 2), (16, 4)]}


@pytest.mark.parametrize("name", sorted(PLANS))
@pytest.mark.parametrize("p,dtype", [(1024, kv.KVTC_BF16), (320, kv.KVTC_F32), (1088, kv.KVTC_BF16), (1152, kv.KVTC_F32)])
def test_shares_of_groups_are_coded_as_whole_tiles(name, p, dtype):
    """1152 features in fp32 are the most of which the LDS holds 32 tokens."""
    groups = PLANS[name]
    if sum(n for n, _ in groups) > p:
        pytest.skip("more coordinates than features")
    plan = _gpu_plan(_manual(p, groups, 5))
    R, n_bulk = plan.record_bytes, bulk_tokens()
    gen = torch.Generator(device=DEV).manual_seed(p)
    x = torch.randn((200, p), generator=gen, device=DEV)
    x[40] *= 3e4                                                     # scales of 65504: every code is clamped
    x = x.to(torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32)
    rows = x.repeat(n_bulk // 200 + 1, 1)[:n_bulk]
    bulk = torch.zeros((n_bulk, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, rows, dtype, n_bulk, p, bulk, bulk.numel())
    bulk = bulk[:200]
    for n in (1, 31, 32, 33, 97):
        got = torch.full((n * R + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, x, dtype, n, p, got, n * R)
        torch.cuda.synchronize()
        assert torch.equal(got[:n * R].view(n, R), bulk[:n]), n
        assert bool((got[n * R:] == 0xA5).all()), n
    # appends of 1, 16 and 33 tokens, each between records that a region holds and room that it has left; one without room
    lens, before = [1, 16, 33, 5], [2, 0, 7, 60]
    jobs = torch.from_numpy(kv.make_jobs([0] * 4, lens, [3, 30, 100, 0]).view(np.uint8)).to(DEV)
    region = torch.arange(5, dtype=torch.int64, device=DEV) * (64 * R + 16 - 64 * R % 16)
    coded = torch.tensor(before, dtype=torch.int64, device=DEV)
    offs = torch.zeros(5, dtype=torch.int64, device=DEV)
    out = torch.full((int(region[-1].item()) + 64,), 0xA5, dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    batch = kv.Batch([plan])
    kv.kvtc_offsets_append(batch.handle, jobs, 4, region, coded, offs)
    kv.kvtc_encode_batch(batch.handle, jobs, 4, x, dtype, p, offs, out, out.numel() - 64, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 4
    want = torch.full_like(out, 0xA5)
    for n, row, b, at in list(zip(lens, [3, 30, 100, 0], before, region.tolist()))[:3]:
        want[at + b * R:at + (b + n) * R] = bulk[row:row + n].reshape(-1)
    assert torch.equal(out, want)
    batch.close()
    plan.close()


@pytest.mark.parametrize("p", [64, 128, 192, 256, 320, 448, 512, 576, 1536])
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_features_on_both_sides_of_what_is_fetched_ahead(p, dtype):
    """8, 16 and 32 k-steps of 16 features ahead: fewer steps than that, as many, and rounds of the main loop that end with less than a whole one."""
    plan = _gpu_plan(_manual(p, [(16, 6), (32, 3), (16, 2)], p))
    R, n_bulk = plan.record_bytes, bulk_tokens()
    x = torch.randn((70, p), generator=torch.Generator(device=DEV).manual_seed(p), device=DEV).to(torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32)
    rows = x.repeat(n_bulk // 70 + 1, 1)[:n_bulk].contiguous()
    bulk = torch.zeros((n_bulk, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, rows, dtype, n_bulk, p, bulk, bulk.numel())
    batch = kv.Batch([plan])
    for n in (1, 32, 70):
        got = torch.zeros((n, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, x, dtype, n, p, got, got.numel())
        jobs = torch.from_numpy(kv.make_jobs([0, 0], [n, 17], [0, 50]).view(np.uint8)).to(DEV)
        offs = torch.zeros(3, dtype=torch.int64, device=DEV)
        out = torch.zeros((n + 17, R), dtype=torch.uint8, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtc_offsets(batch.handle, jobs, 2, offs)
        kv.kvtc_encode_batch(batch.handle, jobs, 2, x, dtype, p, offs, out, out.numel(), status)
        torch.cuda.synchronize()
        assert torch.equal(got, bulk[:n]) and int(status.item()) == 0, n
        assert torch.equal(out, torch.cat([bulk[:n], bulk[50:67]])), n
    batch.close()
    plan.close()


@pytest.mark.parametrize("dtype,jobs_of,lens,room", [
    (kv.KVTC_BF16, 4, [16], 4), (kv.KVTC_BF16, 4, [17, 0, 33, 5], 4),                     # room for 64 tokens a job: a share for every compute unit, and fewer
    (kv.KVTC_BF16, 4, [48], 1), (kv.KVTC_BF16, 4, [100, 20, 64, 1], 1),                   # no room left: more shares than run at once
    (kv.KVTC_F32, 16, [40, 7, 64, 1], 4), (kv.KVTC_F32, 16, [97, 129], 1), (kv.KVTC_BF16, 2, [40, 64], 1),      # (the last: of the plan of one share)
])
@pytest.mark.parametrize("groups", [[(16, 8), (16, 6), (80, 4), (64, 3), (64, 2)], [(16, 8), (32, 6), (64, 4), (96, 3), (64, 2)], [(16, 8), (96, 5), (144, 3), (16, 2)], [(16, 6), (80, 3)]])
def test_small_batches_whose_form_the_jobs_lengths_decide(dtype, jobs_of, lens, room, groups):
    """Batches that may be more shares than run at once: the kernel that counts them, on both sides of its line, in a buffer of just their records
    and in a roomy one, and as a job more or fewer for the launches on either side of it; two, three and one coordinate tile to a wave of the short jobs'
    form (plans of 8 and 10 tiles with shares of up to four, one with a share of five, and one of a single share).  The bulk kernels' bits."""
    p = 1024
    plan = _gpu_plan(_manual(p, groups, 9))
    R, n_bulk = plan.record_bytes, bulk_tokens()
    x = torch.randn((400, p), generator=torch.Generator(device=DEV).manual_seed(room), device=DEV).to(torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32)
    rows = x.repeat(n_bulk // 400 + 1, 1)[:n_bulk].contiguous()
    bulk = torch.zeros((n_bulk, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, rows, dtype, n_bulk, p, bulk, bulk.numel())
    batch = kv.Batch([plan])
    most = torch.cuda.get_device_properties(0).multi_processor_count // jobs_of
    for n_jobs in (most, most - 1, most + 1, most // 3):
        ns = [lens[j % len(lens)] for j in range(n_jobs)]
        row0 = [(37 * j) % (400 - max(lens)) for j in range(n_jobs)]
        jobs = torch.from_numpy(kv.make_jobs([0] * n_jobs, ns, row0).view(np.uint8)).to(DEV)
        offs = torch.zeros(n_jobs + 1, dtype=torch.int64, device=DEV)
        size = sum(ns) * R
        out = torch.full((room * size + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtc_offsets(batch.handle, jobs, n_jobs, offs)
        kv.kvtc_encode_batch(batch.handle, jobs, n_jobs, x, dtype, p, offs, out, room * size, status)
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and torch.equal(out[:size].view(-1, R), torch.cat([bulk[a:a + n] for a, n in zip(row0, ns)])), n_jobs
        assert bool((out[size:] == 0xA5).all()), n_jobs
    batch.close()
    plan.close()


@pytest.mark.parametrize("r", [528, 560, 592, 608, 640])
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_bulk_plans_of_17_to_20_tiles_leave_the_padding_out(r, dtype):
    """Whole tiles and a half, shared out over four waves as 5 and 4: the bits of a call of 130 tokens, which is coded by parts, and of one that is too long for
    that and not for the short-job kernel."""
    plan = _gpu_plan(_manual(1024, [(16, 8), (r - 144, 3), (128, 2)], r))
    R, n_bulk = plan.record_bytes, bulk_tokens()
    x = torch.randn((130, 1024), generator=torch.Generator(device=DEV).manual_seed(r), device=DEV).to(torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32)
    want = torch.zeros((130, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, x, dtype, 130, 1024, want, want.numel())
    rows = x.repeat(n_bulk // 130 + 1, 1)[:n_bulk].contiguous()
    got = torch.zeros((n_bulk, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, rows, dtype, n_bulk, 1024, got, got.numel())
    torch.cuda.synchronize()
    assert torch.equal(got, want.repeat(n_bulk // 130 + 1, 1)[:n_bulk])
    n_short = short_tokens() + 33
    got = torch.zeros((n_short, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, rows, dtype, n_short, 1024, got, got.numel())
    torch.cuda.synchronize()
    assert torch.equal(got, want.repeat(n_short // 130 + 1, 1)[:n_short])
    plan.close()


@pytest.mark.parametrize("p,dtype", [(1216, kv.KVTC_F32), (2560, kv.KVTC_BF16)])
def test_more_features_than_the_lds_holds_of_32_tokens_are_not_shared_out(p, dtype):
    """Groups that can be shared out, of a plan too wide for it: alone, and in a batch beside a plan that is not (no job of which may be coded by parts then)."""
    groups = PLANS["wide codes"]
    narrow = {kv.KVTC_F32: 1152, kv.KVTC_BF16: 1024}[dtype]
    plans = [_gpu_plan(_manual(p, groups, 6)), _gpu_plan(_manual(narrow, groups, 7))]
    n_bulk = bulk_tokens()
    x = torch.randn((100, p), generator=torch.Generator(device=DEV).manual_seed(p), device=DEV).to(torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32)
    rows, bulk = x.repeat(n_bulk // 100 + 1, 1)[:n_bulk].contiguous(), []
    for plan in plans:
        out = torch.zeros((n_bulk, plan.record_bytes), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, rows, dtype, n_bulk, p, out, out.numel())
        bulk.append(out[:100])
    for plan, want in zip(plans, bulk):
        for n in (1, 32, 97):
            got = torch.zeros((n, plan.record_bytes), dtype=torch.uint8, device=DEV)
            kv.kvtc_encode(plan.handle, x, dtype, n, p, got, got.numel())
            torch.cuda.synchronize()
            assert torch.equal(got, want[:n]), n
    batch = kv.Batch(plans)
    which, ns, row0 = [0, 1, 1, 0], [16, 16, 33, 5], [0, 20, 40, 90]
    jobs = torch.from_numpy(kv.make_jobs(which, ns, row0).view(np.uint8)).to(DEV)
    offs = torch.zeros(5, dtype=torch.int64, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = torch.zeros(sum(n * plans[w].record_bytes for n, w in zip(ns, which)), dtype=torch.uint8, device=DEV)
    kv.kvtc_offsets(batch.handle, jobs, 4, offs)
    kv.kvtc_encode_batch(batch.handle, jobs, 4, x, dtype, p, offs, out, out.numel(), status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and torch.equal(out, torch.cat([bulk[w][a:a + n].reshape(-1) for w, n, a in zip(which, ns, row0)]))
    batch.close()
    for plan in plans:
        plan.close()
