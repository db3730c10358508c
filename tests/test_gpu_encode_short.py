"""The encode kernel for short jobs against the bulk kernels: the same bits, for plans of every width class, token counts around
its tiles, feature counts with and without a part of a chunk left over, both input types and a heads-major layout."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _gpu_plan, _manual

pytestmark = pytest.mark.gpu

WIDE = {64: [(32, 4)], 192: [(16, 8), (64, 4), (16, 2)], 320: [(64, 5), (96, 3)], 448: [(128, 5), (128, 3)], 1024: [(16, 8), (64, 5), (128, 3), (112, 2)],
        1088: [(64, 6), (256, 3), (64, 2)], 1152: [(256, 4), (240, 3)], 2048: [(64, 12), (512, 3), (64, 2)], 832: [(256, 3), (512, 1)]}


@pytest.mark.parametrize("p", sorted(WIDE))
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_short_jobs_are_coded_as_long_ones(p, dtype):
    plan = _gpu_plan(_manual(p, WIDE[p], 11))
    other = _gpu_plan(_manual(p, [(16, 6)], 12))                 # a narrow plan in the same launch
    R, T = plan.record_bytes, 200
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    g = torch.Generator(device=DEV)
    g.manual_seed(p)
    x = torch.randn((T, p), generator=g, device=DEV).to(tdt)
    batch = kv.Batch([plan, other])

    def coded(which, lens, row0):
        jobs = torch.from_numpy(kv.make_jobs(which, lens, row0).view(np.uint8)).to(DEV)
        size = sum(n * (plan, other)[w].record_bytes for w, n in zip(which, lens))
        offs = torch.zeros(len(lens) + 1, dtype=torch.int64, device=DEV)
        out = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtc_offsets(batch.handle, jobs, len(lens), offs)
        kv.kvtc_encode_batch(batch.handle, jobs, len(lens), x, dtype, p, offs, out, size, status)
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and bool((out[size:] == 0xA5).all())
        return out[:size], offs.cpu().tolist()

    bulk, _ = coded([0], [T], [0])
    bulk = bulk.view(T, R)
    lens = [1, 16, 31, 32, 33, 63, 64, 0]
    row0 = [0, 5, 100, 168, 7, 137, 64, 0]
    out, offs = coded([0, 1] * len(lens), [n for n in lens for _ in (0, 1)], [r for r in row0 for _ in (0, 1)])
    for k, (n, r) in enumerate(zip(lens, row0)):
        got = out[offs[2 * k]:offs[2 * k] + n * R].view(n, R)
        assert torch.equal(got, bulk[r:r + n]), (p, n)
    for n in (1, 32, 64, 65, 129, T):                            # single calls run tile by tile
        got = torch.zeros((n, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, x, dtype, n, p, got, got.numel())
        torch.cuda.synchronize()
        assert torch.equal(got, bulk[:n]), (p, n, "single call")
    if p % 64 == 0 and p > 64:
        heads = x.view(T, p // 64, 64).permute(1, 0, 2).contiguous()
        got = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode_blocked(plan.handle, heads, dtype, T, kv.layout(64, 64, T * 64), got, got.numel())
        torch.cuda.synchronize()
        assert torch.equal(got, bulk), (p, "heads-major")
