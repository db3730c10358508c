"""Decode of plans of more than 320 coordinates: every width the kernels distinguish, token counts around their tiles, launches
whose workgroups share a tile's features and launches with several tiles per workgroup, feature counts that deal unevenly to
the waves, codes of more than 8 bits.  Held to the oracle once per plan; the output must not depend on the size of the call."""
import pytest
import torch

import kvtc_oracle as ko
import numpy as np
import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _from_dev, _gpu_plan, _manual, check_recon

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,groups", [(384, [(336, 3)]), (448, [(64, 5), (336, 2)]), (576, [(16, 12), (64, 6), (400, 2)]), (1024, [(64, 5), (496, 3)]),
                                      (640, [(64, 4), (528, 2)]), (704, [(256, 4), (432, 2)]), (1088, [(16, 9), (64, 5), (700 + 4, 2)]),
                                      (896, [(64, 6), (832, 2)]), (1088, [(64, 6), (960, 3)])])
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_wide_plans_at_the_edges_of_the_tiles(p, groups, dtype):
    oplan = _manual(p, groups, 70 + p % 9)
    plan = _gpu_plan(oplan)
    R, T = plan.record_bytes, 64 * 1200
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    g = torch.Generator(device=DEV)
    g.manual_seed(p)
    base = torch.randn((1200, p), generator=g, device=DEV).to(tdt)
    rec = torch.zeros((1200, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, base, dtype, 1200, p, rec, rec.numel())
    stream = rec.repeat(T // 1200, 1)                      # more tiles than twice the compute units
    whole = torch.full((T, p), 7.0, dtype=tdt, device=DEV)
    kv.kvtc_decode(plan.handle, stream, stream.numel(), T, whole, dtype, p)
    torch.cuda.synchronize()
    check_recon(oplan, rec[:200].cpu().numpy(), _from_dev(whole[:200]), ko.bf16_round(_from_dev(base[:200])), dtype == kv.KVTC_BF16, f"wide-{p}")
    assert torch.equal(whole[1200:], whole[:-1200])
    batch = kv.Batch([plan])
    for n in (1, 31, 63, 64, 65, 127, 129, 1000, 9000):
        got = torch.full((n + 1, p), 7.0, dtype=tdt, device=DEV)
        kv.kvtc_decode(plan.handle, stream, n * R, n, got, dtype, p)
        again = torch.full((n + 1, p), 7.0, dtype=tdt, device=DEV)
        jobs = torch.from_numpy(kv.make_jobs([0], [n], [0]).view(np.uint8)).to(DEV)
        offs = torch.tensor([0, n * R], dtype=torch.int64, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtc_decode_batch(batch.handle, jobs, 1, stream, n * R, offs, again, dtype, p, status)
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        for out in (got, again):
            assert torch.equal(out[:n], whole[:n]) and bool((out[n:] == 7.0).all()), (p, n)
