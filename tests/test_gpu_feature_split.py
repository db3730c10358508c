"""Decode of few tiles, whose features are shared out among workgroups: feature counts of one span, of fewer and of more spans
than workgroups per tile, token counts from one to where every tile has a workgroup to itself again.  A token's features are
independent, so the output must not depend on the split: rows decoded in calls of other sizes must be the same bits, and
they are held to the oracle once."""
import numpy as np
import pytest
import torch

import kvtc_oracle as ko
import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _from_dev, _gpu_plan, _manual, check_recon

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,groups", [(64, [(16, 5), (32, 3)]), (192, [(16, 8), (64, 4), (16, 2)]), (1024, [(16, 8), (64, 5), (64, 3), (64, 2), (16, 2)]),
                                      (1024, [(64, 6), (256, 4), (256, 3), (16, 2)]), (4096, [(64, 4), (64, 2)])])
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_split_sweep_gives_the_bits_of_a_whole_sweep(p, groups, dtype):
    oplan = _manual(p, groups, 60 + p % 7)
    plan = _gpu_plan(oplan)
    R, T = plan.record_bytes, 66000
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    g = torch.Generator(device=DEV)
    g.manual_seed(p)
    base = torch.randn((1200, p), generator=g, device=DEV).to(tdt)
    rec = torch.zeros((1200, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, base, dtype, 1200, p, rec, rec.numel())
    stream = rec.repeat(T // 1200, 1)                      # 66000 records: more than one tile for every two workgroup slots, so no tile is shared
    whole = torch.full((T, p), 7.0, dtype=tdt, device=DEV)
    kv.kvtc_decode(plan.handle, stream, stream.numel(), T, whole, dtype, p)
    torch.cuda.synchronize()
    h = _from_dev(whole[:200])
    check_recon(oplan, rec[:200].cpu().numpy(), h, ko.bf16_round(_from_dev(base[:200])), dtype == kv.KVTC_BF16, f"split-{p}")
    batch = kv.Batch([plan])
    for n in (1, 31, 128, 129, 1000, 4097, 20000, 33000):
        got = torch.full((n, p), 7.0, dtype=tdt, device=DEV)
        kv.kvtc_decode(plan.handle, stream, n * R, n, got, dtype, p)
        again = torch.full((n, p), 7.0, dtype=tdt, device=DEV)
        jobs = torch.from_numpy(kv.make_jobs([0], [n], [0]).view(np.uint8)).to(DEV)
        offs = torch.tensor([0, n * R], dtype=torch.int64, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtc_decode_batch(batch.handle, jobs, 1, stream, n * R, offs, again, dtype, p, status)
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        assert torch.equal(got, whole[:n]), (p, n, "single call")
        assert torch.equal(again, whole[:n]), (p, n, "batch of one")
