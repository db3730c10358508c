"""Batched decode of few tokens.  A stream buffer that can hold only a round of 128-token tiles sends the batch to the variant with
one token tile per wave, a larger one sends the same jobs to 256-token tiles: the same bits, the same status."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, _gpu_plan, _variant_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("ranks", [(64,), (64, 192, 240), (192, 544)])
def test_small_batches_decode_to_the_same_bits(ranks, dtype):
    plans = [_gpu_plan(_variant_plan(r)) for r in ranks]
    batch, p, k = kv.Batch(plans), 1024, len(plans)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    rows = 128 * cus
    x = torch.randn((rows, p), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV).to(tdt)
    rng = np.random.default_rng(k)
    # a token, the edges of both tiles, many jobs with empty ones, one that is not valid, and about the most that one round takes
    lists = [[(0, 1)], [(j % k, n) for j, n in enumerate([127, 128, 129, 255, 256, 257, 0, 300])], [(j % k, int(rng.integers(0, 140))) for j in range(70)],
             [(0, 65), (k, 40), (k - 1, -3), (0, 200)], [(k - 1, 128 * cus // 2 - 5)], [(k - 1, 128 * cus)]]
    for jobs in lists:
        n_jobs = len(jobs)
        which, lens = [w for w, _ in jobs], [n for _, n in jobs]
        ok = [0 <= w < k and n >= 0 for w, n in jobs]
        at = np.concatenate([[0], np.cumsum([n if v else 0 for n, v in zip(lens, ok)])]).tolist()       # each job's first row
        size = sum(n * plans[w].record_bytes for (w, n), v in zip(jobs, ok) if v)
        dev = torch.from_numpy(kv.make_jobs(which, lens, at[:-1]).view(np.uint8)).to(DEV)
        offs = torch.zeros(n_jobs + 1, dtype=torch.int64, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        room = 128 * 4 * cus * max(q.record_bytes for q in plans)
        buf = torch.zeros(size + room, dtype=torch.uint8, device=DEV)
        kv.kvtc_offsets(batch.handle, dev, n_jobs, offs)
        kv.kvtc_encode_batch(batch.handle, dev, n_jobs, x, dtype, p, offs, buf, size, status)
        got = []
        for in_bytes in (size, size + room):
            y = torch.full((rows + 1, p), -7.0, dtype=tdt, device=DEV)
            status.zero_()
            kv.kvtc_decode_batch(batch.handle, dev, n_jobs, buf, in_bytes, offs, y, dtype, p, status)
            torch.cuda.synchronize()
            assert int(status.item()) == (0 if all(ok) else 1 + ok.index(False))
            assert bool((y[at[-1]:] == -7.0).all()) and not bool((y[:at[-1]] == -7.0).all(dim=1).any())
            got.append(y)
        assert torch.equal(*got), (jobs[:8], (got[0].float() - got[1].float()).abs().max().item())
