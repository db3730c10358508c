"""The encode kernel for short jobs against the bulk kernels: the same bits, for plans of every width class, token counts around
its tiles, feature counts with and without a part of a chunk left over, both input types and a heads-major layout.  And the
bulk kernels against each other in those types and layouts, at token counts that only they code."""
import numpy as np
import pytest
import torch

import paper_2511_01815_amd as kv
from test_gpu_parity import DEV, VARIANT_RANKS, _from_dev, _gpu_plan, _manual, _variant_plan, check_stream

pytestmark = pytest.mark.gpu


def bulk_tokens():
    """Tokens of a tensor, or of a lone job, that the bulk kernels code whatever its plan and type: more 64-token tiles than two for
    every compute unit, the most that the short-job kernel is given."""
    return 2 * 64 * torch.cuda.get_device_properties(0).multi_processor_count + 200


def short_tokens():
    """Tokens of a tensor that the short-job kernel codes whatever its plan (of up to 640 coordinates) and type, with up to 64 times the compute units less
    this more: more shares of 32-token tiles than one and a half for every compute unit, the most that are coded by parts, and no more 64-token tiles than compute units."""
    return 48 * torch.cuda.get_device_properties(0).multi_processor_count + 64


WIDE = {64: [(32, 4)], 192: [(16, 8), (64, 4), (16, 2)], 320: [(64, 5), (96, 3)], 448: [(128, 5), (128, 3)], 1024: [(16, 8), (64, 5), (128, 3), (112, 2)],
        1088: [(64, 6), (256, 3), (64, 2)], 1152: [(256, 4), (240, 3)], 2048: [(64, 12), (512, 3), (64, 2)], 832: [(256, 3), (512, 1)]}


@pytest.mark.parametrize("p", sorted(WIDE))
@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
def test_short_jobs_are_coded_as_long_ones(p, dtype):
    """Single calls of up to 200 tokens and the batch of 16 jobs go by parts where the plan's groups can be shared out and X fits the LDS (not of 2048 features in fp32);
    the single calls of short_tokens() and more, with last tiles of 1, 31, 32, 33 and 63 tokens, are the short-job kernel's, and so are the batches of more jobs
    than compute units have places for by parts."""
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

    base, n_bulk = x, bulk_tokens()
    x = base.repeat(n_bulk // T + 1, 1)                          # (read by coded())
    bulk, _ = coded([0], [n_bulk], [0])
    bulk = bulk.view(n_bulk, R)
    assert torch.equal(bulk[T:], bulk[:-T])
    x, bulk = base, bulk[:T]
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
    for n_jobs in (150, 300):                                    # (300: of plans of up to 256 coordinates)
        which, ns, at = [j % 2 for j in range(n_jobs)], [lens[j // 2 % 7] for j in range(n_jobs)], [row0[j // 2 % 7] for j in range(n_jobs)]
        out, offs = coded(which, ns, at)
        for j in range(0, n_jobs, 2):
            assert torch.equal(out[offs[j]:offs[j] + ns[j] * R].view(ns[j], R), bulk[at[j]:at[j] + ns[j]]), (p, n_jobs, j)
    longer = base.repeat((short_tokens() + 63) // T + 1, 1)
    for n in (short_tokens() + k for k in (1, 31, 32, 33, 63)):
        got = torch.zeros((n, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, longer, dtype, n, p, got, got.numel())
        torch.cuda.synchronize()
        assert torch.equal(got, bulk.repeat(n // T + 1, 1)[:n]), (p, n, "longer call")
    if p % 64 == 0 and p > 64:
        heads = x.view(T, p // 64, 64).permute(1, 0, 2).contiguous()
        got = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode_blocked(plan.handle, heads, dtype, T, kv.layout(64, 64, T * 64), got, got.numel())
        torch.cuda.synchronize()
        assert torch.equal(got, bulk), (p, "heads-major")


@pytest.mark.parametrize("r", VARIANT_RANKS)
def test_bulk_kernels_code_the_same_bits_from_every_type_and_layout(r):
    """A tensor that no call gives to the short-job kernel: bf16 rows on sampled tokens against the oracle; the same values in
    fp32, with a row pitch, heads-major and as jobs of a batch beside shorter ones must give the same records."""
    oplan = _variant_plan(r)
    plan = _gpu_plan(oplan)
    p, R, T = 1024, plan.record_bytes, bulk_tokens()
    mix = torch.from_numpy((np.arange(1, p + 1, dtype=np.float64)[:, None] ** -0.7 * np.linalg.qr(np.random.default_rng(77).standard_normal((p, p)))[0]).astype(np.float32))
    x = (torch.randn((T, p), generator=torch.Generator(device=DEV).manual_seed(r), device=DEV) @ mix.to(DEV) + 0.05).to(torch.bfloat16)
    ref = torch.zeros((T, R), dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, x, kv.KVTC_BF16, T, p, ref, ref.numel())
    rows = np.unique(np.concatenate([[0, 63, 64, 127, 128, 191, 192, 255, 256, T - 2, T - 1], np.random.default_rng(r).integers(0, T, size=400)]))
    idx = torch.from_numpy(rows).to(DEV)
    check_stream(oplan, _from_dev(x.index_select(0, idx)), ref.index_select(0, idx).cpu().numpy(), f"bulk{r}")
    batch = kv.Batch([plan])
    lens = [300, T - 500, 5, 70]
    row0 = [0, 300, T - 200, T - 195]
    jobs = torch.from_numpy(kv.make_jobs([0] * 4, lens, row0).view(np.uint8)).to(DEV)
    offs = torch.zeros(5, dtype=torch.int64, device=DEV)
    kv.kvtc_offsets(batch.handle, jobs, 4, offs)
    want = torch.cat([ref[a:a + n] for a, n in zip(row0, lens)])
    assert T - 500 > bulk_tokens() // 4 + 64                     # beyond what one of four jobs may have on the short-job kernel
    for dtype in (kv.KVTC_BF16, kv.KVTC_F32):
        xd = x if dtype == kv.KVTC_BF16 else x.float()
        pitched = torch.full((T, p + 72), float("nan"), dtype=xd.dtype, device=DEV)
        pitched[:, :p] = xd
        heads = xd.view(T, p // 128, 128).permute(1, 0, 2).contiguous()
        for name, src, lay in (("plain", xd, kv.layout(p)), ("pitch", pitched, kv.layout(p + 72)), ("heads-major", heads, kv.layout(128, 128, T * 128))):
            got = torch.full((T * R + 64,), 0xA5, dtype=torch.uint8, device=DEV)
            kv.kvtc_encode_blocked(plan.handle, src, dtype, T, lay, got, T * R)
            status = torch.zeros(1, dtype=torch.int32, device=DEV)
            out = torch.full((want.numel() + 64,), 0xA5, dtype=torch.uint8, device=DEV)
            kv.kvtc_encode_batch_blocked(batch.handle, jobs, 4, src, dtype, lay, offs, out, want.numel(), status)
            torch.cuda.synchronize()
            assert int(status.item()) == 0
            assert torch.equal(got[:T * R].view(T, R), ref) and bool((got[T * R:] == 0xA5).all()), (name, dtype)
            assert torch.equal(out[:want.numel()].view(-1, R), want) and bool((out[want.numel():] == 0xA5).all()), (name, dtype, "batch")


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("form", ["batch", "static"])
def test_batches_with_jobs_on_both_sides_of_the_limit(form, dtype):
    """Jobs that fit the short-job kernel go to it unless a longer job needs their plan's bulk kernel anyway and has room for them: batches
    in which that is so for no plan, for one and for all, in which the bulk kernel's round of tiles is full, with plans that have
    no short-job kernel and jobs that are not valid (those are skipped and the lowest is reported).  Whatever the route, a job's records are those of its single call."""
    plans = [_gpu_plan(_variant_plan(r)) for r in (64, 192, 544, 1024)]
    batch, p = kv.Batch(plans), 1024
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    limit = cus // 11 * 64                                       # the batches below have 11 jobs, one wide plan among them
    rows = max(2 * limit, cus * 128)
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    x = torch.randn((rows, p), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV).to(tdt)
    single = []
    for plan in plans:
        out = torch.zeros((rows, plan.record_bytes), dtype=torch.uint8, device=DEV)
        kv.kvtc_encode(plan.handle, x, dtype, rows, p, out, out.numel())
        single.append(out)
    small = [(0, limit), (0, 3), (1, 200), (1, 64), (2, 65), (2, limit - 1), (3, 200), (3, 5)]
    none = small + [(1, 0), (0, 64), (2, 1)]
    one = small + [(1, limit + 1), (0, 64), (2, 1)]
    all_ = small + [(1, 2 * limit), (0, limit + 64), (2, limit + 1)]
    full = small + [(1, 2 * limit), (0, 64), (2, cus * 128)]     # one round of the 640-coordinate kernel's 128-token tiles
    invalid = [(0, 500), (9, 3 * limit), (-1, 70), (1, -5), (1, limit)] + small[2:]
    for jobs in (none, one, all_, full, invalid):
        assert len(jobs) == 11
        which, lens = [w for w, _ in jobs], [n for _, n in jobs]
        row0 = [(37 * j) % max(1, rows - n + 1) if n > 0 else 0 for j, n in enumerate(lens)]
        ok = [0 <= w < 4 and n >= 0 for w, n in jobs]
        size = sum(n * plans[w].record_bytes for (w, n), v in zip(jobs, ok) if v)
        dev = torch.from_numpy(kv.make_jobs(which, lens, row0).view(np.uint8)).to(DEV)
        offs = torch.zeros(12, dtype=torch.int64, device=DEV)
        out = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        if form == "batch":
            kv.kvtc_offsets(batch.handle, dev, 11, offs)
            kv.kvtc_encode_batch(batch.handle, dev, 11, x, dtype, p, offs, out, size, status)
        else:
            kv.kvtc_encode_batch_static([q.handle for q in plans], dev, 11, x, dtype, p, out, size, offs, status)
        torch.cuda.synchronize()
        assert int(status.item()) == (0 if all(ok) else 1 + ok.index(False))
        assert bool((out[size:] == 0xA5).all())
        at = offs.cpu().tolist()
        for j, (w, n) in enumerate(jobs):
            if ok[j]:
                got = out[at[j]:at[j] + n * plans[w].record_bytes].view(n, plans[w].record_bytes)
                assert torch.equal(got, single[w][row0[j]:row0[j] + n]), (j, w, n)


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("ranks", [(64, 192, 240), (192, 544)])
@pytest.mark.parametrize("form", ["batch", "static"])
def test_small_batches_are_coded_by_one_launch(form, ranks, dtype):
    """A stream buffer that can hold only a few tiles of records sends the whole batch to the short-job kernel, a larger one sends the
    same jobs through the bulk kernels: the same bytes and the same status, for jobs of one to many tiles, empty, not valid and beyond
    the buffer, in lists of less and more than a wave's lanes, up to the most that one round takes."""
    plans = [_gpu_plan(_variant_plan(r)) for r in ranks]
    batch, p = kv.Batch(plans), 1024
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    rows = 64 * cus
    x = torch.randn((rows, p), generator=torch.Generator(device=DEV).manual_seed(9), device=DEV).to(tdt)
    rng = np.random.default_rng(len(ranks))
    k = len(plans)
    lists = [[(0, 1)], [(k - 1, 64 * cus // 4)], [(j % k, 16) for j in range(64)], [(j % k, int(rng.integers(0, 130))) for j in range(65)],
             [(j % k, int(n)) for j, n in enumerate(rng.integers(0, 40, size=190))],
             [(0, 65), (7, 40), (1, -3), (-1, 200), (1, 700), (0, 0), (1, 64)]]
    for jobs in lists:
        n_jobs = len(jobs)
        which, lens = [w for w, _ in jobs], [n for _, n in jobs]
        row0 = [(101 * j) % max(1, rows - n + 1) if n > 0 else 0 for j, n in enumerate(lens)]
        dev = torch.from_numpy(kv.make_jobs(which, lens, row0).view(np.uint8)).to(DEV)
        ok = [0 <= w < k and n >= 0 for w, n in jobs]
        size = sum(n * plans[w].record_bytes for (w, n), v in zip(jobs, ok) if v)
        for short_by in (0, 4):                                  # the last job that codes anything does not fit
            got = []
            for room in (0, 16 << 20):
                out = torch.full((size + room + 64,), 0xA5, dtype=torch.uint8, device=DEV)
                offs = torch.zeros(n_jobs + 1, dtype=torch.int64, device=DEV)
                status = torch.zeros(1, dtype=torch.int32, device=DEV)
                cap = size + room
                if form == "batch":
                    kv.kvtc_offsets(batch.handle, dev, n_jobs, offs)
                    if short_by:
                        last = max(j for j in range(n_jobs) if ok[j] and lens[j] > 0)
                        offs[last] = cap - lens[last] * plans[which[last]].record_bytes + short_by
                    kv.kvtc_encode_batch(batch.handle, dev, n_jobs, x, dtype, p, offs, out, cap, status)
                else:
                    kv.kvtc_encode_batch_static([q.handle for q in plans], dev, n_jobs, x, dtype, p, out, cap - short_by if room == 0 else cap, offs, status)
                torch.cuda.synchronize()
                assert bool((out[cap:] == 0xA5).all())
                got.append((out, int(status.item())))
            (a, sa), (b, sb) = got
            if short_by == 0:
                assert torch.equal(a[:size], b[:size]) and sa == sb == (0 if all(ok) else 1 + ok.index(False)), (jobs[:8], sa, sb)
            else:
                last = max(j for j in range(n_jobs) if ok[j] and lens[j] > 0)
                n = lens[last] * plans[which[last]].record_bytes
                bad = min([last] + [j for j in range(n_jobs) if not ok[j]])
                assert sa == 1 + bad and torch.equal(a[:size - n], b[:size - n]) and bool((a[size - n:] == 0xA5).all()), (jobs[:8], sa)


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("layout", ["pitched", "heads-major"])
def test_small_batches_of_long_lists_and_other_layouts(layout, dtype):
    """Lists of up to the most jobs that one launch takes, with jobs at both ends of each 64 that a wave looks at together and empty ones between:
    the bytes of the bulk kernels, which a larger buffer gets."""
    plans = [_gpu_plan(_variant_plan(r)) for r in (64, 192, 240)]
    batch, p, block = kv.Batch(plans), 1024, 128
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tdt = torch.bfloat16 if dtype == kv.KVTC_BF16 else torch.float32
    rows = 700
    x = torch.randn((rows, p), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV).to(tdt)
    if layout == "pitched":
        buf = torch.zeros((rows, p + 64), dtype=tdt, device=DEV)
        buf[:, :p] = x
        lay = kv.layout(p + 64)
    else:
        buf, lay = x.view(rows, p // block, block).transpose(0, 1).contiguous(), kv.layout(block, block, rows * block)
    for n_jobs in (64, 65, 256, 257, 449, min(512, 2 * cus - 24)):
        lens = np.zeros(n_jobs, dtype=int)
        lens[[0, 63] + [j for j in (64, 127, 255, 256, 319, 447, 448) if j < n_jobs] + [n_jobs - 1]] = 5
        lens[n_jobs // 2] = 70
        which, row0 = [j % 3 for j in range(n_jobs)], [(29 * j) % (rows - 70) for j in range(n_jobs)]
        dev = torch.from_numpy(kv.make_jobs(which, lens.tolist(), row0).view(np.uint8)).to(DEV)
        size = sum(int(n) * plans[w].record_bytes for w, n in zip(which, lens))
        got = []
        for room in (0, 16 << 20):
            out = torch.full((size + room + 64,), 0xA5, dtype=torch.uint8, device=DEV)
            offs = torch.zeros(n_jobs + 1, dtype=torch.int64, device=DEV)
            status = torch.zeros(1, dtype=torch.int32, device=DEV)
            kv.kvtc_offsets(batch.handle, dev, n_jobs, offs)
            kv.kvtc_encode_batch_blocked(batch.handle, dev, n_jobs, buf, dtype, lay, offs, out, size + room, status)
            torch.cuda.synchronize()
            assert int(status.item()) == 0 and bool((out[size:] == 0xA5).all())
            got.append(out[:size])
        assert torch.equal(*got), n_jobs
