"""The lossless stage where its launches change shape: records of one and of two table segments with whole and partial store
batches, code tables that fit the LDS and that do not, workgroups of every number of waves, launches whose waves take several
chunks each, jobs that read their tables from global memory, and code lengths at both ends of what a table may hold.
Containers must equal the oracle's byte for byte."""
import numpy as np
import pytest
import torch

import kvtc_entropy as ke
import paper_2511_01815_amd as kv
from test_gpu_entropy import DEV, _gpu_decode, _gpu_encode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,T", [(64, 65), (100, 1), (144, 200), (148, 130), (212, 64), (264, 129), (268, 129), (272, 129), (4, 525_000), (12, 263_000)])
def test_container_at_the_edges_of_the_launch_shapes(R, T):
    """264 bytes: the largest record whose code table fits the LDS.  T = 525 000: 8204 chunks, on 256 compute units a few more than
    there are waves on the chip (8192 in encode); 263 000: 4110 chunks, all at once."""
    rng = np.random.default_rng(R + T)
    rec = np.stack([np.minimum(255, rng.geometric(1.0 / (1.2 + (11 * k) % 120), T) - 1) for k in range(R)], axis=1).astype(np.uint8)
    lengths = ke.calibrate_tables(rec[:4096])
    tab = kv.EntropyTables(R, lengths)
    ref = ke.encode(rec, lengths)
    out, n, bound = _gpu_encode(tab, rec)
    assert n == len(ref) and out[:n].tobytes() == ref
    assert np.all(out[bound:] == 0xA5)
    assert np.array_equal(_gpu_decode(tab, ref, T, R), rec)
    tab.close()


@pytest.mark.parametrize("kind", ["all 12", "all 10", "one of 1", "9 to 12"])
def test_code_lengths_at_the_limits(kind):
    """All codes of 12 bits or of 10 (the sum of Kraft's inequality far below one), a code of one bit among long ones, and no
    code of 8 bits or less."""
    R, T = 8, 700
    L = np.full(256, 12, dtype=np.uint8)
    if kind == "all 10":
        L[:] = 10
    if kind == "one of 1":
        L[7] = 1
    if kind == "9 to 12":
        L[:64], L[64:128], L[128:192] = 9, 10, 11
    lengths = np.tile(L, (R, 1))
    rec = np.random.default_rng(5).integers(0, 256, (T, R)).astype(np.uint8)
    rec[::3] = 7
    tab = kv.EntropyTables(R, lengths)
    ref = ke.encode(rec, lengths)
    out, n, _ = _gpu_encode(tab, rec)
    assert n == len(ref) and out[:n].tobytes() == ref
    assert np.array_equal(_gpu_decode(tab, ref, T, R), rec)
    tab.close()


def _check_batch(R, lens, period):
    """A batch whose job j codes tensor j % period (its first lens[j] tokens; lens repeats with the period too) with table set j % 2
    against the oracle's containers, and back."""
    n, rng = len(lens), np.random.default_rng(R + len(lens))
    assert period % 2 == 0 and all(lens[j] == lens[j % period] for j in range(n))
    recs = [np.stack([np.minimum(255, rng.geometric(1.0 / (1.2 + (11 * k + 17 * i) % 120), lens[i]) - 1) for k in range(R)], axis=1).astype(np.uint8)
            for i in range(period)]
    sample = np.concatenate(recs)[:4096]
    tables = np.stack([ke.calibrate_tables(sample), ke.calibrate_tables(sample[:300])])
    refs = [np.frombuffer(ke.encode(r, tables[i % 2]), dtype=np.uint8) for i, r in enumerate(recs)]
    tab = kv.EntropyTables(R, tables)
    rec_at = np.concatenate([[0], np.cumsum([v * R for v in lens])]).tolist()
    caps = [ke.bound_bytes(v, R) for v in lens]
    cod_at = np.concatenate([[0], np.cumsum(caps)]).tolist()
    dev = torch.from_numpy(np.concatenate([r.reshape(-1) for r in recs])).to(DEV).repeat(n // period + 1)[:rec_at[-1]]
    coded = torch.full((cod_at[-1] + 64,), 0xA5, dtype=torch.uint8, device=DEV)
    sizes = torch.zeros(n, dtype=torch.int64, device=DEV)

    def jobs(room):
        return torch.from_numpy(kv.make_entropy_jobs([j % 2 for j in range(n)], lens, rec_at[:-1], cod_at[:-1], room).view(np.uint8)).to(DEV)

    kv.kvtc_entropy_encode_batch(tab.handle, jobs(caps), n, max(lens), dev, dev.numel(), coded, cod_at[-1], sizes)
    torch.cuda.synchronize()
    assert sizes.cpu().tolist() == [len(refs[j % period]) for j in range(n)]
    want = [torch.from_numpy(r.copy()).to(DEV) for r in refs]
    for j in range(n):
        assert torch.equal(coded[cod_at[j]:cod_at[j] + len(refs[j % period])], want[j % period]), j
    assert bool((coded[cod_at[-1]:] == 0xA5).all())
    back = torch.full((dev.numel() + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    kv.kvtc_entropy_decode_batch(tab.handle, jobs([len(refs[j % period]) for j in range(n)]), n, max(lens), coded, cod_at[-1], back, dev.numel())
    torch.cuda.synchronize()
    assert torch.equal(back[:dev.numel()], dev) and bool((back[dev.numel():] == 0x5A).all())
    tab.close()


@pytest.mark.parametrize("chunks", [16, 20, 30, 45, 60, 70, 256])
def test_workgroups_of_every_size_and_waves_of_several_chunks(chunks):
    """64 tensors of 128-byte records.  Decode has one workgroup on each of 256 compute units: 4, 6, 8, 12 and 16 waves in turn, then
    more workgroups than places, and with 256 chunks per tensor waves that take four chunks (strings four, sizes two)."""
    _check_batch(128, [64 * chunks, 64 * chunks - 17] * 32, 2)


@pytest.mark.parametrize("R,n_jobs", [(128, 600), (148, 600), (36, 1400)])
@pytest.mark.parametrize("most", [64, 150, 250])
def test_many_tensors_of_a_few_chunks(R, n_jobs, most):
    """More jobs than places: up to two chunks the strings are coded from tables in global memory, up to four the records decoded."""
    lens = np.random.default_rng(most).integers(1, most + 1, 10).tolist()
    lens[3], lens[5] = most, max(1, most - 64)
    _check_batch(R, [lens[j % 10] for j in range(n_jobs)], 10)


@pytest.mark.parametrize("R,n_jobs,most", [(8, 40, 130), (12, 40, 130), (12, 300, 130), (16, 300, 130), (36, 260, 385), (36, 260, 449), (36, 260, 833), (64, 300, 321), (200, 300, 130)])
def test_both_sides_of_what_the_staged_decoder_takes(R, n_jobs, most):
    """Records of less than 16 bytes in few jobs and in more than there are compute units; jobs of 7, 8 and 14 chunks of which the staged decoder runs one round of
    workgroups and two; records too long for it, and strings from tables in global memory, in more jobs than compute units."""
    lens = [most, 1, max(1, most - 64), most, 65, most - 1]
    _check_batch(R, [lens[j % 6] for j in range(n_jobs)], 6)


@pytest.mark.parametrize("R,T", [(128, 262_100), (200, 172_101), (256, 140_000), (576, 62_300), (576, 123_000)])
def test_strings_read_a_piece_at_a_time(R, T):
    """One long tensor whose records, of one to four table segments, do not fit the L2s of 256 compute units, in one round and in two, and short
    ones of the same launch, whose payloads are a few dwords or end in a chunk of few tokens."""
    lens = [T, 1, 2, 63, 64, 65, 129, 200]
    n = len(lens)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R)
    mean = 1.2 + (11 * torch.arange(R, device=DEV)) % 120
    rec = torch.cat([torch.zeros((m, R), device=DEV).exponential_(generator=gen).mul_(mean).clamp_(max=255).to(torch.uint8).view(-1) for m in lens])
    tab = kv.EntropyTables(R, ke.calibrate_tables(rec[:4096 * R].view(-1, R).cpu().numpy()))
    rec_at = np.concatenate([[0], np.cumsum([m * R for m in lens])]).tolist()
    caps = [ke.bound_bytes(m, R) for m in lens]
    cod_at = np.concatenate([[0], np.cumsum(caps)]).tolist()
    coded = torch.zeros(cod_at[-1], dtype=torch.uint8, device=DEV)
    sizes = torch.zeros(n, dtype=torch.int64, device=DEV)

    def jobs(room):
        return torch.from_numpy(kv.make_entropy_jobs([0] * n, lens, rec_at[:-1], cod_at[:-1], room).view(np.uint8)).to(DEV)

    kv.kvtc_entropy_encode_batch(tab.handle, jobs(caps), n, T, rec, rec.numel(), coded, cod_at[-1], sizes)
    torch.cuda.synchronize()
    back = torch.full((rec.numel() + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    kv.kvtc_entropy_decode_batch(tab.handle, jobs(sizes.cpu().tolist()), n, T, coded, cod_at[-1], back, rec.numel())
    torch.cuda.synchronize()
    assert torch.equal(back[:rec.numel()], rec) and bool((back[rec.numel():] == 0x5A).all())
    tab.close()


@pytest.mark.parametrize("R,T", [(100, 300), (576, 62_300)])
def test_damaged_container_stays_inside_its_buffers(R, T):
    """Random token lengths (up to 65535 bits, far behind a short payload), random chunk offsets and a payload cut short: the records are wrong,
    but nothing else is written, and the tensor decoded beside it is right.  The second size reads a piece at a time."""
    rng = np.random.default_rng(R)
    rec = np.stack([np.minimum(255, rng.geometric(1.0 / (1.2 + (11 * k) % 120), 2048) - 1) for k in range(R)], axis=1).astype(np.uint8)
    lengths = ke.calibrate_tables(rec)
    tab = kv.EntropyTables(R, lengths)
    good = np.frombuffer(ke.encode(rec[:130], lengths), dtype=np.uint8)
    n_chunks = (T + 63) // 64
    for payload in (0, 4, 24, 4000):
        offs = rng.integers(0, 2 ** 32, n_chunks + 1, dtype=np.uint64).astype(np.uint32)
        offs[::3] = rng.integers(0, payload + 8, len(offs[::3]))
        bits = rng.integers(0, 65536, 64 * n_chunks).astype(np.uint16)
        bad = np.concatenate([offs.view(np.uint8), bits.view(np.uint8), rng.integers(0, 256, payload).astype(np.uint8)])
        blob = torch.from_numpy(np.concatenate([bad, good])).to(DEV)
        back = torch.full((T * R + 130 * R + 64,), 0x5A, dtype=torch.uint8, device=DEV)
        jobs = kv.make_entropy_jobs([0, 0], [T, 130], [0, T * R], [0, len(bad)], [len(bad), len(good)])
        kv.kvtc_entropy_decode_batch(tab.handle, torch.from_numpy(jobs.view(np.uint8)).to(DEV), 2, T, blob, blob.numel(), back, T * R + 130 * R)
        torch.cuda.synchronize()
        assert np.array_equal(back[T * R:T * R + 130 * R].cpu().numpy().reshape(130, R), rec[:130]), payload
        assert bool((back[T * R + 130 * R:] == 0x5A).all()), payload
    tab.close()
