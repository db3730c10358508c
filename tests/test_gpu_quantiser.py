"""Headers and codes at the edges of fp16 and of every width, bit for bit: with unit columns for a basis and no mean a coefficient IS
its feature, so the records of chosen features are known without a tolerance."""
import numpy as np
import pytest
import torch

import kvtc_oracle as ko
import paper_2511_01815_amd as kv
import test_gpu_encode_short as es
from test_gpu_encode_short import bulk_tokens, short_tokens
from test_gpu_parity import DEV, _gpu_plan

pytestmark = pytest.mark.gpu


def _rows(n, p):
    """Tokens whose values span fp16's normal, subnormal and saturated ranges (bf16 numbers, no -0, nothing bf16 cannot hold as a normal)."""
    rng = np.random.default_rng(41)
    x = rng.standard_normal((n, p)) * 10.0 ** rng.uniform(-9, 6, (n, 1))
    x[::7] = np.abs(x[::7])                                      # shift above zero
    x[1::7] = -np.abs(x[1::7])
    x[2::7] += 10.0 ** rng.uniform(-3, 5, (len(x[2::7]), 1))     # a narrow range far from zero
    x[3::35, :] = x[3::35, :1]                                   # a range of nothing
    x[8::35, 5] = 3e38                                           # one value beyond any scale
    x[13::35, 2] = -3e38
    x[18::35] = np.where(rng.random((len(x[18::35]), p)) < 0.5, 65504.0, -70000.0)
    x[23::35] *= 1e30
    x[28::35] = rng.integers(0, 256, (len(x[28::35]), p)) * 0.5  # ties of the code's rounding
    return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).float().numpy() + 0.0


@pytest.mark.parametrize("groups", [[(16, 1), (16, 2), (16, 3), (16, 4)], [(16, 5), (16, 6), (16, 7), (16, 8)], [(32, 8), (32, 8)], [(16, 8), (48, 3)],
                                    [(16, 9), (16, 10), (16, 11), (16, 12)], [(16, 13), (16, 14), (16, 15), (16, 16)], [(48, 4), (16, 13)]])
def test_records_of_known_coefficients(groups):
    p, T = 64, bulk_tokens()
    blocks, at = [], 0
    for n, b in groups:
        blocks.append(ko.Block(at, n, b))
        at += n
    oplan = ko.compile_plan(np.zeros(p), np.eye(p), blocks)
    plan = _gpu_plan(oplan)
    n = 1400
    x = _rows(n, p)
    x[-1, 3] = np.nan                                            # every product with it: a token of nothing but NaN
    with np.errstate(all="ignore"):
        shift, scale, codes = ko.quantise(oplan, x)
    want = ko.pack(oplan, shift, scale, codes)
    # no minimum and no maximum: infinity and its opposite saturate, the scale is negative and the codes are 0
    shift[-1], scale[-1], codes[-1] = np.float16(65504.0), np.float16(-65504.0), 0
    want[-1] = ko.pack(oplan, shift[-1:], scale[-1:], codes[-1:])
    x_dev = torch.from_numpy(x).to(DEV)
    for tokens in (n, short_tokens() + 33, T):                   # by parts, the short-job kernel, the bulk kernel
        for dtype, src in ((kv.KVTC_F32, x_dev), (kv.KVTC_BF16, x_dev.to(torch.bfloat16))):
            src = src.repeat(tokens // n + 1, 1)[:tokens].contiguous()
            out = torch.zeros((tokens, plan.record_bytes), dtype=torch.uint8, device=DEV)
            kv.kvtc_encode(plan.handle, src, dtype, tokens, p, out, out.numel())
            got = out.cpu().numpy()
            bad = np.nonzero((got[:n] != want).any(axis=1))[0]
            assert bad.size == 0, (tokens, dtype, bad[:5], x[bad[0]], got[bad[0]], want[bad[0]])
            for t0 in range(n, tokens - n + 1, n):
                assert np.array_equal(got[t0:t0 + n], want), (tokens, dtype, t0)


@pytest.mark.parametrize("p,r,tokens", [(128, 112, 150_000), (192, 160, 120_000), (192, 192, 120_000), (256, 224, 220_000), (256, 256, 220_000), (320, 304, 150_000),
                                        (448, 400, 70_000), (512, 512, 70_000), (640, 608, 70_000), (704, 672, 40_000), (1024, 1024, 40_000)])
def test_records_of_known_coefficients_in_every_kernel(p, r, tokens):
    """The same in kernels whose waves share a token's record, in whole plans and in plans whose last wave has a tile fewer; tiles with a scale of
    65504 and tiles without follow each other in a workgroup."""
    groups, at = [], 0
    for k in range(64):
        n = min([16, 32, 16, 48, 16, 16, 64, 16][k % 8] if r < 600 else [16, 64, 96, 16][k % 4], r - at)
        if n == 0:
            break
        groups.append((n, [3, 1, 7, 2, 5, 8, 4, 6][k % 8] if r < 600 else [6, 3, 2, 5][k % 4]))
        at += n
    assert at == r
    blocks, at = [], 0
    for n, b in groups:
        blocks.append(ko.Block(at, n, b))
        at += n
    oplan = ko.compile_plan(np.zeros(p), np.eye(p), blocks)
    plan = _gpu_plan(oplan)
    n = 700
    mixed = _rows(n, p)
    tame = torch.from_numpy(np.random.default_rng(p).standard_normal((n, p)).astype(np.float32) * 3).to(torch.bfloat16).float().numpy() + 0.0
    x = np.concatenate([mixed, tame, tame])                       # tiles are of 64 to 256 tokens
    with np.errstate(all="ignore"):
        shift, scale, codes = ko.quantise(oplan, x)
    want = torch.from_numpy(ko.pack(oplan, shift, scale, codes)).to(DEV)
    saturated = (np.abs(scale.astype(np.float32)) == 65504).any(axis=1)
    assert saturated[:n].any() and not saturated[n:].any()
    x_dev = torch.from_numpy(x).to(DEV)
    for dtype, src in ((kv.KVTC_BF16, x_dev.to(torch.bfloat16)), (kv.KVTC_F32, x_dev)):
        # the bulk kernel, several tiles to a workgroup; where there is one, the short-job kernel; by parts, or the short-job kernel where the groups are too many tiles for that
        for T in (tokens, short_tokens() + 31, 3 * n):
            rows = src.repeat(T // (3 * n) + 1, 1)[:T].contiguous()
            out = torch.zeros((T, plan.record_bytes), dtype=torch.uint8, device=DEV)
            kv.kvtc_encode(plan.handle, rows, dtype, T, p, out, out.numel())
            for t0 in range(0, T, 3 * n):
                part = out[t0:t0 + 3 * n]
                bad = torch.nonzero((part != want[:len(part)]).any(dim=1))[:, 0]
                assert bad.numel() == 0, (dtype, T, t0, bad[:5].tolist())


@pytest.mark.parametrize("r", [144, 160, 208, 272, 304])
def test_plans_of_fewer_tiles_than_their_variant(r):
    """5, 7 and 9 coordinate tiles (whole and half a last one) run in the variants of 6, 8 and 10, which leave the padding out."""
    es.test_bulk_kernels_code_the_same_bits_from_every_type_and_layout(r)


@pytest.mark.parametrize("bits", range(1, 17))
def test_the_kernels_numerics_are_the_plain_ones_for_every_value(bits):
    """Directed roundings, headers and codes as the kernels work them out against the definitions that the CPU tests hold to the oracle."""
    counts = torch.zeros(4, dtype=torch.int64, device=DEV)
    assert kv.lib().kvtc_test_numeric(bits, counts.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert counts.tolist() == [2 ** 32 - 2 * (2 ** 23 - 1), 0, 0, 0]
