"""The calibration passes at the edges of what their kernels are built for: block sizes around each lane-group width (16, 64,
256, 1024 coordinates), token counts around the groups of four and the split of long blocks in two halves, feature counts of
one, two and several strips; against the oracle's scalar numerics and NumPy in float64."""
import numpy as np
import pytest
import torch

import kvtc_oracle as ko
import paper_2511_01815_amd as kv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_tok", [1, 3, 4, 5, 63, 66, 129, 1030])
def test_block_errors_at_every_lane_group_edge(n_tok):
    rng = np.random.default_rng(n_tok)
    ld = 1037
    P = (rng.standard_normal((n_tok, ld)) * np.arange(1, ld + 1) ** -0.6).astype(np.float32)
    cand = [(s, n) for n in (1, 3, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1000, 1023, 1024) for s in (0, ld - n)]
    blocks = torch.tensor(cand, dtype=torch.int32, device=DEV)
    out = torch.full((len(cand), 8), -7.0, dtype=torch.float64, device=DEV)
    pd = torch.from_numpy(P).to(DEV)
    for _ in range(2):
        kv.kvtc_calib_block_errors(pd, n_tok, ld, blocks, len(cand), 8, out)
        first = out.clone() if _ == 0 else first
    torch.cuda.synchronize()
    assert torch.equal(out, first)                       # the same bits again
    got = out.cpu().numpy()
    for i, (s, n) in enumerate(cand):
        d = P[:, s:s + n]
        energy = float((d.astype(np.float64) ** 2).sum())
        for b in range(1, 9):
            sh, sc, codes = ko.quantise_group(d, b)
            dh = ko.dequantise_group(sh, sc, codes).astype(np.float64)
            ref = float(((d - dh) ** 2).sum()) - energy
            # the same terms in another order: n_tok * n sums of double precision, each term within energy's scale
            assert abs(got[i, b - 1] - ref) <= 1e-12 * (energy + abs(ref)), (n_tok, s, n, b)


@pytest.mark.parametrize("n_tok", [50, 1030])
@pytest.mark.parametrize("max_bits", [1, 2, 3, 7])
def test_tables_of_fewer_widths_hold_the_same_rows(max_bits, n_tok):
    """One width to a workgroup (lists that leave compute units idle) or two, the last of them alone where their number is odd: an
    entry has the same bits in the table of eight widths, in a short list and in a long one (a width's sums keep their order), and
    nothing beyond the table is written."""
    rng = np.random.default_rng(n_tok + max_bits)
    ld = 1030
    coef = torch.from_numpy(rng.standard_normal((n_tok, ld)).astype(np.float32)).to(DEV)
    cand = [(s, n) for n in (3, 16, 17, 64, 65, 256, 257, 1024) for s in (0, ld - n)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def table(reps, widths):
        blocks = torch.tensor(cand * reps, dtype=torch.int32, device=DEV)
        out = torch.full((len(blocks) * widths + 3,), -7.0, dtype=torch.float64, device=DEV)
        kv.kvtc_calib_block_errors(coef, n_tok, ld, blocks, len(blocks), widths, out)
        torch.cuda.synchronize()
        assert bool((out[len(blocks) * widths:] == -7.0).all())
        return out[:len(blocks) * widths].view(reps, len(cand), widths)

    want = table(1, 8)[0, :, :max_bits]
    for reps in (1, cus // (len(cand) * max_bits) + 1):
        got = table(reps, max_bits)
        assert all(torch.equal(g, want) for g in got), (reps, (got - want).abs().max().item())


@pytest.mark.parametrize("n_tok,p", [(1, 64), (3, 64), (4, 128), (17, 192), (130, 64), (515, 320)])
def test_moments_at_strip_and_token_edges(n_tok, p):
    rng = np.random.default_rng(n_tok + p)
    for dtype in (kv.KVTC_BF16, kv.KVTC_F32):
        X = rng.standard_normal((n_tok, p + 8)).astype(np.float32)
        xd = torch.from_numpy(X).to(DEV)
        if dtype == kv.KVTC_BF16:
            xd = xd.to(torch.bfloat16)
        x64 = xd.double().cpu().numpy()[:, :p]
        s = torch.full((p,), -7.0, dtype=torch.float64, device=DEV)
        g = torch.full((p, p), -7.0, dtype=torch.float64, device=DEV)
        kv.kvtc_calib_moments(xd, dtype, n_tok, p, kv.layout(p + 8), s, g)
        torch.cuda.synchronize()
        # double-precision sums of n_tok terms: n_tok * 2^-53 of the sum of magnitudes at most
        assert np.all(np.abs(s.cpu().numpy() - x64.sum(0)) <= n_tok * 2.0 ** -52 * np.abs(x64).sum(0))
        assert np.all(np.abs(g.cpu().numpy() - x64.T @ x64) <= n_tok * 2.0 ** -52 * (np.abs(x64).T @ np.abs(x64)))


@pytest.mark.parametrize("n_tok,long_list", [(1, False), (5, False), (200, False), (259, False), (5, True), (259, True)])
def test_blocks_with_coefficients_that_are_not_finite_come_out_as_nan(n_tok, long_list):
    """The squared error and the energy of such a block are both infinite, so their difference is not a number -- for every block that
    holds the coefficient, in any lane group, at any width and wherever the token stands, and for no other block.  259 tokens: all blocks of more than
    64 coordinates in halves, the first of which ends at the middle token.  A long list: two widths to a workgroup."""
    ld = 1100
    rng = np.random.default_rng(n_tok)
    cand = [(s, n) for n in (3, 16, 40, 64, 200, 256, 300, 1024) for s in (0, 16, ld - n)]
    if long_list:
        cand *= torch.cuda.get_device_properties(0).multi_processor_count // (8 * len(cand)) + 1
    blocks = torch.tensor(cand, dtype=torch.int32, device=DEV)
    P = rng.standard_normal((n_tok, ld)).astype(np.float32)

    def table(p):
        out = torch.full((len(cand), 8), -7.0, dtype=torch.float64, device=DEV)
        kv.kvtc_calib_block_errors(torch.from_numpy(p).to(DEV), n_tok, ld, blocks, len(cand), 8, out)
        return out.cpu().numpy()

    clean = table(P)
    assert np.all(np.isfinite(clean))
    for bad in (np.inf, -np.inf, np.nan):
        for t in {0, n_tok // 2, n_tok - 1}:
            for at in (0, 17, ld - 1):
                Q = P.copy()
                Q[t, at] = bad
                got = table(Q)
                hit = np.array([s <= at < s + n for s, n in cand])
                assert np.all(np.isnan(got[hit])), (bad, t, at)
                assert np.array_equal(got[~hit], clean[~hit]), (bad, t, at)
    big = P.copy()
    big[0, 5], big[n_tok - 1, 6] = 3.4e38, -3.4e38                # the range of a block overflows fp32, its terms do not overflow
    assert np.all(np.isfinite(table(big)))


def _features_of_split(parts):
    """The smallest number of features whose tiles, or those of its last round, run in this many parts."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for p in range(192, 4096, 64):
        rest = (p // 32) * (p // 32 + 1) // 2 % cus
        if parts == (4 if rest * 4 <= cus else 2 if rest * 2 <= cus else 1):
            return p
    raise AssertionError(parts)


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("parts", [1, 2, 4])
def test_moments_of_whole_tiles_halves_and_quarters(parts, dtype):
    """The number of features decides whether tiles run whole or in parts: every form against double precision, for rows with a pitch and, the same
    bits, heads-major."""
    n_tok, p, block = 131, _features_of_split(parts), 64
    x = torch.randn((n_tok, p + 8), generator=torch.Generator(device=DEV).manual_seed(p), device=DEV)
    x = x.to(torch.bfloat16) if dtype == kv.KVTC_BF16 else x
    heads = x[:, :p].reshape(n_tok, p // block, block).transpose(0, 1).contiguous()
    got = []
    for buf, lay in ((x, kv.layout(p + 8)), (heads, kv.layout(block, block, n_tok * block))):
        s = torch.full((p,), -7.0, dtype=torch.float64, device=DEV)
        g = torch.full((p, p), -7.0, dtype=torch.float64, device=DEV)
        kv.kvtc_calib_moments(buf, dtype, n_tok, p, lay, s, g)
        torch.cuda.synchronize()
        got.append((s, g))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    x64 = x.double().cpu().numpy()[:, :p]
    # double-precision sums of n_tok terms: n_tok * 2^-53 of the sum of magnitudes at most
    assert np.all(np.abs(got[0][0].cpu().numpy() - x64.sum(0)) <= n_tok * 2.0 ** -52 * np.abs(x64).sum(0))
    assert np.all(np.abs(got[0][1].cpu().numpy() - x64.T @ x64) <= n_tok * 2.0 ** -52 * (np.abs(x64).T @ np.abs(x64)))


@pytest.mark.parametrize("dtype", [kv.KVTC_BF16, kv.KVTC_F32])
@pytest.mark.parametrize("parts", [1, 2, 4])
def test_moments_into_buffers_that_are_8_byte_aligned_only(parts, dtype):
    """sum_dev and gram_dev need 8-byte alignment, no more: results one double past a 16-byte boundary are the same bits, and
    nothing around them is written (whole tiles and halves store pairs, quarters single entries)."""
    n_tok, p = 77, _features_of_split(parts)
    x = torch.randn((n_tok, p), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV)
    x = x.to(torch.bfloat16) if dtype == kv.KVTC_BF16 else x

    def moments(shift):
        s = torch.full((p + 2,), -7.0, dtype=torch.float64, device=DEV)
        g = torch.full((p * p + 2,), -7.0, dtype=torch.float64, device=DEV)
        assert g.data_ptr() % 16 == 0
        kv.kvtc_calib_moments(x, dtype, n_tok, p, kv.layout(p), s[shift:], g[shift:])
        torch.cuda.synchronize()
        for buf, n in ((s, p), (g, p * p)):
            assert bool((buf[:shift] == -7.0).all()) and bool((buf[shift + n:] == -7.0).all())
        return s[shift:shift + p], g[shift:shift + p * p]

    for a, b in zip(moments(0), moments(1)):
        assert torch.equal(a, b)


def test_lists_longer_than_one_launch_takes():
    """2^22 + 5 blocks, once more than 2^32 threads side by side: every row is that of the same block in a short list."""
    n_tok, ld, n = 3, 64, (1 << 22) + 5
    coef = torch.randn((n_tok, ld), generator=torch.Generator(device=DEV).manual_seed(9), device=DEV)
    short = torch.tensor([(s, 16) for s in range(0, 49)] + [(60, 16)], dtype=torch.int32, device=DEV)        # the last one ends beyond the row
    want = torch.zeros((len(short), 1), dtype=torch.float64, device=DEV)
    kv.kvtc_calib_block_errors(coef, n_tok, ld, short, len(short), 1, want)
    which = torch.arange(n, device=DEV) % len(short)
    got = torch.full((n + 1, 1), -7.0, dtype=torch.float64, device=DEV)
    kv.kvtc_calib_block_errors(coef, n_tok, ld, short[which].contiguous(), n, 1, got)
    torch.cuda.synchronize()
    assert bool(torch.isnan(want[-1]).all()) and float(got[n]) == -7.0
    assert torch.equal(torch.nan_to_num(got[:n], nan=1e300), torch.nan_to_num(want[which], nan=1e300))
