"""GPU parity of the positional rotation of keys (kvtc_rope) against the float64 oracle, and the whole
key path -- rotation undone, coded, decoded, rotated again -- against the oracle's."""
import numpy as np
import pytest
import torch

import kvtc_oracle as ko
import kvtc_rope as kr
import kvtc_synth as ks
import paper_2511_01815_amd as kv

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _bf16_bits(a32):
    """bf16 bit patterns of float32 values that are exactly representable."""
    return (np.ascontiguousarray(a32, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _to_dev_bf16(a32):
    return torch.from_numpy(_bf16_bits(a32).view(np.int16)).to(DEV).view(torch.bfloat16)


def _from_dev_bf16(t):
    return (t.view(torch.int16).cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("pairing", ["half", "interleaved"])
@pytest.mark.parametrize("inverse", [False, True])
def test_rotation_matches_the_oracle_bf16(pairing, inverse):
    """8 heads x 128 features, 1111 tokens at scattered positions up to 131071 (one at 0): the result, rounded once to
    bf16, must be the oracle's float64 rotation rounded to bf16 -- bit for bit up to the last-bit freedom of sin/cos
    (a result within 1e-15 relative of a bf16 rounding boundary), which may move at most 1e-6 of the entries by one ulp."""
    rng = np.random.default_rng(31)
    H, d, T = 8, 128, 1111
    x = ko.bf16_round((rng.standard_normal((T, H * d)) * np.exp(rng.normal(0, 1.5, (1, H * d)))).astype(np.float32))
    pos = rng.integers(0, 131072, size=T).astype(np.int32)
    pos[0], pos[1] = 0, 131071
    want64 = kr.rope(x, pos, H, d, base=10000.0, pairing=pairing, inverse=inverse)
    want = ko.bf16_round(want64)          # one rounding from float64
    xd = _to_dev_bf16(x).reshape(T, H * d).clone()
    kv.kvtc_rope(xd, kv.KVTC_BF16, T, H, d, H * d, d, torch.from_numpy(pos).to(DEV), 0, 10000.0,
                 kv.ROPE_HALF if pairing == "half" else kv.ROPE_INTERLEAVED, inverse)
    torch.cuda.synchronize()
    got = _from_dev_bf16(xd).reshape(T, H * d)
    np.testing.assert_array_equal(got[0], x[0])                    # position 0: identity
    ne = _bf16_bits(got) != _bf16_bits(want.astype(np.float32))
    assert ne.mean() <= 1e-6, ne.mean()
    if ne.any():
        assert np.abs(_bf16_bits(got)[ne].astype(np.int64) - _bf16_bits(want.astype(np.float32))[ne].astype(np.int64)).max() <= 1


def test_rotation_layouts_positions_and_fp32():
    """fp32 tensors (within one float ulp of the float64 result), consecutive positions from position0, a padded row
    pitch, and the heads-major [H][T][d] layout: all the same rotation."""
    rng = np.random.default_rng(32)
    H, d, T = 4, 64, 300
    x = rng.standard_normal((T, H * d)).astype(np.float32)
    pos0 = 70000
    want = kr.rope(x, np.arange(T) + pos0, H, d, base=500000.0, pairing="half")
    # token-major with a padded pitch
    ld = H * d + 32
    xd = torch.zeros((T, ld), dtype=torch.float32, device=DEV)
    xd[:, :H * d] = torch.from_numpy(x).to(DEV)
    kv.kvtc_rope(xd, kv.KVTC_F32, T, H, d, ld, d, None, pos0, 500000.0, kv.ROPE_HALF, False)
    torch.cuda.synchronize()
    got = xd.cpu().numpy()
    assert np.all(got[:, H * d:] == 0.0)                                           # padding untouched
    np.testing.assert_allclose(got[:, :H * d], want, rtol=2.0 ** -23, atol=1e-30)
    # heads-major
    xh = torch.from_numpy(kr.heads_first(x, H, d)).to(DEV).contiguous()           # [H, T, d]
    kv.kvtc_rope(xh, kv.KVTC_F32, T, H, d, d, T * d, None, pos0, 500000.0, kv.ROPE_HALF, False)
    torch.cuda.synchronize()
    np.testing.assert_allclose(kr.tokens_first(xh.cpu().numpy()), want, rtol=2.0 ** -23, atol=1e-30)
    # undo after redo returns the input to float accuracy
    kv.kvtc_rope(xh, kv.KVTC_F32, T, H, d, d, T * d, None, pos0, 500000.0, kv.ROPE_HALF, True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(kr.tokens_first(xh.cpu().numpy()), x, rtol=0, atol=2e-6 * np.abs(x).max())


def test_key_path_rotation_undone_coded_decoded_rotated_again():
    """Keys of config 2's shape with the rotation applied (what a cache holds): kvtc_rope(inverse) + kvtc_encode must
    give the stream the oracle gives for the un-rotated keys (its bars for codes and headers), and kvtc_decode +
    kvtc_rope must give the oracle's decode rotated by the oracle, within the coder's reconstruction bar."""
    from test_gpu_parity import check_stream
    from paper_2511_01815_amd import bundles as kb
    H, d, T = 8, 128, 2000
    b = kb.load_plan_arrays("c2_K_cr16")
    L = ks.make_layer(ks.layer_spec("c2", 0, 0))
    k_plain = ko.bf16_round(ks.draw_f32(L, T, ks.TEST_DRAW))                      # keys before the rotation
    pos = np.arange(T) + 5000
    k_rot = ko.bf16_round(kr.rope(k_plain, pos, H, d).astype(np.float32))         # what the cache holds (bf16)
    # oracle path: undo in float64, round once to bf16 (the coder's input type), encode
    k_undone = ko.bf16_round(kr.rope(k_rot, pos, H, d, inverse=True).astype(np.float32))
    groups = list(zip(b["group_n"].tolist(), b["group_bits"].tolist()))
    oplan = ko.plan_from_arrays(b["mu32"], b["v_bits"], b["group_n"], b["group_bits"])
    plan = kv.Plan(1024, b["v_bits"].shape[1], b["mu32"], b["v_bits"], groups)
    xd = _to_dev_bf16(k_rot).reshape(T, H * d).clone()
    kv.kvtc_rope(xd, kv.KVTC_BF16, T, H, d, H * d, d, None, 5000, 10000.0, kv.ROPE_HALF, True)
    torch.cuda.synchronize()
    undone_gpu = _from_dev_bf16(xd).reshape(T, H * d)
    assert (_bf16_bits(undone_gpu) != _bf16_bits(k_undone)).mean() <= 1e-6
    out = torch.zeros(T * plan.record_bytes, dtype=torch.uint8, device=DEV)
    kv.kvtc_encode(plan.handle, xd, kv.KVTC_BF16, T, H * d, out, out.numel())
    xh = torch.empty_like(xd)
    kv.kvtc_decode(plan.handle, out, out.numel(), T, xh, kv.KVTC_BF16, H * d)
    kv.kvtc_rope(xh, kv.KVTC_BF16, T, H, d, H * d, d, None, 5000, 10000.0, kv.ROPE_HALF, False)
    torch.cuda.synchronize()
    recs = out.cpu().numpy().reshape(T, -1)
    check_stream(oplan, undone_gpu, recs, "keys-rope")
    want = kr.rope(ko.decode(oplan, recs), pos, H, d)                             # oracle decode, rotated again by the oracle
    got = _from_dev_bf16(xh).reshape(T, H * d)
    rng_x = float(k_rot.max() - k_rot.min())
    assert np.abs(got - want).max() <= 1e-2 * rng_x
    # and the point of it all: the round trip is as close to the cached keys as the coder is to the un-rotated ones
    rel = np.linalg.norm(got - k_rot) / np.linalg.norm(k_rot - k_rot.mean(0))
    assert rel < 0.3, rel


@pytest.mark.parametrize("d,H,T,offset,pairing,base,bits", [
    (16, 1, 1, 0, "half", 1e4, 17), (16, 9, 513, 0, "interleaved", 256.0, 31),    # one lane to a token; heads in shares with one left over
    (80, 3, 260, 0, "half", 5e5, 17), (256, 5, 130, 0, "interleaved", 1e4, 17),   # lanes of a token that are no power of two; the widest head
    (128, 8, 3000, 0, "half", 2.0 ** 64, 31),                                     # a share's heads more than are on their way at a time
    (128, 2, 70, 1, "half", 1e4, 17), (24, 4, 70, 0, "half", 1e4, 17),            # an address, a head that whole pieces do not fit
    (64, 2, 70, 0, "interleaved", 0.9, 17),                                       # angles above the positions
    (64, 2, 3600, 0, "interleaved", 0.9, 17), (128, 2, 1800, 1, "half", 1e4, 17), # (these and the address, with tokens enough for whole pieces)
    (16, 1, 20001, 0, "half", 1e4, 17), (128, 1, 2500, 0, "half", 1e4, 17), (128, 1, 2499, 0, "interleaved", 1e4, 17),          # from 20000 items of eight pairs on
    (128, 2, 1750, 0, "interleaved", 1e4, 17), (128, 3, 15, 0, "half", 1e4, 17), (128, 3, 16, 0, "half", 1e4, 17), (128, 5, 4, 0, "half", 1e4, 17),
    (128, 6, 1, 0, "interleaved", 1e4, 17), (48, 7, 300, 0, "half", 1e4, 17),     # a row's heads over neighbouring lanes: all of them, and shares that are not equal
    (64, 33, 130, 0, "half", 1e4, 17), (128, 17, 1100, 0, "interleaved", 1e4, 17),  # long rows
    (16, 2, 16385, 0, "half", 1e4, 17), (32, 16, 16385, 0, "half", 1e4, 17),      # narrow heads of many tokens
])
def test_whole_pieces_and_what_they_do_not_fit_bf16(d, H, T, offset, pairing, base, bits):
    """Scattered positions, token-major and heads-major.  The kernel's sine and cosine are within 1e-15, and only a value within that of a
    rounding boundary can come out otherwise: no entry of these may.  Positions of all 31 bits come with frequencies that are powers of two:
    another base's differ from the oracle's by 2^-53 where two libraries' powers do, and angles of 2^31 then by 2e-7, which moves one
    entry in 10^4 to 10^5."""
    rng = np.random.default_rng(d * H + T)
    x = ko.bf16_round(rng.standard_normal((T, H * d)).astype(np.float32))
    pos = rng.integers(0, 2 ** bits - 1, size=T).astype(np.int32)
    pos[:2] = (2 ** bits - 1, 0)[:T]
    pos_dev = torch.from_numpy(pos).to(DEV)
    for inverse in (False, True):
        want = _bf16_bits(ko.bf16_round(kr.rope(x, pos, H, d, base=base, pairing=pairing, inverse=inverse)).astype(np.float32))
        for heads_major in (False, True):
            src = kr.heads_first(x, H, d) if heads_major else x
            room = torch.zeros(offset + src.size, dtype=torch.bfloat16, device=DEV)
            xd = room[offset:]
            xd.copy_(_to_dev_bf16(np.ascontiguousarray(src)).reshape(-1))
            ts, hs = (d, T * d) if heads_major else (H * d, d)
            kv.kvtc_rope(xd, kv.KVTC_BF16, T, H, d, ts, hs, pos_dev, 0, base, kv.ROPE_HALF if pairing == "half" else kv.ROPE_INTERLEAVED, inverse)
            torch.cuda.synchronize()
            got = _from_dev_bf16(xd).reshape(src.shape)
            got = kr.tokens_first(got) if heads_major else got
            assert np.array_equal(_bf16_bits(got), want), (inverse, heads_major, (_bf16_bits(got) != want).mean())


@pytest.mark.parametrize("pairing", ["half", "interleaved"])
def test_values_of_every_kind_and_positions_below_zero_bf16(pairing):
    """NaN, infinities, zeros of both signs, subnormal and the largest numbers, at position 0 too, where an infinity meets a sine of 0; positions from below
    zero on, by position0 and by an array.  A result is NaN where the oracle's is, and otherwise the same bits."""
    rng = np.random.default_rng(8)
    H, d, T = 8, 128, 600
    bits = rng.integers(0, 65536, size=(T, H * d)).astype(np.uint16)                                     # every kind of number
    kinds = np.array([0x7f80, 0xff80, 0x7fc0, 0xffff, 0x7f81, 0x0000, 0x8000, 0x0001, 0x807f, 0x7f7f, 0xff7f, 0x3f80], dtype=np.uint16)
    bits[::3] = rng.choice(kinds, size=bits[::3].shape)
    bits[1::3] = (bits[1::3] & 0x80ff)                                                                   # subnormal, and the smallest normal ones
    x = (bits.astype(np.uint32) << 16).view(np.float32)
    pos = np.arange(T) - 299
    with np.errstate(all="ignore"):
        want64 = kr.rope(x, pos, H, d, base=10000.0, pairing=pairing)
        want = torch.from_numpy(want64.astype(np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    nan = np.isnan(want64)
    assert 0.01 < nan.mean() < 0.9 and (np.abs(want64[~nan]) < 2.0 ** -126).any()
    for positions in (None, torch.from_numpy(pos.astype(np.int32)).to(DEV)):
        xd = torch.from_numpy(bits.view(np.int16)).to(DEV).view(torch.bfloat16).clone()
        kv.kvtc_rope(xd, kv.KVTC_BF16, T, H, d, H * d, d, positions, -299, 10000.0, kv.ROPE_HALF if pairing == "half" else kv.ROPE_INTERLEAVED, False)
        torch.cuda.synchronize()
        got = xd.view(torch.int16).cpu().numpy().view(np.uint16)
        assert np.array_equal((got & 0x7fff) > 0x7f80, nan)
        bad = (got != want) & ~nan
        assert not bad.any(), (bad.sum(), x[bad][:4], got[bad][:4], want[bad][:4])
