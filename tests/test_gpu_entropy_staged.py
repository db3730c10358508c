"""The decoder of records of up to 128 bytes under complete codes, where it can go wrong: complete codes of every shape (each bound between two
lengths has to fall between two entries of its length table), records that end inside a unit of 32 positions or are no multiple of
16 bytes, chunks of few tokens, strings up to 12 bits a byte and payloads that end with the last string; and a record of 132 bytes
and an incomplete code, which the other decoder serves.  The oracle codes the records; the bytes must come back.
And the encoder's strings, which leave in whole pieces of 16 bytes with the rest carried on, against the oracle's byte for byte."""
import numpy as np
import pytest

import kvtc_entropy as ke
import paper_2511_01815_amd as kv
from test_gpu_entropy import _gpu_decode, _gpu_encode

pytestmark = pytest.mark.gpu


def _complete_code(rng, kind):
    """256 code lengths of a complete code: a leaf of the tree split 255 times, chosen at random, the shallowest, or the deepest that may be."""
    leaves = [0]
    while len(leaves) < 256:
        open_ = [i for i, d in enumerate(leaves) if d < 12]
        if kind == "deep":                     # as deep as 256 leaves under 12 bits can be made: one leaf a level, the rest under the last
            i = max(open_, key=lambda k: (leaves[k], -k)) if len(leaves) < 12 else rng.choice(open_)
        else:
            i = min(open_, key=lambda k: leaves[k]) if kind == "even" else rng.choice(open_)
        d = leaves.pop(i) + 1
        leaves += [d, d]
    out = np.array(leaves, dtype=np.uint8)
    rng.shuffle(out)
    return out


@pytest.mark.parametrize("R,T", [(4, 65), (28, 64), (32, 130), (36, 63), (60, 200), (64, 1), (100, 129), (124, 64), (128, 700), (132, 65)])
def test_complete_codes_of_every_shape(R, T):
    rng = np.random.default_rng(1000 * R + T)
    lengths = np.stack([_complete_code(rng, ("random", "even", "deep", "random")[k % 4]) for k in range(R)])
    lengths[0] = 9                             # one symbol of 1 bit, the others of 9 but for the one that completes the code
    lengths[0, :2] = 1, 8
    assert np.all((2.0 ** -lengths.astype(float)).sum(axis=1) == 1.0)
    rec = rng.integers(0, 256, (T, R)).astype(np.uint8)
    longest = lengths.argmax(axis=1)
    rec[::5] = longest                         # strings as long as they can be
    tab = kv.EntropyTables(R, lengths)
    assert np.array_equal(_gpu_decode(tab, ke.encode(rec, lengths), T, R), rec)
    tab.close()


def test_one_incomplete_code_among_complete_ones():
    rng = np.random.default_rng(3)
    R, T = 64, 300
    lengths = np.stack([_complete_code(rng, "random") for _ in range(R)])
    k = 37
    lengths[k, lengths[k].argmin()] += 1       # strings that begin no code, below the longest ones
    rec = rng.integers(0, 256, (T, R)).astype(np.uint8)
    tab = kv.EntropyTables(R, lengths)
    assert np.array_equal(_gpu_decode(tab, ke.encode(rec, lengths), T, R), rec)
    tab.close()


@pytest.mark.parametrize("R,T", [(4, 1), (4, 65), (12, 200), (16, 64), (36, 129), (48, 700), (128, 63), (132, 65), (264, 70), (268, 66)])
@pytest.mark.parametrize("kind", ["longest", "shortest", "mixed"])
def test_strings_of_carried_pieces(R, T, kind):
    """Records whose pieces of 16 bytes lie within a record and across two, chunks that end inside a step, tables in LDS and (268 bytes) not; codes of
    12 bits throughout (the most a step can carry and store), of one bit (less than a piece a step, at 4 bytes), and both."""
    rng = np.random.default_rng(100 * R + T)
    lengths = np.full((R, 256), 9, dtype=np.uint8)
    lengths[:, 0], lengths[:, 1:18] = 1, 12      # 1/2 + 17/4096 + 238/512 <= 1
    rec = rng.integers(0, 256, (T, R)).astype(np.uint8)
    if kind == "longest":
        rec = (1 + rec % 17).astype(np.uint8)
    elif kind == "shortest":
        rec[:] = 0
    else:
        rec[rng.random((T, R)) < 0.6] = 0
    tab = kv.EntropyTables(R, lengths)
    ref = ke.encode(rec, lengths)
    out, n, bound = _gpu_encode(tab, rec)
    assert n == len(ref) and out[:n].tobytes() == ref
    assert np.all(out[bound:] == 0xA5), "wrote past the bound"
    assert np.array_equal(_gpu_decode(tab, ref, T, R), rec)
    tab.close()
