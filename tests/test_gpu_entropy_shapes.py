"""The lossless stage where its launches change shape: records of one and of two table segments with whole and partial store
batches, code tables that fit the LDS and that do not, launches whose waves take several chunks each, and code lengths at
both ends of what a table may hold.  Containers must equal the oracle's byte for byte."""
import numpy as np
import pytest

import kvtc_entropy as ke
import paper_2511_01815_amd as kv
from test_gpu_entropy import _gpu_decode, _gpu_encode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,T", [(64, 65), (100, 1), (144, 200), (148, 130), (212, 64), (268, 129), (272, 129), (4, 525_000), (12, 263_000)])
def test_container_at_the_edges_of_the_launch_shapes(R, T):
    """T = 525 000: 8204 chunks, two per 16-wave workgroup's wave on 256 compute units; 263 000: one."""
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
