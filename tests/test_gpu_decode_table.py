"""The decode table's entries (bins of two codewords, their lengths) at the ends of what they can hold: every radius with its
shortest and its longest code limit, the outermost bins, escapes, tables of one symbol; reconstructions against the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_util import DeviceRun

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -12)  # bins are exact multiples of 2^-11


@pytest.mark.parametrize("dtype", [np.float32, np.float16], ids=["f32", "f16"])
@pytest.mark.parametrize("radius,lmax", [(8, 4), (8, 12), (32, 6), (512, 10), (512, 12), (1024, 11), (1024, 12), (2048, 12)])
def test_outermost_bins(radius, lmax, dtype):
    rng = np.random.default_rng(radius * 16 + lmax)
    T, B, D, S = 6, 331, 13, 64  # two groups, the second ragged, n odd
    bins = np.empty((T, B * D))
    bins[0] = rng.integers(-(radius - 1), radius, B * D)                                # all symbols alike
    bins[1] = np.where(rng.random(B * D) < 0.5, radius - 1, -(radius - 1))              # the two outermost, a bit each
    bins[2] = (np.minimum(rng.geometric(0.5, B * D), radius) - 1) * rng.choice([-1, 1], B * D)  # codes of every length
    bins[3] = radius - 1                                                                # one symbol, no bits
    bins[4] = np.where(rng.random(B * D) < 0.4, 4 * radius, 1 - radius)                 # escapes and the lowest bin
    bins[5] = 4 * radius                                                                # escapes only
    x = (bins * (2.0 * float(EB))).astype(dtype).reshape(T, B, D)
    ebs = np.full(T, EB, np.float32)
    run = DeviceRun(x, ebs, R=radius, S=S, LMAX=lmax)
    o = oracle.compress(x, ebs, radius, S, lmax)
    assert run.status == 0 and o.rc == 0 and np.array_equal(run.data, o.data)
    st, rec = run.decompress()
    rc, orec = oracle.decompress(o.data, x.shape, dtype)
    u = np.uint16 if dtype == np.float16 else np.uint32
    assert st == 0 and rc == 0 and np.array_equal(rec.view(u), orec.view(u))
