"""GPU: more than 512 tables of one to five groups each (a work-group of more wavefronts than groups a table), ragged last groups, and
numbers of tables around what one launch finishes the container of."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,D", [
    (513, 16, 8), (520, 64, 64), (520, 65, 64), (513, 128, 64), (520, 171, 65), (513, 256, 64), (515, 257, 64),   # groups of 4096
    (257, 513, 64),
])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_containers(T, B, D, dtype):
    from gpu_util import DeviceRun
    rng = np.random.default_rng(T + B)
    x = (rng.normal(0, 1, (T, B, D)) * np.exp(rng.uniform(-3, 0, T))[:, None, None]).astype(dtype)
    x[3] = 0.25                                           # one symbol
    x[5, 0, :3] = 1e4 if dtype == np.float16 else 1e9     # escapes
    ebs = np.full(T, 0.02, np.float32)
    g = DeviceRun(x, ebs, S=64)
    o = oracle.compress(x, ebs, S=64)
    assert g.status == 0 and np.array_equal(g.sizes, o.sizes) and np.array_equal(g.data, o.data)
    st, rec = g.decompress()
    rc, want = oracle.decompress(o.data, x.shape, x.dtype)
    assert st == 0 and rc == 0 and np.array_equal(rec.view(np.uint8), want.view(np.uint8))
