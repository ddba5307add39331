"""Row matching and statistics with every number of tables at which their kernels deal the tables to the chip in another way."""
import numpy as np
import pytest

import oracle
from gpu_util import DeviceRun, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,D", [(T, 300, 16) for T in (1, 7, 8, 12, 13, 16, 47, 48, 49, 64, 73)] +  # two work-groups a table, five in the copy
                         [(T, 2085, 128) for T in (1, 8, 9, 12, 13, 17)])                          # nine, and as many as the copy has
def test_every_table_once(T, B, D):
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(T)
    x = (rng.standard_normal((T, 90, D)) * 0.1).astype(np.float32)
    x = np.take_along_axis(x, rng.integers(0, 90, (T, B, 1)), axis=1)
    ebs = np.full(T, 0.01, np.float32)
    r = DeviceRun(x, ebs, flags=b.FLAG_ROW_MATCH)
    o = oracle.compress(x, ebs, row_match=True)
    assert r.status == 0 and np.array_equal(r.data, o.data)
    st, rec = r.decompress()
    assert st == 0 and np.array_equal(rec.view(np.uint32), oracle.decompress(o.data, x.shape, np.float32)[1].view(np.uint32))
    got, want = b.Context(b.make_config(b.F32, T, B, D)).stats(to_device(x), ebs), oracle.stats(x, ebs)
    assert [(s.min, s.max, s.n_unique_raw, s.n_unique_quant) for s in got] == [(s.min, s.max, s.n_unique_raw, s.n_unique_quant) for s in want]
