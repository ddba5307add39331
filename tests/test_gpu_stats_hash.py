"""GPU: the statistics' row hash at the edges of its steps (64 bytes of a row), chunks (512 bytes) and row sets (16 and 64 rows)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# bytes of a row at and beside 16 (a piece), 64 (a step), every number of steps of one chunk, 512 (a chunk) and beyond
WIDTHS = {np.float32: [1, 3, 4, 5, 16, 17, 33, 48, 50, 79, 80, 96, 97, 112, 127, 128, 129, 257, 1000],
          np.float16: [1, 2, 7, 8, 9, 31, 32, 33, 65, 96, 97, 150, 161, 192, 193, 224, 255, 256, 257, 513, 1003]}


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 65, 333])
def test_rows_and_range_at_the_edges(dtype, B):
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(B)
    T = 3
    for D in WIDTHS[dtype]:
        x = rng.normal(0, 1, (T, B, D)).astype(dtype)
        for t in range(T):
            src = rng.integers(0, B, B)                    # about a third of the rows repeat another
            x[t] = np.where((rng.random(B) < 0.5)[:, None], x[t][src], x[t])
        x[1, B // 2] = x[1, 0]
        x[1, B // 2, D - 1] += dtype(0.004)                # differs in the last element only, raw and perhaps quantised
        x[2] = -np.abs(x[2])                               # no element with a positive sign
        x[0, B - 1, D - 1] = np.inf                        # what is not finite, first, last and in the middle
        x[0, 0, 0] = np.nan
        x[2, B // 2, D // 2] = -np.inf
        probe = np.array([0.05, 0.01, 0.5], np.float32)
        got = b.Context(b.make_config(b.F16 if dtype == np.float16 else b.F32, T, B, D)).stats(torch.from_numpy(x).cuda(), probe)
        for t, want in enumerate(oracle.stats(x, probe)):
            a = got[t]
            assert (a.n_unique_raw, a.n_unique_quant) == (want.n_unique_raw, want.n_unique_quant), (B, D, t)
            assert (a.min, a.max) == (want.min, want.max), (B, D, t)


def test_rows_longer_than_the_table_of_coefficients():
    import torch
    from paper_2407_04272_amd import binding as b
    D = 3 * 65536 + 5                                      # 256 KiB of a row have coefficients of their own
    rng = np.random.default_rng(3)
    x = rng.normal(0, 1, (1, 6, D)).astype(np.float32)
    x[0, 3] = x[0, 1]
    x[0, 4] = x[0, 1]
    x[0, 4, [70, 70 + 65536]] = x[0, 4, [70 + 65536, 70]]  # two elements whose coefficients lie in one place, exchanged
    x[0, 5] = x[0, 2]
    x[0, 5, D - 1] += 1.0
    probe = np.array([0.01], np.float32)
    got = b.Context(b.make_config(b.F32, 1, 6, D)).stats(torch.from_numpy(x).cuda(), probe)[0]
    want = oracle.stats(x, probe)[0]
    assert (got.n_unique_raw, got.n_unique_quant, got.min, got.max) == (want.n_unique_raw, want.n_unique_quant, want.min, want.max)
