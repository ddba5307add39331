"""GPU: the sets of rows by hash at the edges of their sizes: batches around a power of two of slots, and around the largest
batch whose rows lie in the sets with a part of their hash."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [63, 64, 65, 4095, 4097, 8193, 16384, 16385, 65535, 65536, 65537])
@pytest.mark.parametrize("distinct", [1, 3, 0])  # rows that occur (0: nearly all differ)
def test_counts_of_distinct_rows(B, distinct):
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(B + distinct)
    T, D = 2, 4
    pool = rng.normal(0, 1, (distinct or 2 * B, D)).astype(np.float32)
    x = pool[rng.integers(0, len(pool), (T, B))]
    x[1, B - 1] = 5.0                                      # the last row by itself
    probe = np.full(T, 1e-3, np.float32)
    got = b.Context(b.make_config(b.F32, T, B, D)).stats(torch.from_numpy(x).cuda(), probe)
    for a, want in zip(got, oracle.stats(x, probe)):
        assert (a.n_unique_raw, a.n_unique_quant) == (want.n_unique_raw, want.n_unique_quant)


@pytest.mark.parametrize("B", [64, 4097, 65536, 65537])
def test_references_are_the_first_equal_row(B):
    from gpu_util import DeviceRun
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(B)
    x = rng.normal(0, 0.1, (2, 40 if B < 100 else B // 3, 8)).astype(np.float32)
    x = np.stack([t[rng.integers(0, len(t), B)] for t in x])
    g = DeviceRun(x, 1e-2, S=64, flags=b.FLAG_ROW_MATCH)
    o = oracle.compress(x, [1e-2, 1e-2], S=64, row_match=True)
    assert g.status == 0 and np.array_equal(g.data, o.data) and np.array_equal(g.sizes, o.sizes)


def _unmix(z):
    """The number whose mix (two xor-shifts and multiplications and a last xor-shift) is z."""
    m = (1 << 64) - 1
    for shift, factor in ((31, 0x94D049BB133111EB), (27, 0xBF58476D1CE4E5B9), (30, None)):
        x = z
        for _ in range(64 // shift):
            x = z ^ (x >> shift)
        z = x if factor is None else x * pow(factor, -1, 1 << 64) & m
    return z


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_rows_whose_hashes_agree_in_the_tag_alone(seed):
    """Two rows whose hashes differ, but not in the 48 bits that lie beside the index in a slot, and lead to the same place: with
    these multipliers a hash is the mix of eight of a row's bytes."""
    import torch
    from gpu_util import to_device
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(seed)
    B, D, eb = 40, 16, np.float32(2.0 ** -10)  # (64 places)
    while True:  # (each byte has to be an index of the window: 0 to 252)
        h = int(rng.integers(0, 1 << 63))
        pair = [_unmix(h), _unmix(h ^ (int(rng.integers(1, 1024)) << 6))]
        idx = np.array([[(v >> (8 * k)) & 255 for k in range(8)] for v in pair])
        if idx.max() <= 252:
            break
    rows = np.full((2, D), 127)
    rows[:, [0, 1, 4, 5, 8, 9, 12, 13]] = idx  # the lower halves of the row's four pieces
    mult = np.zeros((D // 4, 8), np.uint32)
    mult[0, 0] = mult[2, 2] = 1
    mult[1, 0] = mult[3, 2] = 1 << 16
    x = ((rows[rng.integers(0, 2, B)] - 127) * (2 * float(eb))).astype(np.float32)[None]
    x[0, :4] = x[0, [list(x[0, :, 0]).index(v) for v in dict.fromkeys(x[0, :, 0])]][[0, 1, 1, 0]]  # both at the start, both again
    cfg = b.make_config(b.F32, 1, B, D, 512, 64, 12, b.FLAG_ROW_MATCH)
    ctx = b.Context(cfg)
    ctx.set_row_hash_multipliers(mult)
    ctx.set_error_bounds(eb=[eb])
    out = torch.zeros(b.dlc_compress_bound(cfg), dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(2, dtype=torch.int64, device="cuda")
    assert ctx.compress(to_device(x), out, sizes) == 0 and ctx.sync_status() == 0
    want = np.array([min(j for j in range(B) if np.array_equal(x[0, j], x[0, i])) for i in range(B)])
    assert sorted(set(want)) == [0, 1] and np.array_equal(ctx.read_row_refs()[0], want)
    o = oracle.compress(x, [eb], S=64, row_match=True)
    assert np.array_equal(out[:int(sizes[0])].cpu().numpy(), o.data)
