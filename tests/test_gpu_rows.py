"""GPU parity of row matching (DLC_FLAG_ROW_MATCH: the vector-based LZ step): references, containers and
reconstructions against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device
from test_oracle_rows import first_occurrence

pytestmark = pytest.mark.gpu

R = 512


def _lookups(T, B, D, seed, rows=60, sigma=0.02, dtype=np.float32):
    rng = np.random.default_rng(seed)
    table = (rng.standard_normal((T, rows, D)) * sigma).astype(np.float32)
    idx = rng.integers(0, rows, (T, B))
    x = np.stack([table[t][idx[t]] for t in range(T)]) * (1 + np.arange(T, dtype=np.float32))[:, None, None]
    return x.astype(dtype)


def _compress(x, ebs, S, flags_per_table=None, zero_hash=False):
    import torch
    from paper_2407_04272_amd import binding as b
    T, B, D = x.shape
    dt = b.F16 if x.dtype == np.float16 else b.F32
    cfg = b.make_config(dt, T, B, D, R, S, 12, b.FLAG_ROW_MATCH)
    ctx = b.Context(cfg)
    if flags_per_table is not None:
        ctx.set_row_match(flags_per_table)
    if zero_hash:
        ctx.set_row_hash_multipliers(np.zeros(8 * (D // 4), np.uint32))
    cap = b.dlc_compress_bound(cfg)
    d = to_device(x)
    out = torch.full((cap + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    ctx.set_error_bounds(eb=ebs)
    assert ctx.compress(d, out, sizes, capacity=cap) == 0
    assert ctx.sync_status() == 0
    h = out.cpu().numpy()
    assert np.all(h[cap:] == 0xA5)
    sz = sizes.cpu().numpy().astype(np.uint64)
    return ctx, d, out, h[:int(sz[0])].copy(), sz


CASES = [  # T, B, D, S, dtype
    (2, 300, 16, 64, np.float32),
    (3, 1000, 48, 256, np.float32),     # several groups, a partial last one
    (4, 2048, 128, 256, np.float32),
    (2, 700, 40, 128, np.float16),
    (1, 257, 20, 64, np.float32),       # rows that straddle the turns of a chunk
    (1, 200, 260, 64, np.float32),      # long rows: more 4-byte pieces than a wavefront has lanes
    (1, 130, 1040, 128, np.float32),    # the same with 16-byte pieces
    (2, 9000, 32, 256, np.float16),     # more rows than one pass of the set kernel's threads
    (1, 280000, 4, 256, np.float32),    # more rows than 32 row sets hold: the rows are divided further
]


@pytest.mark.parametrize("T,B,D,S,dtype", CASES)
def test_containers_and_references_match_the_oracle(T, B, D, S, dtype):
    print("row matching", T, B, D, S, np.dtype(dtype).name, flush=True)
    x = _lookups(T, B, D, 3 * B + D, dtype=dtype)
    big = 1e9 if dtype == np.float32 else 6e4
    x[0, 3, 1] = big
    x[0, 8] = x[0, 3]                       # a repeated row with an escape
    x[0, 11] = x[0, 3]
    x[0, 11, 1] = -big                      # escape at the same place, other raw bits: not a repeat
    ebs = (np.float32(2e-3) * (1 + np.arange(T, dtype=np.float32))).astype(np.float32)
    ctx, d, out, data, sizes = _compress(x, ebs, S)
    sym, _ = oracle.quantize(x[0:1], float(ebs[0]), R)
    for t in range(T):
        s_t, _ = oracle.quantize(x[t:t + 1], float(ebs[t]), R)
        assert np.array_equal(ctx.read_row_refs()[t], first_occurrence(x[t:t + 1], s_t)[0]), t
    o = oracle.compress(x, ebs, R, S, 12, row_match=True)
    assert o.rc == 0 and data.size == o.data.size
    diff = np.nonzero(data != o.data)[0]
    assert diff.size == 0, f"first differing byte {diff[:8]} of {data.size}"
    assert np.array_equal(sizes, o.sizes)
    # the GPU decoder: coded rows decoded, the others copied; equal to the oracle's output and within the bound
    import torch
    rec = torch.full_like(d, 7.0)
    assert ctx.decompress(out, data.size, rec) == 0 and ctx.sync_status() == 0
    rc, orec = oracle.decompress(o.data, x.shape, dtype)
    u = np.uint32 if dtype == np.float32 else np.uint16
    r = rec.cpu().numpy()
    assert rc == 0 and np.array_equal(r.view(u), orec.view(u))
    fin = np.isfinite(x.astype(np.float32)) & (np.abs(x.astype(np.float32)) < 1e4)
    err = np.abs(x.astype(np.float64) - r.astype(np.float64))
    for t in range(T):
        assert np.all(err[t][fin[t]] <= float(ebs[t]) * (1 + 1e-6))


def test_row_matching_per_table():
    x = _lookups(3, 400, 32, 5)
    ebs = np.full(3, 1e-3, np.float32)
    _, _, _, data, sizes = _compress(x, ebs, 128, flags_per_table=[0, 1, 0])
    o = oracle.compress(x, ebs, R, 128, 12, row_match=[0, 1, 0])
    assert np.array_equal(data, o.data) and np.array_equal(sizes, o.sizes)
    _, _, _, data, _ = _compress(x, ebs, 128, flags_per_table=[0, 0, 0])
    assert np.array_equal(data, oracle.compress(x, ebs, R, 128, 12).data)      # all off: the plain container


def test_damaged_references_are_rejected_on_the_gpu():
    import torch
    from paper_2407_04272_amd import binding as b
    import container_reader as cr
    x = _lookups(2, 300, 16, 9)
    ebs = np.full(2, 1e-3, np.float32)
    ctx, d, out, data, sizes = _compress(x, ebs, 64)
    tb = cr.parse(data).tables[1]
    i = int(np.nonzero(tb.ref != np.arange(300))[0][0])
    for bad_value in (i + 1, 0xFFFFFFF0):                  # points forward; points far outside the table
        bad = data.copy()
        bad[tb.ref_off + 4 * i:tb.ref_off + 4 * i + 4] = np.frombuffer(np.uint32(bad_value).tobytes(), np.uint8)
        comp = to_device(np.concatenate([bad, np.zeros(16, np.uint8)]))
        rec = torch.full_like(d, 7.0)
        assert ctx.decompress(comp, bad.size, rec) == 0
        assert ctx.sync_status() == b.ECORRUPT
        r = rec.cpu().numpy()
        refers = tb.ref != np.arange(300)
        assert np.all(r[1][refers] == 7.0)                 # none of the damaged table's references was followed
    # a context without the flag does not take a container with references
    plain = b.Context(b.make_config(b.F32, 2, 300, 16, R, 64, 12))
    rec = torch.full_like(d, 7.0)
    assert plain.decompress(out, data.size, rec) == 0
    assert plain.sync_status() == b.ECORRUPT


@pytest.mark.parametrize("dtype,rows", [(np.float32, 200), (np.float32, 100000), (np.float16, 200), (np.float16, 100000)])
def test_references_of_many_work_groups(dtype, rows):
    """Tables of more groups than a work-group decodes, with many repeated rows (decoded through the caches) and with few (past
    them): the reconstruction is the oracle's; one bad reference, wherever it is, spoils its own table alone."""
    import torch
    from paper_2407_04272_amd import binding as b
    import container_reader as cr
    T, B, D, S = 3, 1500, 96, 64                           # 36 groups: rows lie across their ends
    x = _lookups(T, B, D, 17, rows=rows, dtype=dtype)
    x[:, -1] = x[:, 2]
    x[:, 700] = x[:, 2]
    ebs = np.full(T, 2e-3 if dtype == np.float32 else 4e-3, np.float32) * (1 + np.arange(T, dtype=np.float32))
    ctx, d, out, data, sizes = _compress(x, ebs, S)
    assert np.array_equal(data, oracle.compress(x, ebs, R, S, 12, row_match=True).data)
    u = np.uint32 if dtype == np.float32 else np.uint16
    _, orec = oracle.decompress(data, x.shape, dtype)
    own = np.arange(B)
    refers = [np.nonzero(t.ref != own)[0] for t in cr.parse(data).tables]
    assert all(len(r) * 4 > B for r in refers) == (rows == 200)
    ref_off = cr.parse(data).tables[1].ref_off
    last, mid = B - 1, 700
    for row, value in ((None, 0), (last, mid), (mid, mid + 1), (0, 1), (last, B), (mid, 0x80000000)):
        bad = data.copy()                                  # (a reference to a row that refers itself; forward; past the table)
        if row is not None:
            bad[ref_off + 4 * row:ref_off + 4 * row + 4] = np.frombuffer(np.uint32(value).tobytes(), np.uint8)
        comp = to_device(np.concatenate([bad, np.zeros(16, np.uint8)]))
        rec = torch.full_like(d, 7.0)
        assert ctx.decompress(comp, bad.size, rec) == 0
        assert ctx.sync_status() == (0 if row is None else b.ECORRUPT), (row, value)
        r = rec.cpu().numpy()
        for t in range(T):
            if row is None or t != 1:
                assert np.array_equal(r[t].view(u), orec[t].view(u)), (row, value, t)
        if row is not None:
            assert np.all(r[1][refers[1][refers[1] != row]] == 7.0), (row, value)


def test_random_shapes_rows_and_statistics():
    """A seeded sweep over row lengths (every team size and load width of the row kernels), batch sizes and both
    element types: references, containers, reconstructions and the statistics' distinct-row counts against the
    oracle."""
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(2024)
    dims = [4, 8, 12, 16, 20, 36, 64, 68, 96, 132, 200, 256, 272, 320, 516]
    for case, D in enumerate(dims):
        T = int(rng.integers(1, 4))
        B = int(rng.integers(1, 700))
        dtype = np.float16 if case % 3 == 2 else np.float32
        S = int(rng.choice([64, 128, 256]))
        print("sweep", T, B, D, S, np.dtype(dtype).name, flush=True)
        x = _lookups(T, B, D, 100 + case, rows=max(2, B // 3), dtype=dtype)
        if B > 5:
            x[0, 4, D - 1] = 3e4          # an escape in the last element of a row ...
            x[0, 5] = x[0, 4]             # ... of a row that is repeated
        ebs = (np.float32(3e-3) * (1 + np.arange(T, dtype=np.float32))).astype(np.float32)
        ctx, d, out, data, sizes = _compress(x, ebs, S)
        o = oracle.compress(x, ebs, R, S, 12, row_match=True)
        assert o.rc == 0 and data.size == o.data.size and np.array_equal(data, o.data), (T, B, D, S)
        assert np.array_equal(sizes, o.sizes)
        rec = torch.full_like(d, 7.0)
        assert ctx.decompress(out, data.size, rec) == 0 and ctx.sync_status() == 0
        rc, orec = oracle.decompress(o.data, x.shape, dtype)
        u = np.uint32 if dtype == np.float32 else np.uint16
        assert rc == 0 and np.array_equal(rec.cpu().numpy().view(u), orec.view(u)), (T, B, D, S)
        plain = b.Context(b.make_config(b.F16 if dtype == np.float16 else b.F32, T, B, D, R, S, 12))
        st = plain.stats(d, ebs)
        ost = oracle.stats(x, ebs)
        for t in range(T):
            assert (st[t].n_unique_raw, st[t].n_unique_quant) == (ost[t].n_unique_raw, ost[t].n_unique_quant), (T, B, D, t)
            assert st[t].min == ost[t].min and st[t].max == ost[t].max


def test_compressor_selection_matches_the_oracle():
    """Section III-D, algorithm "Compressor Selection": the per-table choice between the entropy coder alone and row
    matching in front of it, made by the library on a sample, against the oracle's choice from its own containers; the
    container written afterwards is the oracle's container for that choice."""
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(21)
    B, D, S = 900, 32, 128
    distinct = (rng.standard_normal((B, D)) * 0.02).astype(np.float32)                       # no repeats
    few = (rng.standard_normal((5, D)) * 0.02).astype(np.float32)[rng.integers(0, 5, B)]     # five rows, repeated
    some = (rng.standard_normal((300, D)) * 0.02).astype(np.float32)[rng.integers(0, 300, B)]
    x = np.stack([distinct, few, some, few[::-1].copy(), distinct[::-1].copy()])
    T = x.shape[0]
    ebs = np.full(T, 1e-3, np.float32)
    cfg = b.make_config(b.F32, T, B, D, R, S, 12, b.FLAG_ROW_MATCH)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    cap = b.dlc_compress_bound(cfg)
    d = to_device(x)
    out = torch.zeros(cap, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    seen = set()
    for net, tc, td in ((25.0, (2000.0, 1400.0), (4000.0, 2500.0)), (5000.0, (2000.0, 1400.0), (4000.0, 2500.0)),
                        (400.0, (2000.0, 1400.0), (4000.0, 2500.0)), (25.0, (2000.0, 2000.0), (4000.0, 4000.0))):
        print("selection at", net, tc, td, flush=True)
        choice, est = ctx.select_compressors(d, out, sizes, net, tc, td)
        want, want_est = oracle.select_compressors(x, ebs, net, tc, td, R, S, 12)
        assert np.array_equal(choice.astype(np.int32), want), (net, choice, want)
        assert np.array_equal(est, want_est)                       # same sizes, same arithmetic: the same doubles
        seen.add(tuple(int(v) for v in choice))
        assert ctx.compress(d, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
        sz = sizes.cpu().numpy().astype(np.uint64)
        o = oracle.compress(x, ebs, R, S, 12, row_match=want.astype(np.uint8))
        assert np.array_equal(sz, o.sizes)
        assert np.array_equal(out[:int(sz[0])].cpu().numpy(), o.data)
    assert len(seen) >= 2                                          # the cases do not all choose alike
    # rates measured by the call itself: a valid choice (0 / 1 per table) and a positive estimate
    rec = torch.empty_like(d)
    choice, est = ctx.select_compressors(d, out, sizes, 25.0, rec=rec)
    assert set(np.unique(choice)) <= {0, 1} and np.all(est > 0)
    # a context without both compressors cannot select
    plain = b.Context(b.make_config(b.F32, T, B, D, R, S, 12))
    plain.set_error_bounds(eb=ebs)
    with pytest.raises(b.DlcError):
        plain.select_compressors(d, out, sizes, 25.0, tc, td)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_rows_with_equal_hashes_still_get_the_first_occurrence(dtype):
    """With every multiplier of the row hash zero all rows of a table hash alike: every repeated row but the
    repeats of the table's first row meets a different row under its hash.  References and container must be the
    oracle's all the same (the references are defined by content, not by the hash)."""
    import torch
    for (T, B, D, S) in ((2, 300, 16, 64), (1, 130, 40, 128), (1, 70, 260, 64)):
        print("equal hashes", T, B, D, S, np.dtype(dtype).name, flush=True)
        x = _lookups(T, B, D, 33 + D, rows=25, dtype=dtype)
        big = 1e9 if dtype == np.float32 else 6e4
        x[0, 3, 1] = big
        x[0, 8] = x[0, 3]                       # a repeated row with an escape
        x[0, 11] = x[0, 3]
        x[0, 11, 1] = -big                      # the escape's raw bits differ: not a repeat
        ebs = np.full(T, 1e-3 if dtype == np.float32 else 4e-3, np.float32)
        ctx, d, out, data, sizes = _compress(x, ebs, S, zero_hash=True)
        refs = ctx.read_row_refs()
        for t in range(T):
            s_t, _ = oracle.quantize(x[t:t + 1], float(ebs[t]), R)
            assert np.array_equal(refs[t], first_occurrence(x[t:t + 1], s_t)[0]), t
        o = oracle.compress(x, ebs, R, S, 12, row_match=True)
        assert o.rc == 0 and np.array_equal(sizes, o.sizes) and np.array_equal(data, o.data)
        rec = torch.full_like(d, 7.0)
        assert ctx.decompress(out, int(sizes[0]), rec) == 0 and ctx.sync_status() == 0
        rc, orec = oracle.decompress(o.data, x.shape, x.dtype)
        u = np.uint32 if dtype == np.float32 else np.uint16
        assert rc == 0 and np.array_equal(rec.cpu().numpy().view(u), orec.view(u))


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("T,B,D", [(2, 9, 256), (1, 131, 272), (3, 70, 1008), (1, 65, 1024), (1, 37, 1040), (2, 21, 2064),
                                   (1, 8300, 64), (1, 1, 512)])
def test_long_rows_and_few_rows(T, B, D, dtype):
    """Rows that are the work of a team of lanes (one piece a lane, the last lanes without one, several pieces a lane) and
    batches whose rows are spread over more wavefronts: references and container are the oracle's."""
    print("long rows", T, B, D, np.dtype(dtype).name, flush=True)
    x = _lookups(T, B, D, B + D, rows=max(2, B // 3), dtype=dtype)
    if B > 4:
        big = 1e9 if dtype == np.float32 else 6e4
        x[0, 1, D - 1] = big
        x[0, 2] = x[0, 1]                       # a repeated row with an escape in its last element
        x[0, 3] = x[0, 1]
        x[0, 3, D - 1] = -big                   # the escape's raw bits differ: not a repeat
        x[0, 4, 0] += 1
    ebs = np.full(T, 1e-3 if dtype == np.float32 else 4e-3, np.float32)
    ctx, d, out, data, sizes = _compress(x, ebs, 64)
    refs = ctx.read_row_refs()
    for t in range(T):
        s_t, _ = oracle.quantize(x[t:t + 1], float(ebs[t]), R)
        assert np.array_equal(refs[t], first_occurrence(x[t:t + 1], s_t)[0]), t
    o = oracle.compress(x, ebs, R, 64, 12, row_match=True)
    assert o.rc == 0 and np.array_equal(sizes, o.sizes) and np.array_equal(data, o.data)


@pytest.mark.parametrize("T,B,D,on", [
    (3, 301, 40, [1, 0, 1]),                 # blocks padded to 16 bytes; a table without references in between
    (2, 4500, 16, [0, 1]),                   # more references than a thread loads back to back
    (3, 64, 16, [0, 0, 0]),                  # none at all
    (1, 41000, 8, [1]),                      # several work-groups share them
    (70, 130, 12, [1] * 70),                 # a container of many tables, small blocks
])
def test_references_at_the_end_of_the_container(T, B, D, on):
    """The coding launch writes the references, too: the container is the oracle's; one byte less capacity is refused and leaves
    the context as it was."""
    import torch
    from paper_2407_04272_amd import binding as b
    print("references in place", T, B, D, flush=True)
    x = _lookups(T, B, D, 7 * B + T, rows=max(3, B // 5))
    ebs = np.full(T, 1e-3, np.float32)
    ctx, d, out, data, sizes = _compress(x, ebs, 64, flags_per_table=on)
    o = oracle.compress(x, ebs, R, 64, 12, row_match=np.array(on, bool))
    assert o.rc == 0 and np.array_equal(sizes, o.sizes) and np.array_equal(data, o.data)
    sz = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    for capacity, ok in ((data.size, True), (data.size - 1, False), (data.size - 4 * B, False), (data.size, True)):
        out.fill_(0xA5)
        rc = ctx.compress(d, out, sz, capacity=capacity)
        status = ctx.sync_status()
        h = out.cpu().numpy()
        assert np.all(h[capacity:] == 0xA5), capacity
        if ok:
            assert rc == 0 and status == 0 and np.array_equal(h[:data.size], data)
        else:
            assert status == b.ECAPACITY and int(sz[0]) == 0, capacity


def test_more_escapes_in_a_group_than_the_encoder_remembers():
    """More than 128 escapes in one group, many of them in rows that are stored as references: the records are those
    of the coded rows only (the encoder's second look at such a group goes by the symbol plane, where an element of a
    referencing row is marked as such)."""
    x = _lookups(1, 130, 64, 4, rows=40)
    x.reshape(-1)[::53] = 1e9                   # 157 escapes in the one group of 8320 elements
    x[0, 100:130] = x[0, 10:40]                 # repeated rows, escapes and all
    ebs = np.full(1, 1e-2, np.float32)
    ctx, d, out, data, sizes = _compress(x, ebs, 256)
    o = oracle.compress(x, ebs, R, 256, 12, row_match=True)
    assert o.rc == 0 and np.array_equal(sizes, o.sizes) and np.array_equal(data, o.data)
