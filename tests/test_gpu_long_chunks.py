"""Chunks of more words than the kernels keep in LDS at a time (4 bits a symbol in a grid that fills the chip): the group
encoder's further passes over a group and the decoder's windows, against the oracle byte for byte."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -10)  # bins are exact multiples of 2^-9


def _payload(rng, kind, shape):
    name, arg = kind
    n = int(np.prod(shape))
    if name == "span":       # `arg` neighbouring symbols, all equally frequent: 33 words a chunk of 256 at 17, 43 at 40, 54 at 100
        b = rng.integers(0, arg, n).astype(np.float32) - arg // 2
    elif name == "wide":     # symbols outside the window on both sides: up to 96 words
        b = np.rint(rng.standard_normal(n, np.float32) * arg)
    else:                    # "escapes": long codes and `arg` escapes in a thousand elements
        b = np.rint(rng.standard_normal(n, np.float32) * 12)
        b[rng.random(n, np.float32) < arg / 1000.0] = 4000
    return (np.where(np.abs(b) < 3000, np.clip(b, -511, 511), b) * np.float32(2 * EB)).reshape(shape)


def _check(T, B, D, S, dtype, rows, x):
    import torch
    from paper_2407_04272_amd import binding as b
    x = x.astype(dtype)
    ebs = np.full(T, EB, np.float32)
    cfg = b.make_config(b.F16 if dtype == np.float16 else b.F32, T, B, D, 512, S, 12, b.FLAG_ROW_MATCH if rows else 0)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    cap = b.dlc_compress_bound(cfg)
    out = torch.full((cap + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    d = to_device(x)
    rec = torch.full_like(d, 7.0)
    for _ in range(2):  # (the second call finds what the first has left in the workspace)
        assert ctx.compress(d, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
    h, n = out.cpu().numpy(), int(sizes[0])
    assert np.all(h[cap:] == 0xA5)
    o = oracle.compress(x, ebs, 512, S, 12, row_match=True if rows else None)
    assert o.rc == 0 and n == o.data.size and np.array_equal(h[:n], o.data)
    assert ctx.decompress(out, n, rec) == 0 and ctx.sync_status() == 0
    rc, orec = oracle.decompress(o.data, x.shape, dtype)
    u = np.uint16 if dtype == np.float16 else np.uint32
    assert rc == 0 and np.array_equal(rec.cpu().numpy().view(u), orec.view(u))


KINDS = [("span", 17), ("span", 40), ("span", 100), ("wide", 90), ("escapes", 2), ("escapes", 30)]
_ids = [f"{a}{b}" for a, b in KINDS]


@pytest.mark.parametrize("kind", KINDS, ids=_ids)
@pytest.mark.parametrize("T,B,D,S,dtype", [
    (104, 17 * 128 - 3, 128, 256, np.float32),  # eight groups a work-group, sixteen wavefronts a compute unit
    (260, 150, 109, 256, np.float32),           # a work-group a table, more tables than compute units; n % 4 != 0, a ragged group
    (3, 20 * 128, 128, 256, np.float16),        # a small grid: longer columns, larger staging areas
    (530, 128, 64, 128, np.float32),            # chunks of 128: 17 to 48 words
])
def test_default_path(kind, T, B, D, S, dtype):
    if dtype == np.float16 and kind[0] == "escapes":
        kind = (kind[0], kind[1] / 10)
    rng = np.random.default_rng(T + kind[1] * 7919 if isinstance(kind[1], int) else T)
    _check(T, B, D, S, dtype, False, _payload(rng, kind, (T, B, D)))


@pytest.mark.parametrize("kind", KINDS, ids=_ids)
@pytest.mark.parametrize("T,B,D,dtype", [(258, 640, 128, np.float32), (520, 130, 128, np.float16)])  # eight and four groups a work-group
def test_row_matching(kind, T, B, D, dtype):
    rng = np.random.default_rng(T + kind[1])
    x = _payload(rng, kind, (T, (B + 1) // 2, D))
    _check(T, B, D, 256, dtype, True, np.take_along_axis(x, rng.integers(0, x.shape[1], (T, B, 1)), axis=1))


@pytest.mark.parametrize("kind", [("span", 5), ("span", 17), ("span", 100)], ids=["linear", "two_windows", "three_windows"])
def test_a_chunk_that_ends_early_is_refused(kind):
    """A word of one chunk booked to the next: the group's words are all there, the chunk's last codeword reaches past its end."""
    import torch
    from paper_2407_04272_amd import binding as b
    T, B, D, S = 260, 150, 128, 256
    x = _payload(np.random.default_rng(5), kind, (T, B, D))
    ebs = np.full(T, EB, np.float32)
    ctx = b.Context(b.make_config(b.F32, T, B, D, 512, S, 12, 0))
    ctx.set_error_bounds(eb=ebs)
    good = oracle.compress(x, ebs, 512, S, 12).data
    off_chunk = int(good[48:].view(np.uint64)[3])  # after escapes, words and the group table's offset
    rec = torch.zeros((T, B, D), dtype=torch.float32, device="cuda")
    assert ctx.decompress(to_device(good), good.size, rec) == 0 and ctx.sync_status() == 0
    for chunk in (0, 30, 62, 64 * 517 + 17):
        bad = good.copy()
        bad[off_chunk + chunk] -= 1
        bad[off_chunk + chunk + 1] += 1
        assert oracle.decompress(bad, x.shape, x.dtype)[0] != 0
        assert ctx.decompress(to_device(bad), bad.size, rec) == 0
        assert ctx.sync_status() == b.ECORRUPT, chunk
    assert ctx.decompress(to_device(good), good.size, rec) == 0 and ctx.sync_status() == 0
    assert np.array_equal(rec.cpu().numpy().view(np.uint32), oracle.decompress(good, x.shape, x.dtype)[1].view(np.uint32))


@pytest.mark.parametrize("T,groups,D,refs,wide,narrow,dtype", [
    (258, 2, 128, 41, 400, 32, np.float32),   # more than 256 work-groups: windows from 1920 words a group on
    (258, 2, 128, 41, 400, 32, np.float16),
    (130, 9, 128, 41, 400, 32, np.float32),   # eight groups a work-group, the ninth on its own
    (5, 3, 64, 36, 1000, 32, np.float32),    # a small grid: windows from 3072 words on
])
@pytest.mark.parametrize("side", [0, 1], ids=["first_row", "second_row"])
def test_lanes_without_bits_until_after_a_new_window(side, T, groups, D, refs, wide, narrow, dtype):
    """Two or four rows a turn: in every group one of them is a reference for the first `refs` turns, so its lanes have taken
    no bit when the others need their next window; all their words are still to come."""
    S, rows = 256, 256 // D  # (64 turns a group)
    rng = np.random.default_rng(T + wide + side)
    bins = rng.integers(0, narrow, (T, groups, 64, rows, D)) - narrow // 2
    bins[:, :, :, side] = rng.integers(0, wide, (T, groups, 64, D)) - wide // 2
    bins[:, :, :refs, side] = bins[:, :1, :1, side]  # one row of the table again and again
    x = (bins * (2 * float(EB))).astype(dtype).reshape(T, groups * 64 * rows, D)
    o = oracle.compress(x, np.full(T, EB, np.float32), 512, S, 12, row_match=True)
    q = o.data[48:104].view(np.uint64)  # escapes, words, then the sections' offsets
    ng = T * groups
    starts = o.data[int(q[2]):int(q[2]) + 4 * ng].view(np.uint32).astype(np.int64)
    words = np.diff(np.append(starts, int(q[1])))
    chunk = o.data[int(q[3]):int(q[3]) + 64 * ng].reshape(T, groups, rows, 64 // rows)[:, 1:].astype(np.int64)  # (a table's first group has the row itself)
    late, busy = chunk[:, :, side], np.delete(chunk, side, axis=2).reshape(T, groups - 1, -1)
    assert words.min() > (1920 if ng > 256 else 3072), words.min()  # windows
    assert np.all(late.max(-1) > 28)                                # a window and more to come,
    assert np.all(busy.max(-1) * 32 * refs >= 64 * 896)             # and the others need a new one before the first bit of it,
    assert busy.max(-1).min() <= 54                                 # in some group without a second one afterwards
    _check(T, groups * 64 * rows, D, S, dtype, True, x)


@pytest.mark.parametrize("T,B,D,dtype", [(520, 128, 128, np.float32), (270, 251, 128, np.float32), (520, 128, 128, np.float16)])
def test_groups_around_the_staging_area_of_two_wavefronts(T, B, D, dtype):
    """One or two groups a table, more than 512 in all, of 1536 to 2020 words: staged as a whole up to 1888."""
    S = 256
    rng = np.random.default_rng(T + B)
    share = np.linspace(0.0, 0.5, T)[:, None, None]  # of elements of sixteen symbols, else of eight
    bins = np.where(rng.random((T, B, D)) < share, rng.integers(0, 16, (T, B, D)), rng.integers(0, 8, (T, B, D))) - 4
    x = (bins * (2 * float(EB))).astype(dtype)
    o = oracle.compress(x, np.full(T, EB, np.float32), 512, S, 12)
    q = o.data[48:104].view(np.uint64)
    ng = T * ((B * D + 64 * S - 1) // (64 * S))
    words = np.diff(np.append(o.data[int(q[2]):int(q[2]) + 4 * ng].view(np.uint32).astype(np.int64), int(q[1])))
    for lo, hi in ((1536, 1856), (1856, 1888), (1888, 1920), (1920, 2100)):
        assert np.any((words > lo) & (words <= hi)), (lo, hi, words.min(), words.max())
    _check(T, B, D, S, dtype, False, x)


@pytest.mark.parametrize("kind", KINDS, ids=_ids)
@pytest.mark.parametrize("flag", ["carried", "sampled"])
@pytest.mark.parametrize("T,B,D,S,dtype", [
    (3, 700, 100, 256, np.float32),   # five groups a table, the last ragged
    (2, 1500, 37, 128, np.float32),   # n % 4 == 0 with an odd row length
    (3, 333, 41, 64, np.float32),     # n % 4 != 0: scalar loads
    (2, 700, 100, 256, np.float16),
    (2, 333, 41, 128, np.float16),
])
def test_single_pass(kind, flag, T, B, D, S, dtype):
    """Groups of more words than a column holds on the single-pass path: walked on from a mark, once and several times."""
    import torch
    from paper_2407_04272_amd import binding as b
    if dtype == np.float16 and kind[0] == "escapes":
        kind = (kind[0], kind[1] / 10)
    print("single pass", flag, kind, T, B, D, S, np.dtype(dtype).name, flush=True)
    x = _payload(np.random.default_rng(int(T + 31 * S + kind[1])), kind, (T, B, D)).astype(dtype)
    ebs = np.full(T, EB, np.float32)
    cfg = b.make_config(b.F16 if dtype == np.float16 else b.F32, T, B, D, 512, S, 12, b.FLAG_CARRY_CODEBOOK if flag == "carried" else b.FLAG_SAMPLE_CODEBOOK)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    cap = b.dlc_compress_bound(cfg)
    out = torch.full((cap + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    d = to_device(x)
    prev = None
    for call in range(3):
        assert ctx.compress(d, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
        h, n = out.cpu().numpy(), int(sizes[0])
        assert np.all(h[cap:] == 0xA5)
        if flag == "carried":
            o = oracle.compress(x, ebs, 512, S, 12, carry_hist=prev, want_hist=True)
            prev = o.hist
        else:
            o = oracle.compress(x, ebs, 512, S, 12, sample_codebook=True)
        assert o.rc == 0 and n == o.data.size and np.array_equal(h[:n], o.data), call
