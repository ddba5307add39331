"""The decoder of few groups (a group's chunks cut into parts that find their first codewords by themselves) against the
oracle: codes that fall into step at once, late and never, every remainder of a group, damaged and padded chunks."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -10)  # bins are exact multiples of 2^-9


def _bins(rng, kind, n):
    name, arg = kind
    if name == "fixed":     # `arg` symbols, equally often: codes of one length (a start off its grid stays off it) or of two
        b = rng.permutation(np.arange(n) % arg) - arg // 2
    elif name == "gauss":
        b = np.clip(np.rint(rng.standard_normal(n) * arg), -500, 500)
    elif name == "steep":   # codes of every length
        b = np.minimum(rng.geometric(0.5, n), arg)
    elif name == "escapes":  # `arg` in a thousand
        b = np.where(rng.random(n) < arg / 1000.0, 3000, np.rint(rng.standard_normal(n) * 3))
    else:                   # one symbol
        b = np.full(n, 7)
    return b.astype(np.float64)


KINDS = [("fixed", 32), ("fixed", 8), ("fixed", 23), ("gauss", 2), ("gauss", 7), ("gauss", 60), ("steep", 12), ("escapes", 20), ("one", 0)]


def _round_trip(x, S, radius=512):
    import torch
    from paper_2407_04272_amd import binding as b
    T, B, D = x.shape
    ebs = np.full(T, EB, np.float32)
    o = oracle.compress(x, ebs, radius, S, 12)
    assert o.rc == 0
    ctx = b.Context(b.make_config(b.F16 if x.dtype == np.float16 else b.F32, T, B, D, radius, S, 12, 0))
    rec = torch.full(x.shape, 7.0, dtype=torch.float16 if x.dtype == np.float16 else torch.float32, device="cuda")
    assert ctx.decompress(to_device(o.data), o.data.size, rec) == 0 and ctx.sync_status() == 0
    rc, orec = oracle.decompress(o.data, x.shape, x.dtype)
    u = np.uint16 if x.dtype == np.float16 else np.uint32
    assert rc == 0 and np.array_equal(rec.cpu().numpy().view(u), orec.view(u))


@pytest.mark.parametrize("kind", KINDS, ids=[f"{a}{c}" for a, c in KINDS])
@pytest.mark.parametrize("T,B,D,S,dtype", [
    (3, 128, 128, 256, np.float32),   # a whole group each
    (2, 40, 103, 256, np.float32),    # 16 turns and a part of one, n % 4 == 0
    (2, 211, 87, 256, np.float16),    # two groups, n odd
    (5, 23, 11, 256, np.float32),     # less than a turn
    (2, 96, 64, 64, np.float32),      # 16 turns of a whole group of short chunks, and half of one
    (301, 23, 49, 128, np.float32),   # more than 256 groups
])
def test_parts(kind, T, B, D, S, dtype):
    rng = np.random.default_rng(T * 1000 + B)
    _round_trip((_bins(rng, kind, T * B * D) * (2.0 * float(EB))).astype(dtype).reshape(T, B, D), S)


@pytest.mark.parametrize("G", [1, 4, 17])
def test_wide_radius(G):
    rng = np.random.default_rng(G)
    x = (np.clip(np.rint(rng.standard_normal((G, 128, 128)) * 500), -2047, 2047) * (2.0 * float(EB))).astype(np.float32)
    _round_trip(x, 256, 2048)


def test_a_chunk_that_ends_early_is_refused():
    import torch
    from paper_2407_04272_amd import binding as b
    T, B, D, S = 4, 128, 128, 256
    for kind in (("fixed", 32), ("gauss", 2), ("gauss", 60)):
        x = (_bins(np.random.default_rng(3), kind, T * B * D) * (2.0 * float(EB))).astype(np.float32).reshape(T, B, D)
        good = oracle.compress(x, np.full(T, EB, np.float32), 512, S, 12).data
        ctx = b.Context(b.make_config(b.F32, T, B, D, 512, S, 12, 0))
        off_chunk = int(good[48:104].view(np.uint64)[3])
        rec = torch.zeros((T, B, D), dtype=torch.float32, device="cuda")
        for chunk in (0, 30, 62, 64 * 3 + 17):
            bad = good.copy()
            bad[off_chunk + chunk] -= 1
            bad[off_chunk + chunk + 1] += 1
            assert oracle.decompress(bad, x.shape, x.dtype)[0] != 0
            assert ctx.decompress(to_device(bad), bad.size, rec) == 0 and ctx.sync_status() == b.ECORRUPT, chunk
        assert ctx.decompress(to_device(good), good.size, rec) == 0 and ctx.sync_status() == 0
        assert np.array_equal(rec.cpu().numpy().view(np.uint32), oracle.decompress(good, x.shape, x.dtype)[1].view(np.uint32))


@pytest.mark.parametrize("extra", [3, 90, 180])
def test_words_behind_a_chunks_codewords_do_not_matter(extra):
    """Every other chunk of a group padded with words of ones, also to more than the longest codes would fill."""
    import torch
    from paper_2407_04272_amd import binding as b
    B, D, S = 128, 128, 256
    x = (_bins(np.random.default_rng(8), ("gauss", 3), B * D) * (2.0 * float(EB))).astype(np.float32).reshape(1, B, D)
    c = oracle.compress(x, np.full(1, EB, np.float32), 512, S, 12).data
    q = c[48:104].view(np.uint64)
    words, off_chunk, off_payload, off_cb, total = (int(q[k]) for k in (1, 3, 4, 5, 6))
    cw = c[off_chunk:off_chunk + 64].astype(int)
    payload = c[off_payload:off_payload + 4 * words].view(np.uint32)
    pieces, at = [], 0
    for k in range(64):
        pieces.append(payload[at:at + cw[k]])
        at += cw[k]
        if k % 2:
            pieces.append(np.full(extra, 0xFFFFFFFF, np.uint32))
    assert at == words  # (no escapes)
    padded = np.concatenate(pieces)
    head = c[:off_payload].copy()
    head[off_chunk:off_chunk + 64] = cw + extra * (np.arange(64) % 2)
    new_cb = (off_payload + 4 * padded.size + 15) // 16 * 16
    hq = head[48:104].view(np.uint64)
    hq[1], hq[5], hq[6] = padded.size, new_cb, new_cb + total - off_cb
    d = head[128:128 + 56]
    d[24:].view(np.uint64)[0] += new_cb - off_cb
    d[24:].view(np.uint64)[3] = padded.size
    out = np.concatenate([head, padded.view(np.uint8), np.zeros(new_cb - off_payload - 4 * padded.size, np.uint8), c[off_cb:]])
    rc, orec = oracle.decompress(out, x.shape, x.dtype)
    assert rc == 0 and np.array_equal(orec, oracle.decompress(c, x.shape, x.dtype)[1])
    ctx = b.Context(b.make_config(b.F32, 1, B, D, 512, S, 12, 0))
    rec = torch.full(x.shape, 7.0, dtype=torch.float32, device="cuda")
    assert ctx.decompress(to_device(out), out.size, rec) == 0 and ctx.sync_status() == 0
    assert np.array_equal(rec.cpu().numpy().view(np.uint32), orec.view(np.uint32))


@pytest.mark.parametrize("kind", [("fixed", 23), ("gauss", 2), ("gauss", 60), ("steep", 12), ("escapes", 20)], ids=lambda k: f"{k[0]}{k[1]}")
@pytest.mark.parametrize("T,B,D,S,dtype", [
    (3, 64, 64, 256, np.float32), (3, 241, 17, 256, np.float32),  # 16 turns (a wavefront a group) and one element more
    (301, 90, 49, 128, np.float32),   # 18 turns, more than 256 groups
    (2, 192, 64, 128, np.float16),    # a whole group of chunks of 128, and half of one
    (512, 65, 64, 128, np.float32), (513, 65, 64, 128, np.float32),  # as many groups as there are parts for, and one more
])
def test_groups_of_few_turns(kind, T, B, D, S, dtype):
    rng = np.random.default_rng(T * 1000 + B)
    _round_trip((_bins(rng, kind, T * B * D) * (2.0 * float(EB))).astype(dtype).reshape(T, B, D), S)
