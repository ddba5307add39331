"""Codebooks of up to 64 used symbols, which one wavefront builds in registers, and of more, at the counts where the order of merging is decided by ties or the
code lengths run into the limit: lengths and codewords against the oracle's, by symbol, on every launch that builds codebooks."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

R, EB = 512, np.float32(2.0 ** -10)  # bins are exact multiples of 2^-9


def _counts(rng, kind, n, total):
    """`n` counts of at least one that add up to `total`."""
    w = {"equal": np.ones(n), "two values": 1.0 + (np.arange(n) % 2), "falling": 1.0 / (1 + np.arange(n)),
         "doubling": 2.0 ** np.minimum(np.arange(n), 40), "fibonacci": 1.618 ** np.minimum(np.arange(n), 60),
         "bell": np.exp(-0.5 * ((np.arange(n) - n / 2) / (n / 7 + 0.3)) ** 2), "steps": 2.0 ** (np.arange(n) // 4),
         "random": rng.integers(1, 5, n).astype(float)}[kind]
    c = np.maximum(1, np.floor(w / w.sum() * (total - n)).astype(np.int64))
    c[np.argmax(c)] += total - c.sum()
    assert c.min() >= 1 and c.sum() == total
    return c


KINDS = ["equal", "two values", "falling", "doubling", "fibonacci", "bell", "steps", "random"]
USED = [1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 62, 63, 64, 65, 66, 100, 127, 128, 129, 130, 193, 400]


@pytest.mark.parametrize("lmax", [10, 12])
@pytest.mark.parametrize("B,S,times,launch", [
    (64, 256, 1, "k_table"),       # a group of 16 turns
    (256, 256, 1, "k_table"),      # one of 64
    (4100, 256, 1, "k_flow"),      # 17 groups: by the last of the work-groups that count the table
    (4100, 256, 1, "k_codebook"),  # the launches apart: from the counts in memory, a work-group a table
    (1025, 64, 3, "k_codebook"),   # 552 tables: four of them a work-group, a wavefront each where it can
])
def test_codebooks_of_every_shape(B, S, times, launch, lmax):
    from paper_2407_04272_amd import binding as b
    import torch
    rng = np.random.default_rng(B + lmax)
    D = 64
    cases = [(k, n) for k in KINDS for n in USED] * times
    T = len(cases)
    x = np.empty((T, B * D), np.float32)
    hists = []
    for t, (kind, n) in enumerate(cases):
        c = _counts(rng, kind, n, B * D)
        bins = np.sort(rng.choice(np.arange(-220, 220), n, replace=False))
        c = c[rng.permutation(n)]
        x[t] = rng.permutation(np.repeat(bins, c)).astype(np.float32) * (2 * EB)
        h = np.zeros(2 * R, np.uint64)
        h[bins + R] = c
        hists.append(h)
    ctx = b.Context(b.make_config(b.F32, T, B, D, R, S, lmax))
    ctx.set_error_bounds(eb=np.full(T, EB, np.float32))
    ctx.profile_enable(2 if launch == "k_codebook" else 1)
    d = to_device(x.reshape(T, B, D))
    out = torch.empty(b.dlc_compress_bound(ctx.cfg), dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    assert ctx.compress(d, out, sizes) == 0 and ctx.sync_status() == 0
    assert ctx.profile_read()[launch][1] == 1
    ln, code = ctx.read_codebook()
    assert np.array_equal(ctx.read_histogram().reshape(T, -1), np.array(hists))
    for t in range(T):
        oln, ocode, _, _ = oracle.codebook(hists[t], lmax)
        assert np.array_equal(ln[t], oln), cases[t]
        assert np.array_equal(code[t].astype(np.uint32) & 0xFFF, np.where(oln > 0, ocode, 0)), cases[t]


def test_a_count_too_large_to_share_a_word_with_its_lane():
    """2^26 elements of one symbol and a few others: the counts are sorted as 64-bit keys."""
    from paper_2407_04272_amd import binding as b
    import torch
    B, D = 1 << 20, 68
    d = torch.zeros((1, B, D), dtype=torch.float32, device="cuda")
    few = torch.arange(1, 18, device="cuda").repeat_interleave(torch.arange(1, 18, device="cuda") % 5 + 1)
    d.view(-1)[: few.numel()] = few.float() * float(2 * EB)
    ctx = b.Context(b.make_config(b.F32, 1, B, D, R, 256, 12))
    ctx.set_error_bounds(eb=np.full(1, EB, np.float32))
    out = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(2, dtype=torch.int64, device="cuda")
    assert ctx.compress(d, out, sizes) == 0 and ctx.sync_status() == 0
    h = ctx.read_histogram().reshape(-1)
    assert int(h[R]) == B * D - few.numel() > 1 << 26
    ln, _ = ctx.read_codebook()
    assert np.array_equal(ln[0], oracle.codebook(h, 12)[0])


@pytest.mark.parametrize("launch", ["k_flow", "k_codebook"])
def test_few_symbols_in_a_table_of_two_to_the_thirty_elements(launch):
    """Counts that leave no room for the wavefront's flag bits below them: 2 to 64 used symbols by the work-group's two queues."""
    from paper_2407_04272_amd import binding as b
    import torch
    B, D = 1 << 20, 1 << 10
    d = torch.empty((1, B, D), dtype=torch.float16, device="cuda")
    ctx = b.Context(b.make_config(b.F16, 1, B, D, R, 256, 12))
    ctx.set_error_bounds(eb=np.full(1, EB, np.float32))
    ctx.profile_enable(2 if launch == "k_codebook" else 1)
    out = torch.empty(1 << 29, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(2, dtype=torch.int64, device="cuda")
    rng = np.random.default_rng(5)
    for kind, n in (("two values", 2), ("steps", 3), ("doubling", 17), ("fibonacci", 33), ("falling", 63), ("bell", 64)):
        print("2^30", launch, kind, n, flush=True)
        few = _counts(rng, kind, n, 4096)  # the largest is as much larger as the rest of the table is long
        bins = np.sort(rng.choice(np.arange(-100, 100), n, replace=False))
        few = few[rng.permutation(n)]
        most = int(np.argmax(few))
        d.fill_(float(bins[most]) * float(2 * EB))
        d.view(-1)[:4096] = torch.from_numpy(np.repeat(bins, few) * (2 * float(EB))).to(torch.float16).cuda()
        h = np.zeros(2 * R, np.uint64)
        h[bins + R] = few
        h[bins[most] + R] += B * D - 4096
        assert ctx.compress(d, out, sizes) == 0 and ctx.sync_status() == 0
        assert ctx.profile_read()[launch][1] == 1
        assert np.array_equal(ctx.read_histogram().reshape(-1), h)
        ln, code = ctx.read_codebook()
        oln, ocode, _, _ = oracle.codebook(h, 12)
        assert np.array_equal(ln[0], oln)
        assert np.array_equal(code[0].astype(np.uint32) & 0xFFF, np.where(oln > 0, ocode, 0))
