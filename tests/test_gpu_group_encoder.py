"""The encoders of whole groups (small tables in one launch, larger ones from the symbol plane) at the sizes and symbol
distributions where their branches change, against the oracle byte for byte.  (Groups that are walked more than once:
test_gpu_long_chunks.py.)"""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -10)  # bins are exact multiples of 2^-9


def _bins(rng, kind, shape):
    """A bin per element; NaN marks an escape."""
    n = int(np.prod(shape))
    name, arg = kind
    if name == "span":      # `arg` neighbouring symbols, all equally frequent
        b = rng.integers(0, arg, n).astype(np.float64) - arg // 2
    elif name == "steep":   # codes of every length up to the limit, four of them more than 32 bits together now and then
        b = np.minimum(rng.geometric(0.5, n), arg).astype(np.float64) - 5
        b[::509] = rng.integers(20, 31, b[::509].size)
    elif name == "escapes":  # `arg` escapes in every 4096 elements
        b = np.rint(rng.standard_normal(n) * 2)
        for s in range(0, n, 4096):
            k = min(arg, n - s)
            b[s + rng.choice(min(4096, n - s), min(k, min(4096, n - s)), replace=False)] = np.nan
    else:                   # far outside the window, both sides
        b = np.rint(rng.standard_normal(n) * arg)
    return b.reshape(shape)


def test_profile_names_the_kernels_that_ran():
    import torch
    from paper_2407_04272_amd import binding as b
    for batch, ran in ((256, {"k_table", "k_finalize"}), (20 * 64, {"k_hist", "k_codebook", "k_encode", "k_finalize"})):
        cfg = b.make_config(b.F32, 2, batch, 64, 512, 64, 12, 0)
        ctx = b.Context(cfg)
        ctx.set_error_bounds(eb=np.full(2, EB, np.float32))
        x = torch.randn((2, batch, 64), device="cuda") * 0.01
        out = torch.empty(b.dlc_compress_bound(cfg), dtype=torch.uint8, device="cuda")
        sizes = torch.zeros(3, dtype=torch.int64, device="cuda")
        for level, want in ((1, ran & {"k_table", "k_encode"}), (2, ran)):
            ctx.profile_enable(level)
            assert ctx.compress(x, out, sizes) == 0 and ctx.sync_status() == 0
            prof = ctx.profile_read()
            assert {k for k, (ms, n) in prof.items() if n} == want
            assert all(n == 1 and ms > 0 for k, (ms, n) in prof.items() if k in want)


def _check(T, B, D, S, R, dtype, nd, kind, seed):
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(seed)
    bins = _bins(rng, kind, (nd, T, B, D))
    lim = R - 1
    x = np.where(np.isnan(bins), np.inf, np.clip(bins, -lim, lim) * (2 * float(EB))).astype(dtype)
    ebs = np.full(T, EB, np.float32)
    cfg = b.make_config(b.F16 if dtype == np.float16 else b.F32, T, B, D, R, S, 12, 0, num_dest=nd)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    cap = b.dlc_compress_bound(cfg)
    stride = (cap // nd) & ~255 if nd > 1 else cap
    out = torch.full((cap + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + nd * T + (nd if nd > 1 else 0), dtype=torch.int64, device="cuda")
    d = to_device(x if nd > 1 else x[0])
    rec = torch.full_like(d, 7.0)
    for _ in range(2):  # (the second call finds what the first has left in the workspace)
        assert ctx.compress(d, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
    h = out.cpu().numpy()
    sz = sizes.cpu().numpy()
    assert np.all(h[cap:] == 0xA5)
    assert ctx.decompress(out, cap if nd > 1 else int(sz[0]), rec) == 0 and ctx.sync_status() == 0
    r = rec.cpu().numpy().reshape(x.shape)
    u = np.uint16 if dtype == np.float16 else np.uint32
    hist = ctx.read_histogram().reshape(nd, T, -1)
    for p in range(nd):
        o = oracle.compress(x[p], ebs, R, S, 12, want_hist=True)
        assert o.rc == 0
        nbytes = int(sz[1 + nd * T + p]) if nd > 1 else int(sz[0])
        assert nbytes == o.data.size and np.array_equal(h[p * stride:p * stride + nbytes], o.data), p
        assert np.array_equal(hist[p], np.asarray(o.hist).reshape(T, -1)), p
        rc, orec = oracle.decompress(o.data, x[p].shape, dtype)
        assert rc == 0 and np.array_equal(r[p].view(u), orec.view(u)), p


@pytest.mark.parametrize("groups", [1, 2, 3, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("tables,ragged", [(3, False), (2, True), (300, False), (130, True)])
def test_groups_per_table(groups, tables, ragged):
    B, D = (64 * groups - 1, 61) if ragged else (64 * groups, 64)
    _check(tables, B, D, 64, 512, np.float32, 1, ("span", 17), groups * 1000 + tables)


@pytest.mark.parametrize("kind", [("span", 1), ("span", 2), ("span", 44), ("span", 45), ("span", 46), ("span", 62), ("span", 63),
                                  ("span", 64), ("span", 65), ("span", 250), ("steep", 40), ("escapes", 1), ("escapes", 128),
                                  ("escapes", 129), ("escapes", 4096), ("wide", 90)], ids=lambda k: f"{k[0]}{k[1]}")
@pytest.mark.parametrize("tables,batch,dim,chunk", [(2, 256, 64, 64), (2, 2048, 16, 128), (2, 2050, 33, 64), (1, 4400, 64, 256),
                                                    (270, 64, 64, 64)])
def test_symbol_distributions(kind, tables, batch, dim, chunk):
    _check(tables, batch, dim, chunk, 512, np.float32, 1, kind, batch)


@pytest.mark.parametrize("radius", [8, 64, 128, 2048])
@pytest.mark.parametrize("batch", [40, 1100])
def test_alphabets(radius, batch):
    for kind in (("wide", radius), ("span", 15)):
        _check(3, batch, 64, 64, radius, np.float32, 1, kind, radius)


@pytest.mark.parametrize("groups", [1, 6, 16, 20])
def test_half_precision_and_destinations(groups):
    _check(4, 64 * groups, 64, 64, 512, np.float16, 3, ("escapes", 20), groups)
    _check(65, 64 * groups - 7, 36, 64, 512, np.float16, 4, ("span", 30), groups)
