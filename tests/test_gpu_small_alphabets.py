"""Alphabets narrower than a wavefront with so many tables that a work-group builds four codebooks, one a wavefront: on every
compress path, against the oracle byte for byte."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -10)  # bins are exact multiples of 2^-9


def _payload(rng, T, B, D, R):
    """Every table with a spread of its own (the neighbours' counts differ), a few escapes, repeated rows."""
    spread = rng.uniform(0.3, R / 2, (T, 1, 1))
    rows = rng.standard_normal((T, (B + 2) // 3, D)) * spread
    x = np.take_along_axis(rows, rng.integers(0, rows.shape[1], (T, B, 1)), axis=1)
    x = np.clip(np.rint(x), 1 - R, R - 1) * (2 * float(EB))
    x = x.astype(np.float32)
    x.reshape(-1)[::997] = 3e4
    return x


@pytest.mark.parametrize("path", ["own", "own, apart", "rows", "carried", "sampled"])
@pytest.mark.parametrize("radius", [8, 16, 32])
@pytest.mark.parametrize("tables", [512, 514])
def test_four_codebooks_per_work_group(tables, radius, path):
    import torch
    from paper_2407_04272_amd import binding as b
    # (a table of up to 16 groups of the default path has a work-group to itself: 17 here.  So large a payload is one launch, whose codebooks a
    # work-group builds one at a time; with every kernel timed by itself they are the work of k_codebook, four a work-group)
    own = path.startswith("own")
    T, B, D, S = tables, 1025 if own else 70, 64, 64
    rng = np.random.default_rng(1000 * tables + radius)
    ebs = np.full(T, EB, np.float32)
    flags = {"own": 0, "own, apart": 0, "rows": b.FLAG_ROW_MATCH, "carried": b.FLAG_CARRY_CODEBOOK, "sampled": b.FLAG_SAMPLE_CODEBOOK}[path]
    cfg = b.make_config(b.F32, T, B, D, radius, S, 12, flags)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    launches = {"own": {"k_flow"}, "own, apart": {"k_hist", "k_codebook", "k_encode", "k_finalize"}}
    ctx.profile_enable({"own": 1, "own, apart": 2}.get(path, 0))
    cap = b.dlc_compress_bound(cfg)
    out = torch.empty(cap + 64, dtype=torch.uint8, device="cuda")
    sizes = torch.zeros(1 + T, dtype=torch.int64, device="cuda")
    prev = None
    for call in range(3 if path == "carried" else 2):  # (a later call finds what the first has left in the workspace)
        x = _payload(rng, T, B, D, radius)
        d = to_device(x)
        rec = torch.full_like(d, 7.0)
        out.fill_(0xA5)
        assert ctx.compress(d, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
        assert {k for k, (ms, n) in ctx.profile_read().items() if n} - {"k_decode"} == launches.get(path, set())
        h, n = out.cpu().numpy(), int(sizes[0])
        assert np.all(h[cap:] == 0xA5)
        o = oracle.compress(x, ebs, radius, S, 12, carry_hist=prev, want_hist=own or path == "carried",
                            row_match=True if path == "rows" else None, sample_codebook=path == "sampled")
        assert o.rc == 0
        assert n == o.data.size and np.array_equal(h[:n], o.data), call
        assert np.array_equal(sizes.cpu().numpy().astype(np.uint64), o.sizes), call
        if own or path == "carried":
            assert np.array_equal(ctx.read_histogram().reshape(T, -1), o.hist), call
        assert ctx.decompress(out, n, rec) == 0 and ctx.sync_status() == 0
        rc, orec = oracle.decompress(o.data, x.shape, x.dtype)
        assert rc == 0 and np.array_equal(rec.cpu().numpy().view(np.uint32), orec.view(np.uint32)), call
        if path == "carried":
            prev = o.hist
