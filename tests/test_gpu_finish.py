"""Containers finished by the launch that codes the groups, against the oracle byte for byte: as many tables as a work-group
has threads and more, blocks of code lengths of every size, work-groups of both kinds of launches, several destinations,
capacities that end anywhere in the code-length blocks."""
import numpy as np
import pytest

import oracle
from gpu_util import to_device

pytestmark = pytest.mark.gpu

EB = np.float32(2.0 ** -10)


def _payload(rng, shape, wide):
    """Tables of few symbols, of many, with escapes (a block from symbol 0 on), of one symbol."""
    x = np.empty(shape, np.float32)
    for t in range(shape[-3]):
        k = t % 4 if wide else (t % 2) * 3
        n = shape[:-3] + shape[-2:]
        b = rng.standard_normal(n) * (2 if k == 0 else 70)
        if k == 1:
            b[..., ::7, :] = 4000
        x[..., t, :, :] = np.full(n, 5) if k == 3 else np.where(np.abs(b) < 3000, np.clip(np.rint(b), -511, 511), b)
    return x * np.float32(2 * EB)


@pytest.mark.parametrize("T,B,D,S,nd,wide", [
    (1, 40, 16, 256, 1, True), (5, 40, 16, 256, 1, True),      # four wavefronts a table
    (250, 40, 16, 256, 1, True), (254, 20, 16, 256, 1, False), (256, 20, 16, 256, 1, False),  # as many work-groups as run at a time, and more
    (9, 300, 64, 256, 1, True), (253, 129, 128, 64, 1, False),  # sixteen
    (300, 70, 16, 256, 1, True), (500, 33, 8, 64, 1, False), (512, 33, 8, 64, 1, False),  # eight
    (33, 20, 16, 64, 24, False), (128, 17, 8, 64, 17, True), (128, 17, 8, 64, 26, False),  # four; several containers, more than run at a time
    (5, 1100, 64, 64, 1, True), (70, 610, 32, 64, 1, True), (300, 610, 32, 64, 1, False), (20, 610, 32, 64, 3, True),  # three launches
])
def test_same_bytes(T, B, D, S, nd, wide):
    import torch
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(T * 7 + B)
    x = _payload(rng, (nd, T, B, D), wide)
    ebs = np.full(T, EB, np.float32)
    want = [oracle.compress(x[d], ebs, 512, S, 12) for d in range(nd)]
    cfg = b.make_config(b.F32, T, B, D, 512, S, 12, 0, num_dest=nd)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    dx = to_device(x if nd > 1 else x[0])
    cap = b.dlc_compress_bound(cfg)
    out = torch.full((cap + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sizes = torch.full((1 + nd * T + (nd if nd > 1 else 0),), 77, dtype=torch.int64, device="cuda")
    for call in range(3):  # (what a call leaves in the control words and records is there for the next)
        assert ctx.compress(dx, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
        h, n = out.cpu().numpy(), sizes.cpu().numpy()
        stride = cap if nd == 1 else cap // nd // 256 * 256
        for d in range(nd):
            o = want[d]
            assert np.array_equal(h[d * stride:d * stride + o.data.size], o.data), (call, d)
            assert np.array_equal(n[1 + d * T:1 + (d + 1) * T].astype(np.uint64), o.sizes[1:])
        assert n[0] == sum(o.data.size for o in want)
        out.fill_(0xA5)
    if nd == 1:
        total = want[0].data.size
        off_cb = int(want[0].data[48:104].view(np.uint64)[5])
        for short in (1, (total - off_cb) // 2, total - off_cb, total - off_cb + 4):
            out.fill_(0xA5)
            assert ctx.compress(dx, out, sizes, capacity=total - short) == 0 and ctx.sync_status() == b.ECAPACITY
            assert int(sizes[0]) == 0 and np.all(out.cpu().numpy()[total - short:] == 0xA5)
        assert ctx.compress(dx, out, sizes, capacity=total) == 0 and ctx.sync_status() == 0
        assert np.array_equal(out.cpu().numpy()[:total], want[0].data)
