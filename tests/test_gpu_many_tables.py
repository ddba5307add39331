"""GPU: more than 512 tables of one to five groups each (a work-group of more wavefronts than groups a table), ragged last groups, and
numbers of tables around what one launch finishes the container of."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,D", [
    (513, 16, 8), (520, 64, 64), (520, 65, 64), (513, 128, 64), (520, 171, 65), (513, 256, 64), (515, 257, 64),   # groups of 4096
    (257, 513, 64),
])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_containers(T, B, D, dtype):
    from gpu_util import DeviceRun
    rng = np.random.default_rng(T + B)
    x = (rng.normal(0, 1, (T, B, D)) * np.exp(rng.uniform(-3, 0, T))[:, None, None]).astype(dtype)
    x[3] = 0.25                                           # one symbol
    x[5, 0, :3] = 1e4 if dtype == np.float16 else 1e9     # escapes
    ebs = np.full(T, 0.02, np.float32)
    g = DeviceRun(x, ebs, S=64)
    o = oracle.compress(x, ebs, S=64)
    assert g.status == 0 and np.array_equal(g.sizes, o.sizes) and np.array_equal(g.data, o.data)
    st, rec = g.decompress()
    rc, want = oracle.decompress(o.data, x.shape, x.dtype)
    assert st == 0 and rc == 0 and np.array_equal(rec.view(np.uint8), want.view(np.uint8))


@pytest.mark.parametrize("T,B,D,nd", [
    (1281, 16, 8, 1), (1536, 70, 64, 1), (1537, 16, 8, 1), (2900, 9, 8, 1),   # two and four wavefronts a table of one and two groups
    (100, 70, 64, 14), (128, 9, 8, 23), (107, 16, 8, 15),                     # ... with the containers' ends in the launch
    (768, 130, 64, 1), (769, 130, 64, 1), (1030, 200, 64, 1), (1540, 130, 64, 1),  # four and eight, of three and four groups
    (96, 130, 64, 8), (200, 200, 64, 4), (200, 130, 64, 6), (400, 200, 64, 2),
    (90, 270, 64, 6), (100, 600, 64, 4),                                      # more groups, several rounds
])
def test_rounds(T, B, D, nd):
    import torch
    from gpu_util import to_device
    from paper_2407_04272_amd import binding as b
    rng = np.random.default_rng(T + nd)
    x = (rng.normal(0, 1, (nd, T, B, D)) * np.exp(rng.uniform(-3, 0, T))[:, None, None]).astype(np.float32)
    x[:, 3] = 0.25                # one symbol
    x[:, 5, 0, :3] = 1e9          # escapes
    ebs = np.full(T, 0.02, np.float32)
    cfg = b.make_config(b.F32, T, B, D, 512, 64, 12, 0, num_dest=nd)
    ctx = b.Context(cfg)
    ctx.set_error_bounds(eb=ebs)
    cap = b.dlc_compress_bound(cfg)
    out = torch.empty(cap, dtype=torch.uint8, device="cuda")
    sizes = torch.full((1 + nd * T + (nd if nd > 1 else 0),), 77, dtype=torch.int64, device="cuda")
    dx = to_device(x if nd > 1 else x[0])
    want = [oracle.compress(x[d], ebs, S=64) for d in range(nd)]
    for call in range(2):
        out.fill_(0xA5)
        assert ctx.compress(dx, out, sizes, capacity=cap) == 0 and ctx.sync_status() == 0
        n, stride = sizes.cpu().numpy().astype(np.uint64), cap if nd == 1 else cap // nd // 256 * 256
        for d, o in enumerate(want):
            assert np.array_equal(out[d * stride:d * stride + o.data.size].cpu().numpy(), o.data), (call, d)
            assert np.array_equal(n[1 + d * T:1 + (d + 1) * T], o.sizes[1:])
