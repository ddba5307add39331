"""Cases for measuring the library: the calls a training program makes through the binding, over the sizes it makes them at.

A case says which call (`do`), which compress path (`path`), and the payload: `tables` embedding tables of `batch` rows of
`dim` elements for each of `dest` receiving GPUs, in `dtype`, coded in chunks of `chunk` symbols.

  do      compress    one dlc_compress call (path "carried": the calls of two successive iterations)
          decompress  one dlc_decompress call on containers the library has made
          step        what an iteration does with a payload: the iteration's bounds, compress, decompress
          stats       the offline analysis of Section III-A (dlc_stats)
  path    own         every table's codebook from its own counts (no flag)
          carried     DLC_FLAG_CARRY_CODEBOOK
          sampled     DLC_FLAG_SAMPLE_CODEBOOK
          rows        DLC_FLAG_ROW_MATCH
  values  gauss       rows of N(0, sigma_t), sigma_t log-uniform in [1e-3, 1e-1], one per sample, Zipf(1.05)
          pooled      sums of 1 to 20 Laplace(0, 0.02) rows a sample, Zipf(1.2)
  bounds  medium      0.03 of the table's range for every table
          mixed       the three classes of the controller in turn: 0.05, 0.03 and 0.01 of the range
          fixed       1e-3 for every table
"""
import numpy as np
import torch

from paper_2407_04272_amd import binding as b

DEV = "cuda"
ROWS = 100_000    # rows of an embedding table
MAX_POOL = 20     # most rows summed for a sample
PHASE_END = 1000  # an iteration past the initial phase of the schedule


def _case(name, do, path, tables, batch, dim, dtype="f32", dest=1, chunk=256, values="gauss", bounds="medium"):
    return {"name": name, "do": do, "path": path, "tables": tables, "batch": batch, "dim": dim, "dtype": dtype,
            "dest": dest, "chunk": chunk, "values": values, "bounds": bounds}


def listed():
    return [
        # one table of 256 lookups, absolute bound 1e-3: the smallest workload of the benchmark, all launches and latency
        _case("one_table", "compress", "own", 1, 256, 16, bounds="fixed"),
        # an iteration at the batch size of the paper's small dataset: 26 tables, 128 samples
        _case("step_batch128", "step", "own", 26, 128, 32, bounds="mixed"),
        # the receiving side at the batch size of the paper's large dataset: 26 tables, 2048 samples
        _case("decompress_batch2048", "decompress", "own", 26, 2048, 64, bounds="mixed"),
        # the sending side of the benchmark's 26 MiB workload
        _case("compress_batch4096", "compress", "own", 26, 4096, 64, bounds="mixed"),
        # odd sizes: no table but the first starts on a 16-byte boundary, the last group of each is ragged
        _case("step_odd", "step", "own", 7, 2999, 37),
        # one rank's share of the all-to-all, 512 MiB, each direction: the benchmark's headline workload
        _case("compress_512M", "compress", "own", 128, 8192, 128),
        _case("decompress_512M", "decompress", "own", 128, 8192, 128),
        # the same size with each iteration coded with the codebook of the one before: two iterations
        _case("carried_512M", "compress", "carried", 128, 8192, 128),
        # multi-hot sums in half precision, codebook from a sample, an iteration in both directions
        _case("step_sampled_f16", "step", "sampled", 64, 16384, 128, dtype="f16", values="pooled"),
        # repeated rows stored as references, both directions
        _case("step_rows", "step", "rows", 64, 8192, 128),
        # the 512 MiB payload cut for 32 receiving GPUs, both directions
        _case("step_dest32", "step", "own", 128, 256, 128, dest=32),
        # the offline analysis of the 512 MiB payload
        _case("stats_512M", "stats", "own", 128, 8192, 128),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    do = rng.choice(["compress"] * 3 + ["decompress"] * 3 + ["step"] * 2 + ["stats"])
    paths = {"compress": ["own", "own", "carried", "sampled", "rows"], "decompress": ["own", "own", "rows"],
             "step": ["own", "sampled", "carried", "rows"], "stats": ["own"]}
    path = rng.choice(paths[do])
    dim = _log_int(rng, 8, 128)
    if path == "rows" or rng.random() < 0.6:  # (row matching wants multiples of four; most models' dimensions are)
        dim = max(8, dim // 4 * 4)
    tables = _log_int(rng, 1, 128)
    dest = rng.choice([2, 4, 8, 32]) if do != "stats" and rng.random() < 0.25 else 1
    batch = _log_int(rng, 64, 16384)
    batch = max(16, min(batch, 2 ** 26 // (tables * dim)) // dest)
    return {"do": do, "path": path, "tables": tables, "batch": batch, "dim": dim,
            "dtype": rng.choice(["f32", "f32", "f32", "f16"]), "dest": dest, "chunk": rng.choice([256, 256, 256, 128, 64]),
            "values": rng.choice(["gauss", "gauss", "pooled"]), "bounds": rng.choice(["medium", "mixed"])}


def _zipf(gen, rows, alpha, size):
    w = torch.arange(1, rows + 1, dtype=torch.float64, device=DEV) ** (-alpha)
    cdf = torch.cumsum(w, 0)
    u = torch.rand(size, dtype=torch.float64, device=DEV, generator=gen) * cdf[-1]
    return torch.clamp(torch.searchsorted(cdf, u), max=rows - 1)


def _payloads(case, seed, count):
    """`count` successive payloads [dest][table][batch][dim] of one set of embedding tables, and every table's bound."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    T, B, D, ND = case["tables"], case["batch"], case["dim"], case["dest"]
    dtype = torch.float16 if case["dtype"] == "f16" else torch.float32
    out = [torch.empty((ND, T, B, D), dtype=dtype, device=DEV) for _ in range(count)]
    sigma = 10.0 ** np.random.default_rng(seed).uniform(-3.0, -1.0, T)
    n = ND * B
    span = torch.empty(T, dtype=torch.float32, device=DEV)
    for t in range(T):
        if case["values"] == "pooled":
            u = torch.rand((ROWS, D), dtype=torch.float32, device=DEV, generator=gen) - 0.5
            table = -0.02 * torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.49999997))
        else:
            sd = 0.01 if case["bounds"] == "fixed" else float(sigma[t])
            table = torch.randn((ROWS, D), dtype=torch.float32, device=DEV, generator=gen) * sd
        for k in range(count):
            if case["values"] == "pooled":
                length = torch.randint(1, MAX_POOL + 1, (n,), device=DEV, generator=gen)
                idx = _zipf(gen, ROWS, 1.2, (n, MAX_POOL))
                acc = torch.zeros((n, D), dtype=torch.float32, device=DEV)
                for j in range(MAX_POOL):
                    acc += table[idx[:, j]] * (length > j).to(torch.float32)[:, None]
            else:
                acc = table[_zipf(gen, ROWS, 1.05, (n,))]
            out[k][:, t] = acc.view(ND, B, D).to(dtype)
            if k == 0:
                span[t] = acc.max() - acc.min()
    span = span.cpu().numpy()
    if case["bounds"] == "fixed":
        eb = np.full(T, 1e-3, np.float32)
    else:
        part = np.array([0.05, 0.03, 0.01])[np.arange(T) % 3] if case["bounds"] == "mixed" else np.full(T, 0.03)
        eb = (part * span).astype(np.float32)
    return out, eb


def _config(case):
    flags = {"own": 0, "carried": b.FLAG_CARRY_CODEBOOK, "sampled": b.FLAG_SAMPLE_CODEBOOK, "rows": b.FLAG_ROW_MATCH}[case["path"]]
    if case["do"] == "stats":
        flags |= b.FLAG_STATS_WORKSPACE
    return b.make_config(b.F16 if case["dtype"] == "f16" else b.F32, case["tables"], case["batch"], case["dim"],
                         chunk_symbols=case["chunk"], flags=flags, num_dest=case["dest"])


def _capacity(case):
    """Room for containers of up to 16 bits an element: a send buffer, all destinations' parts together."""
    per_dest = 2 * case["tables"] * case["batch"] * case["dim"] + 4096 * case["tables"] + 65536
    return case["dest"] * ((per_dest + 255) // 256 * 256)


def _ok(status):
    if status != b.OK:
        raise RuntimeError(b.dlc_strerror(status))


def prepare(case, seed):
    carried = case["do"] in ("compress", "step") and case["path"] == "carried"
    payloads, eb = _payloads(case, seed, 2 if carried else 1)
    T, ND = case["tables"], case["dest"]
    s = {"do": case["do"], "payloads": payloads, "ctx": b.Context(_config(case)), "eb": eb}
    if case["do"] == "stats":
        return s
    s["ctx"].set_error_bounds(eb=eb)
    s["sizes"] = [torch.zeros(1 + T if ND == 1 else 1 + ND * T + ND, dtype=torch.int64, device=DEV) for _ in payloads]
    s["containers"] = [torch.zeros(_capacity(case), dtype=torch.uint8, device=DEV) for _ in payloads]
    if case["do"] in ("decompress", "step"):
        s["rec"] = [torch.zeros_like(p) for p in payloads]
    if carried:  # the iteration before the first one measured: its codebook is in the context (a run's first builds its own)
        for _ in range(2):
            _ok(s["ctx"].compress(payloads[-1], s["containers"][-1], s["sizes"][-1]))
    if case["do"] == "decompress":
        _ok(s["ctx"].compress(payloads[0], s["containers"][0], s["sizes"][0]))
        _ok(s["ctx"].sync_status())
        # the receiver knows a container's size from the exchange of sizes; several containers lie at fixed displacements
        s["bytes"] = int(s["sizes"][0][0].item()) if ND == 1 else s["containers"][0].numel()
    return s


def run(state):
    ctx, do = state["ctx"], state["do"]
    if do == "stats":
        st = ctx.stats(state["payloads"][0], state["eb"])
        return {"min": np.array([x.min for x in st], np.float32), "max": np.array([x.max for x in st], np.float32),
                "rows": np.array([(x.n_rows, x.n_unique_raw, x.n_unique_quant) for x in st], np.int64)}
    if do == "decompress":
        _ok(ctx.decompress(state["containers"][0], state["bytes"], state["rec"][0]))
        return {"rec": state["rec"][0]}
    for k, payload in enumerate(state["payloads"]):
        if do == "step":
            ctx.set_error_bounds(eb=state["eb"], iteration=PHASE_END)
        _ok(ctx.compress(payload, state["containers"][k], state["sizes"][k]))
        if do == "step":
            _ok(ctx.decompress(state["containers"][k], state["containers"][k].numel(), state["rec"][k]))
    got = {"containers": state["containers"], "sizes": state["sizes"]}
    if do == "step":
        got["rec"] = state["rec"]
    return got


def work(case):
    n = case["tables"] * case["batch"] * case["dim"] * case["dest"]
    raw = n * (2 if case["dtype"] == "f16" else 4)
    if case["do"] == "stats":
        return {"bytes": raw, "flops": 0}
    coded = n * (0.2 if case["path"] == "rows" else 0.4)  # 3.2 bits an element, half of the rows once only
    passes = (2 if case["do"] == "step" else 1) * (2 if case["path"] == "carried" and case["do"] != "decompress" else 1)
    return {"bytes": passes * (raw + coded), "flops": 0}


def tolerance(case):
    # the format fixes every byte of a container, and a reconstruction is one rounded product of a whole number and the
    # table's bound: another correct implementation gives the same bits
    return "exact"


def _reconstruction(x, eb, radius=512):
    """What the quantiser keeps of x ([dest][table][batch][dim]) under the tables' bounds, in 64 bits."""
    e = torch.from_numpy(eb.astype(np.float64)).to(x.device).view(1, -1, 1, 1)
    out = torch.empty(x.shape, dtype=torch.float64, device=x.device)
    for t in range(x.shape[1]):  # a table at a time
        v, et = x[:, t:t + 1].double(), e[:, t:t + 1]
        r = torch.round(v / (2.0 * et))
        rec = r * (2.0 * et)
        if x.dtype == torch.float16:
            rec = rec.to(torch.float32).to(torch.float16).double()
        coded = (r.abs() < radius) & ((v - rec).abs() <= et)
        out[:, t:t + 1] = torch.where(coded, rec, v)
    return out


def exact(case, seed):
    if case["do"] == "compress":
        return None  # bytes of containers and their sizes
    carried = case["do"] == "step" and case["path"] == "carried"
    payloads, eb = _payloads(case, seed, 2 if carried else 1)
    if case["do"] == "stats":
        x = payloads[0][0].double().flatten(1)
        return {"min": x.amin(1).cpu().numpy(), "max": x.amax(1).cpu().numpy(), "rows": None}
    recs = [_reconstruction(p, eb) for p in payloads]
    if case["do"] == "decompress":
        return {"rec": recs[0]}
    return {"containers": [None for _ in recs], "sizes": [None for _ in recs], "rec": recs}
