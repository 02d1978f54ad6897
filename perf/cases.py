"""What this library is used for, as measurable cases: the pure-read probe, single GEMVs, multi-column
GEMVs, decode sweeps of whole models (one token, several tokens per weight pass on the vector ALUs
and on the matrix cores, chained by dependencies) and the per-use copy endpoint, each through the
entry points of paper_2608_12114_amd.wsr.

Inputs come from torch's seeded generator: 16-bit weights N(0, 0.02), activations N(0, 1), 4-bit
codes uniform with block scales U[0.005, 0.02], int8 codes uniform with row scales U[2.5e-4, 1e-3],
probe values U[-1, 1) on the 2^-23 grid.  Weights and scales of a state lie in one device buffer,
each tensor at a 2 MiB boundary, as an engine that loads a checkpoint into one allocation holds
them; all outputs lie in one tensor, matrix after matrix, each (tokens, rows)."""
import torch

GEMV_FMTS = ("f16", "bf16", "q4", "i8")
ARENA_ALIGN = 2 << 20
EXACT_CHUNK = 1 << 26              # weights taken to 64 bits at a time
STAGE_BYTES = 128 << 20            # two staging halves of 64 MiB


def _model(name, kind, fmt, layers, d, q, kv, ffn, vocab, tokens=1, chained=False):
    return {"name": name, "kind": kind, "fmt": fmt, "layers": layers, "d": d, "q": q, "kv": kv, "ffn": ffn,
            "vocab": vocab, "tokens": tokens, "chained": chained}


def listed():
    return [
        # the pure-read reference every bandwidth figure is held against: 1 GiB of fp32
        {"name": "probe_1gib", "kind": "probe", "n": 1 << 28},
        # the smallest call of the size sweep: one small projection, latency bound
        {"name": "gemv_bf16_256x4096", "kind": "gemv", "fmt": "bf16", "M": 256, "K": 4096, "count": 1, "columns": 1},
        # the single fp16 GEMV as a program without the sweep issues it: 32 matrices, a call for each
        {"name": "gemv_f16_4096x4096_x32", "kind": "gemv", "fmt": "f16", "M": 4096, "K": 4096, "count": 32, "columns": 1},
        # the matched protocol's int8 matrix with four speculative columns per weight read
        {"name": "cols_i8_12288x7168_t4", "kind": "gemv", "fmt": "i8", "M": 12288, "K": 7168, "count": 4, "columns": 4},
        # batch-1 decode of the 8B model in 4-bit blocks: every weight byte once per token
        _model("sweep_q4_8b", "sweep", "q4", 32, 4096, 4096, 1024, 14336, 128256),
        # the same token with the dependencies of a real decode step: a launch for each dependency group
        _model("sweep_q4_8b_chained", "sweep", "q4", 32, 4096, 4096, 1024, 14336, 128256, chained=True),
        # batch-1 decode of the 70B model in bf16, 6 of its 80 layers and the head
        _model("sweep_bf16_70b", "sweep", "bf16", 6, 8192, 8192, 1024, 28672, 128256),
        # batch-1 decode of the 72B model in int8, 4 of its 80 layers and the head: rows of 29,568 codes,
        # no whole number of the kernels' steps
        _model("sweep_i8_72b", "sweep", "i8", 4, 8192, 8192, 1024, 29568, 152064),
        # 8 sequences per weight pass with the single-token bits (the batched sweep on the vector ALUs)
        _model("batched_q4_8b_t8", "batched", "q4", 32, 4096, 4096, 1024, 14336, 128256, tokens=8),
        # 16 sequences per weight pass on the matrix cores, 4-bit and 16-bit
        _model("mma_q4_8b_t16", "mma", "q4", 32, 4096, 4096, 1024, 14336, 128256, tokens=16),
        _model("mma_bf16_70b_t16", "mma", "bf16", 4, 8192, 8192, 1024, 28672, 128256, tokens=16),
        # the per-use copy endpoint: one layer's bf16 weights in pinned host memory, copied as they are used
        _model("staged_bf16_8b_layer", "staged", "bf16", 1, 4096, 4096, 1024, 14336, 0),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _draw_model(rng, kind):
    """A decoder of drawn sizes: widths are multiples of 64 (heads) and of 32 (feed-forward), odd
    multiples among them; the layer count is what the case's weight bytes allow."""
    fmt = rng.choice(GEMV_FMTS)
    d = 64 * round(_log(rng, 512, 2560 if kind == "staged" else 8192) / 64)
    kv = rng.choice((d, max(64, d // 4), max(64, d // 8 // 64 * 64)))
    ffn = 32 * round(d * rng.uniform(2.0, 4.0) / 32)
    vocab = rng.choice((0, int(_log(rng, 1000, 60000))))
    per = 2 * d * d + 2 * kv * d + 3 * ffn * d
    byte = {"f16": 2.0, "bf16": 2.0, "q4": 0.5625, "i8": 1.0}[fmt]
    most = {"sweep": 6e9, "batched": 1.5e9, "mma": 4e9, "staged": 3e8}[kind]
    want = _log(rng, most / 200, most)
    layers = max(1, min(40, round(want / (per * byte))))
    if kind == "staged":
        vocab, layers = 0, 1
    tokens = {"sweep": 1, "staged": 1, "batched": rng.choice((2, 4, 8, 8, 16)), "mma": rng.randint(2, 16)}[kind]
    return {"kind": kind, "fmt": fmt, "layers": layers, "d": d, "q": d, "kv": kv, "ffn": ffn, "vocab": vocab,
            "tokens": tokens, "chained": kind in ("sweep", "batched", "mma") and rng.random() < 0.4}


def draw(rng):
    kind = rng.choice(("probe", "gemv", "gemv", "cols", "sweep", "sweep", "sweep", "batched", "batched", "mma", "mma",
                       "staged"))
    if kind == "probe":
        return {"kind": "probe", "n": int(_log(rng, 1 << 16, 1 << 28))}
    if kind in ("gemv", "cols"):
        fmt = rng.choice(GEMV_FMTS)
        K = 32 * round(_log(rng, 512, 32768) / 32)
        M = int(_log(rng, 64, 140800))
        M = max(16, min(M, (1 << 30) // (2 * K)))
        count = rng.choice((1, 4, 12)) if M * K < (1 << 27) else 1
        columns = 1 if kind == "gemv" else rng.choice((2, 4, 8, 16) if fmt in ("f16", "bf16") else (2, 4, 8))
        return {"kind": "gemv", "fmt": fmt, "M": M, "K": K, "count": count, "columns": columns}
    return _draw_model(rng, kind)


# ---- inputs, from the seed alone -------------------------------------------------------------------

def _matrices(case):
    """[(M, K, activation id)] in the order the entry points take them."""
    if case["kind"] == "gemv":
        return [(case["M"], case["K"], i) for i in range(case["count"])]
    d, q, kv, ffn, out = case["d"], case["q"], case["kv"], case["ffn"], []
    for l in range(case["layers"]):
        a = 4 * l
        out += [(q, d, a), (kv, d, a), (kv, d, a), (d, q, a + 1), (ffn, d, a + 2), (ffn, d, a + 2), (d, ffn, a + 3)]
    if case["vocab"]:
        out.append((case["vocab"], d, 4 * case["layers"]))
    return out


def _tokens(case):
    return case["columns"] if case["kind"] == "gemv" else case["tokens"]


def _sizes(fmt, M, K):
    """Bytes of a matrix's weights or codes and of its scales."""
    if fmt == "q4":
        return M * K // 2, M * (K // 32) * 2
    if fmt == "i8":
        return M * K, M * 2
    return M * K * 2, 0


def _inputs(case, seed):
    """Weights and scales (views into one buffer) and activations of a case, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    fmt, mats, T = case["fmt"], _matrices(case), _tokens(case)
    half = torch.bfloat16 if fmt == "bf16" else torch.float16
    pad = lambda n: -(-n // ARENA_ALIGN) * ARENA_ALIGN  # noqa: E731
    arena = torch.empty(sum(pad(n) for M, K, _ in mats for n in _sizes(fmt, M, K)), dtype=torch.uint8, device="cuda")
    at, w, s, x = 0, [], [], {}

    def take(n):
        nonlocal at
        v = arena[at:at + n]
        at += pad(n)
        return v

    for M, K, a in mats:
        nw, ns = _sizes(fmt, M, K)
        b = take(nw)
        if fmt in ("q4", "i8"):
            b.view(torch.int32).random_(-(1 << 31), 1 << 31, generator=g)
            c = take(ns).view(torch.float16)
            lo, hi = (0.005, 0.02) if fmt == "q4" else (2.5e-4, 1e-3)
            c.copy_(torch.empty(c.numel(), dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=g))
            s.append(c)
        else:
            b = b.view(half)
            b.copy_(torch.empty(M * K, dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=g))
            s.append(None)
        w.append(b)
        if a not in x:
            x[a] = torch.empty((T, K), dtype=torch.float32, device="cuda").normal_(generator=g).to(half)
    return arena, w, s, x


def _probe_input(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(case["n"], dtype=torch.float32, device="cuda", generator=g).mul_(2).sub_(1)


# ---- the measured calls ----------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2608_12114_amd import wsr
    kind = case["kind"]
    if kind == "probe":
        n = case["n"]
        ws = torch.empty(wsr.wsr_probe_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        return {"kind": kind, "n": n, "buf": _probe_input(case, seed), "ws": ws, "y": torch.zeros(1, dtype=torch.float64, device="cuda")}
    arena, w, s, x = _inputs(case, seed)
    mats, T = _matrices(case), _tokens(case)
    code = {"f16": wsr.WSR_F16, "bf16": wsr.WSR_BF16, "q4": wsr.WSR_Q4, "i8": wsr.WSR_I8}[case["fmt"]]
    y = torch.zeros(sum(M for M, _, _ in mats) * T, dtype=torch.float32, device="cuda")
    st = {"kind": kind, "fmt": case["fmt"], "code": code, "T": T, "keep": (arena, x), "y": y}
    if kind == "staged":                   # the weights live in pinned host memory
        host = torch.empty(arena.numel(), dtype=torch.uint8, pin_memory=True)
        host.copy_(arena)
        view = lambda t: None if t is None else host.data_ptr() + (t.data_ptr() - arena.data_ptr())  # noqa: E731
        w, s = [view(t) for t in w], [view(t) for t in s]
        st["keep"] = (host, x)
        st["stage"] = torch.empty(STAGE_BYTES, dtype=torch.uint8, device="cuda")
        st["copy_stream"] = torch.cuda.Stream()
    specs, at, last = [], 0, None
    for (M, K, a), wm, sm in zip(mats, w, s):
        flags = wsr.WSR_MAT_AFTER_PREVIOUS if case.get("chained") and last not in (None, a) else 0
        last = a
        specs.append(dict(fmt=code, flags=flags, M=M, K=K, w=wm, scales=sm, x=x[a], x_tok_stride=2 * K,
                          y=y[at:at + T * M], y_tok_stride=4 * M))
        at += T * M
    if kind == "gemv":
        st["calls"] = specs
    else:
        st["mats"] = wsr.make_mats(specs)
        st["ws"] = torch.empty(wsr.wsr_sweep_workspace_bytes(st["mats"]), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    from paper_2608_12114_amd import wsr
    stream, kind = torch.cuda.current_stream(), st["kind"]
    if kind == "probe":
        wsr.wsr_probe_read(st["buf"], st["n"], st["y"], st["ws"], st["ws"].numel(), stream)
    elif kind == "gemv":
        T, fmt = st["T"], st["fmt"]
        for c in st["calls"]:
            M, K = c["M"], c["K"]
            if fmt in ("f16", "bf16"):
                if T == 1:
                    wsr.wsr_gemv_f16(c["w"], c["x"], c["y"], M, K, st["code"], stream)
                else:
                    wsr.wsr_gemv_f16_cols(c["w"], c["x"], 2 * K, c["y"], 4 * M, M, K, T, st["code"], stream)
            elif T == 1:
                (wsr.wsr_gemv_q4 if fmt == "q4" else wsr.wsr_gemv_i8)(c["w"], c["scales"], c["x"], c["y"], M, K, stream)
            else:
                (wsr.wsr_gemv_q4_cols if fmt == "q4" else wsr.wsr_gemv_i8_cols)(c["w"], c["scales"], c["x"], 2 * K, c["y"],
                                                                               4 * M, M, K, T, stream)
    elif kind == "sweep":
        wsr.wsr_decode_sweep(st["mats"], 1, st["ws"], st["ws"].numel(), stream)
    elif kind == "batched":
        wsr.wsr_decode_sweep_batched(st["mats"], st["T"], st["T"], st["ws"], st["ws"].numel(), stream)
    elif kind == "mma":
        wsr.wsr_decode_sweep_mma(st["mats"], st["T"], st["ws"], st["ws"].numel(), stream)
    else:
        wsr.wsr_sweep_staged(st["mats"], 0, st["stage"], STAGE_BYTES, stream, st["copy_stream"])
    return st["y"]


def work(case):
    if case["kind"] == "probe":
        return {"bytes": 4 * case["n"] + 8, "flops": case["n"]}
    mats, T = _matrices(case), _tokens(case)
    inputs = {a: 2 * K * T for _, K, a in mats}
    return {"bytes": sum(sum(_sizes(case["fmt"], M, K)) + 4 * M * T for M, K, _ in mats) + sum(inputs.values()),
            "flops": sum(2 * M * K * T for M, K, _ in mats)}


def tolerance(case):
    """The probe's values and partial sums are multiples of 2^-23 below 2^30: its fp64 sum is exact in
    any order.  All others are fp32 sums of exact products: four times the relative error against
    64-bit sums measured on the widest rows of each format (q4 products carry their block's bias
    through the sums, which costs them the most)."""
    if case["kind"] == "probe":
        return "exact"
    return {"rel": 3e-5 if case["fmt"] == "q4" else 1e-5}


def exact(case, seed):
    """The outputs in 64 bits, laid out as run() returns them."""
    if case["kind"] == "probe":
        return _probe_input(case, seed).double().sum().reshape(1)
    _, w, s, x = _inputs(case, seed)
    fmt, out = case["fmt"], []
    for (M, K, a), wm, sm in zip(_matrices(case), w, s):
        xt = x[a].double().t().contiguous()
        rows, parts = max(1, EXACT_CHUNK // K), []
        for r in range(0, M, rows):
            e = min(M, r + rows)
            if fmt == "q4":
                b = wm.view(M, K // 2)[r:e]
                q = torch.stack((b & 15, b >> 4), dim=-1).reshape(e - r, K // 32, 32)
                q = ((q ^ 8).to(torch.int16) - 8).double() * sm.view(M, K // 32)[r:e].double().unsqueeze(-1)
                wd = q.reshape(e - r, K)
            elif fmt == "i8":
                wd = wm.view(torch.int8).view(M, K)[r:e].double() * sm[r:e].double().unsqueeze(-1)
            else:
                wd = wm.view(M, K)[r:e].double()
            parts.append((wd @ xt).t())
        out.append(torch.cat(parts, dim=1).reshape(-1))
    return torch.cat(out)
